"""Rows of more than one wavefront, whose staged B pieces are cut into one range
per wavefront: chunks of one entry fewer and more than the group, B rows from
empty to longer than a range, all in every class of 128 lanes and more that
holds them.  Integer values: exact."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu


def _csr(nrows, k, lens, dtype, seed):
    rng = np.random.default_rng(seed)
    lens = np.resize(np.asarray(lens), nrows)
    cols = np.concatenate([np.sort(rng.choice(k, size=int(l), replace=False)) for l in lens])
    return gen.csr_from_rows_cols(nrows, k, np.repeat(np.arange(nrows), lens), cols,
                                  rng.integers(-3, 4, size=cols.size).astype(dtype))


@pytest.mark.parametrize("force", [-1, 5, 6, 7, 8, 16, 18, 25, 27])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("blens", [[1], [0, 0, 0, 5], [1, 2, 3, 4, 5, 0, 9], [0, 1500, 1, 0, 7, 3, 2]])
def test_ranges(blens, dtype, force):
    B = _csr(2100, 2000, blens, dtype, 1)
    A = _csr(24, 2100, [1, 63, 64, 65, 127, 128, 129, 256, 257, 513, 1023, 1024, 1025, 2049], dtype, 2)
    rp, c, v, _ = run_gpu(A, B, force_class=force)
    compare(A, B, rp, c, v, exact=True)
