"""Rows stay within SPG_OPT_LDS_LIMIT in either value type: no row of either
phase runs in a tier above the limit, and the product is the same."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu

NTIER = 10


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("limit", [1024, 2048, 4096, 8192, 16384, 32768, 65536])
def test_no_row_above_the_limit(limit, dtype):
    """Rows of C of 1 to some 12000 columns, narrow and wide, few and many of a size."""
    rng = np.random.default_rng(11)
    n, k = 400, 60000
    lens = np.concatenate([np.arange(1, 33), np.arange(1, 200, 3)])
    ci = np.concatenate([np.sort(rng.choice(n, size=int(l), replace=False)) for l in lens])
    A = gen.csr_from_rows_cols(lens.size, n, np.repeat(np.arange(lens.size), lens), ci,
                               rng.integers(-3, 4, size=ci.size).astype(dtype))
    span = np.where(np.arange(n) % 2 == 0, 900, k)
    bl = rng.integers(1, 90, size=n)
    bi = np.concatenate([np.sort(rng.choice(span[j], size=int(bl[j]), replace=False)) for j in range(n)])
    B = gen.csr_from_rows_cols(n, k, np.repeat(np.arange(n), bl), bi, rng.integers(-3, 4, size=bi.size).astype(dtype))
    rp, c, v, op = run_gpu(A, B, lds_limit=limit)
    compare(A, B, rp, c, v, exact=True)  # integers
    st = op.stats()
    for rows in (st["sym_rows"], st["num_rows"]):
        above = {cls: r for cls, r in enumerate(rows) if r and cls % NTIER < NTIER - 1 and (256 << cls % NTIER) > limit}
        assert not above
        assert sum(rows) > 0
