"""Analysis of matrices whose rows are all long, or long side by side: rows of
65 to 512 entries by their own lanes or by a wavefront (whichever takes fewer
round trips), longer ones always by a wavefront, and the larger grid of
matrices of long rows on average."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu


def _rows(lens, n, seed):
    """Rows of the given lengths: runs of neighbouring columns from anywhere, in rotated order."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens)
    first = rng.integers(0, n, size=lens.size)
    at = np.arange(lens.sum()) - np.repeat(np.cumsum(lens) - lens, lens)
    ci = (np.repeat(first, lens) + 2 * at) % n  # n is odd: distinct up to n entries
    return gen.csr_from_rows_cols(lens.size, n, np.repeat(np.arange(lens.size), lens), ci,
                                  rng.integers(-2, 3, size=ci.size).astype(np.float64))


CASES = {
    "all 65": lambda m: np.full(m, 65),
    "all 128": lambda m: np.full(m, 128),
    "all 256": lambda m: np.full(m, 256),
    "all 257": lambda m: np.full(m, 257),
    "all 330": lambda m: np.full(m, 330),
    "all 513": lambda m: np.full(m, 513),
    "two in a wavefront": lambda m: np.where(np.arange(m) % 8 == 3, 100, 4),
    "six in a wavefront": lambda m: np.where(np.arange(m) % 16 < 6, 100, 4),
    "a hub among somewhat long ones": lambda m: np.where(np.arange(m) % 16 == 0, 700, 90),
    "the first rows": lambda m: np.where(np.arange(m) < 40, 600, 3),
}


@pytest.mark.parametrize("m", [3, 70, 3000])
@pytest.mark.parametrize("name", CASES)
def test_long_rows(name, m):
    lens = CASES[name](m)
    A, B = _rows(lens, 901, 1), _rows(np.full(901, 2), 5003, 2)  # long rows of A
    rp, c, v, op = run_gpu(A, B)
    compare(A, B, rp, c, v, exact=True)
    assert op.stats()["products"] == 2 * lens.sum()
    A, B = _rows(np.full(60, 3), m | 1, 3), _rows(np.resize(lens, m | 1), 5003, 4)  # long rows of B
    rp, c, v, _ = run_gpu(A, B)
    compare(A, B, rp, c, v, exact=True)
