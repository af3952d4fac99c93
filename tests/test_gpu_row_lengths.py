"""Row lengths at the edges of the analysis kernels: rows walked by one lane,
by a group of lanes, or by a whole wavefront (more than 64 or 128 entries),
matrices of few and of many rows, sorted and unsorted rows."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 7, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 511, 512, 513, 700]


def _rows(m, n, lens, seed, sort):
    rng = np.random.default_rng(seed)
    cols = [rng.choice(n, size=int(l), replace=False) for l in lens]
    if sort:
        cols = [np.sort(c) for c in cols]
    ci = np.concatenate(cols) if cols else np.zeros(0, dtype=np.int64)
    vals = rng.integers(-3, 4, size=ci.size).astype(np.float64)
    return gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), lens), ci, vals)


@pytest.mark.parametrize("sort", [True, False])
@pytest.mark.parametrize("m", [len(EDGES), 3001])
def test_long_and_short_rows_of_small_matrices(m, sort):
    """Integer values: exact.  Runs of neighbouring columns included (every
    fifth row of B is a contiguous range)."""
    lens = np.array([EDGES[i % len(EDGES)] if i % 37 < len(EDGES) else i % 5 for i in range(m)])
    A = _rows(m, 900, lens, 1, sort)
    blens = np.array([EDGES[(3 * i) % len(EDGES)] if i % 11 == 0 else i % 9 for i in range(900)])
    B = _rows(900, 5000, blens, 2, sort)
    ci = B.col_idx.copy()
    for j in range(0, 900, 55):
        s, e = B.row_ptr[j], B.row_ptr[j + 1]
        ci[s:e] = (np.arange(e - s) + 40 * j) % 5000 if sort is False else np.sort((np.arange(e - s) + 40 * j) % 5000)
    B = gen.Csr(B.m, B.n, B.row_ptr, ci, B.values)
    rp, c, v, _ = run_gpu(A, B)
    compare(A, B, rp, c, v, exact=True)


@pytest.mark.parametrize("extra", [[], [8, 9, 63, 64, 65, 66, 700]])
def test_many_short_rows(extra):
    """More than 2^17 rows of a few entries (one lane each), with and without
    rows that a whole wavefront takes, in both matrices."""
    m = (1 << 17) + 77
    rng = np.random.default_rng(5)
    lens = rng.integers(0, 5, size=m)
    for t, l in enumerate(extra):
        lens[(t * 19001 + 5) % m] = l
    rows = np.repeat(np.arange(m), lens)
    first = (np.arange(m) * 7919) % (m - 1000)
    start = np.repeat(np.cumsum(lens) - lens, lens)
    cols = first[rows] + (np.arange(rows.size) - start)
    A = gen.csr_from_rows_cols(m, m, rows, cols, rng.integers(-2, 3, size=rows.size).astype(np.float64))
    rp, c, v, _ = run_gpu(A, A)
    compare(A, A, rp, c, v, exact=True)
