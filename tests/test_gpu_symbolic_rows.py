"""Symbolic rows at the edges of the slot table and of the sparse direct table
(runs per B row, runs and A entries per row, words of the row's range,
occupied blocks), and numeric rows around full blocks.  Integer values: exact."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare, run_gpu

pytestmark = pytest.mark.gpu


def _b(nrows, k, runs, span, per_run, seed):
    """Rows of `runs` runs of `per_run` neighbouring columns in distinct words, spread over `span` words."""
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    words = k // 32
    for j in range(nrows):
        w0 = int(rng.integers(0, max(1, words - span + 1)))
        w = np.sort(rng.choice(span, size=min(runs, span), replace=False)) + w0
        if runs > 1:
            w[0], w[-1] = w0, w0 + span - 1
        w = np.unique(w)
        c = (w[:, None] * 32 + int(rng.integers(0, 33 - per_run)) + np.arange(per_run)[None, :]).ravel()
        rows.append(np.full(c.size, j))
        cols.append(c)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    return gen.csr_from_rows_cols(nrows, k, rows, cols, rng.integers(-3, 4, size=cols.size).astype(np.float64))


def _a(m, n, lens, seed):
    rng = np.random.default_rng(seed)
    lens = np.resize(np.asarray(lens), m)
    cols = np.concatenate([np.sort(rng.choice(n, size=int(l), replace=False)) for l in lens])
    return gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), lens), cols,
                                  rng.integers(-3, 4, size=cols.size).astype(np.float64))


@pytest.mark.parametrize("runs", [1, 5, 15, 16, 17])
@pytest.mark.parametrize("span", [17, 191, 192, 193, 1279, 1280, 1281])
def test_runs_and_spans(runs, span):
    """Rows of 1 to 66 entries of A: totals below, at and above one batch (320 runs) among them."""
    k = 32 * (span + 3)
    B = _b(150, k, runs, span, 3, 1)
    A = _a(260, 150, [1, 2, 3, 4, 19, 20, 21, 27, 33, 63, 64, 65, 66], 2)
    rp, c, v, _ = run_gpu(A, B)
    compare(A, B, rp, c, v, exact=True)


@pytest.mark.parametrize("blocks", [62, 63, 64, 65, 66, 130])
@pytest.mark.parametrize("force", [-1, 3, 4, 23, 24])
def test_blocks_of_a_row(blocks, force):
    """Occupied blocks around what one wavefront lists at once; also with the class forced."""
    k = 32 * 1000
    w = np.linspace(0, 999, blocks).astype(int)
    cols = (w * 32 + 7).astype(np.int64)
    per = 13
    parts = [cols[i:i + per] for i in range(0, blocks, per)]
    rows = np.concatenate([np.full(p.size, i) for i, p in enumerate(parts)])
    B = gen.csr_from_rows_cols(len(parts), k, rows, np.concatenate(parts), np.arange(1.0, blocks + 1))
    A = _a(40, len(parts), [len(parts), 1, max(1, len(parts) - 1)], 3)
    rp, c, v, _ = run_gpu(A, B, force_class=force)
    compare(A, B, rp, c, v, exact=True)


def test_two_waits():
    """A product past the one-wait bound, wide rows of few blocks."""
    B = _b(3000, 32 * 1260, 9, 1200, 3, 5)
    A = _a(28000, 3000, [3, 5, 9, 27], 6)
    rp, c, v, op = run_gpu(A, B)
    assert op.stats()["sym_waits"] == 2
    compare(A, B, rp, c, v, exact=True)


@pytest.mark.parametrize("per_run", [7, 8, 9, 31, 32])
@pytest.mark.parametrize("runs", [1, 2, 5, 9, 40])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_full_blocks(per_run, runs, dtype):
    """Blocks of 7 to 32 columns (the store of columns changes at 8 per block), narrow rows."""
    B = _b(60, 32 * 48, runs, max(runs, 2) if runs > 1 else 1, per_run, 7).astype(dtype)
    A = _a(700, 60, [1, 2, 3, 8, 20], 8).astype(dtype)
    rp, c, v, _ = run_gpu(A, B)
    compare(A, B, rp, c, v, exact=True)
