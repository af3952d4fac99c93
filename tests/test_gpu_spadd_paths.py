"""Sparse addition at the edges of its row paths: entries per row around the
lane groups (16, 32, 64), the register sorts (64, 128, 256) and the LDS sorts
(1024, longer), column counts around what 32-bit keys hold, and rows of C
around the numeric phase's LDS window (512 columns, 8 of them)."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen

pytestmark = pytest.mark.gpu

TOTALS = [0, 1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025]


def _matrix(n, lens, seed, order):
    rng = np.random.default_rng(seed)
    ci = []
    for l in lens:
        l = int(l)
        c = rng.choice(min(n, 8192), size=l, replace=order == "repeats")
        c = c.astype(np.int64) + (n - min(n, 8192) if rng.random() < 0.5 else 0)  # the first or the last columns
        ci.append(np.sort(c) if order in ("sorted", "repeats") else c)
    ci = np.concatenate(ci) if ci else np.zeros(0, dtype=np.int64)
    vals = rng.integers(-4, 5, size=ci.size).astype(np.float64)
    m = len(lens)
    return gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), lens), ci, vals)


def _check(A, B):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd
    add = SpAdd(DeviceCsr.from_host(A), DeviceCsr.from_host(B))
    rp, _ = add.symbolic()
    col, val = add.numeric(2.0, -1.0)
    torch.cuda.synchronize()
    orp, ocol, oval, _ = oracle.spadd(A, B, 2.0, -1.0)
    np.testing.assert_array_equal(rp.cpu().numpy().astype(np.int64), orp)
    np.testing.assert_array_equal(col.cpu().numpy(), ocol)
    np.testing.assert_array_equal(val.cpu().numpy().astype(np.float64), oval)  # integers: exact


@pytest.mark.parametrize("order", ["sorted", "unsorted", "repeats"])
@pytest.mark.parametrize("n", [2100, 1 << 22, (1 << 22) + 1, (1 << 24) + 1, (1 << 25) + 1, (1 << 26) + 1])
def test_row_totals_and_column_counts(n, order):
    total = np.array(TOTALS * 3)
    la = np.concatenate([np.array(TOTALS) // 2, np.zeros(len(TOTALS), dtype=np.int64), np.array(TOTALS)])
    _check(_matrix(n, la, 1, order), _matrix(n, total - la, 2, order))


@pytest.mark.parametrize("avg", [6, 20, 40])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_lane_groups(avg, dtype):
    """Average lengths that pick 16, 32 and 64 lanes per row, a few rows that do not fit them."""
    rng = np.random.default_rng(avg)
    la, lb = rng.integers(0, avg + 1, size=5003), rng.integers(0, avg + 1, size=5003)
    la[::997] = 70
    A, B = _matrix(3000, la, 3, "sorted"), _matrix(3000, lb, 4, "sorted")
    _check(A.astype(dtype), B.astype(dtype))


@pytest.mark.parametrize("nc", [511, 512, 513, 4095, 4096, 4097, 6000])
def test_numeric_window(nc):
    la = np.array([nc, 0, nc // 2, 3])
    lb = np.array([0, nc, nc - nc // 2, nc])
    _check(_matrix(8192, la, 5, "sorted"), _matrix(8192, lb, 6, "sorted"))
