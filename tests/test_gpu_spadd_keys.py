"""Sparse addition at the largest key of every sort: rows of exactly 64, 128,
256 and 1024 entries whose last entry (the largest index inside the row) lies
in the matrix's last column, at the column counts up to which a key of column
and index fits 32 bits, and one column either side.  The last entry is B's,
or A's where B's row is empty; in half the rows A holds the last column too."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen

pytestmark = pytest.mark.gpu

TOTALS = [64, 128, 256, 1024]


def _columns(n, count, order, last, rng):
    """``count`` distinct columns among the last 4096, the final one n - 1 if ``last``, else below it."""
    c = n - 4096 + np.sort(rng.choice(4095, size=count, replace=False))
    if last and count:
        c[-1] = n - 1
    if order == "unsorted" and count > 1:
        c[:-1] = rng.permutation(c[:-1])
    return c


def _pair(n, order):
    rng = np.random.default_rng(n % 1000003)
    rows = {"A": [], "B": []}
    for total in TOTALS:
        for la in (0, 1, total // 2, total):
            for shared in (False, True):
                lb = total - la
                rows["A"].append(_columns(n, la, order, shared or lb == 0, rng))
                rows["B"].append(_columns(n, lb, order, True, rng))
    out = []
    for s in "AB":
        lens = [c.size for c in rows[s]]
        ci = np.concatenate(rows[s])
        out.append(gen.csr_from_rows_cols(len(lens), n, np.repeat(np.arange(len(lens)), lens), ci,
                                          rng.integers(1, 9, size=ci.size).astype(np.float64)))
    return out


@pytest.mark.parametrize("order", ["sorted", "unsorted"])
@pytest.mark.parametrize("off", [-1, 0, 1])
@pytest.mark.parametrize("bits", [22, 24, 25, 26])
def test_last_column_in_the_last_entry(bits, off, order):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd
    A, B = _pair((1 << bits) + off, order)
    add = SpAdd(DeviceCsr.from_host(A), DeviceCsr.from_host(B))
    rp, _ = add.symbolic()
    col, val = add.numeric(2.0, -1.0)
    torch.cuda.synchronize()
    orp, ocol, oval, _ = oracle.spadd(A, B, 2.0, -1.0)
    np.testing.assert_array_equal(rp.cpu().numpy().astype(np.int64), orp)
    np.testing.assert_array_equal(col.cpu().numpy(), ocol)
    np.testing.assert_array_equal(val.cpu().numpy(), oval)  # integers: exact
