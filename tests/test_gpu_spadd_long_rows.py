"""Numeric phase of sparse addition for rows of more than 64 entries: rows of C
around a wavefront's 512 columns, around every window of the workgroup kernel
(1024, 2048, 4096 columns, by the longest row) and of several windows; rows of
many entries but few columns; and few long rows among very many."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen

pytestmark = pytest.mark.gpu


def _csr(n, rows, dtype, seed):
    rng = np.random.default_rng(seed)
    lens = np.array([r.size for r in rows])
    ci = np.concatenate(rows)
    return gen.csr_from_rows_cols(lens.size, n, np.repeat(np.arange(lens.size), lens), ci,
                                  rng.integers(-4, 5, size=ci.size).astype(dtype))


def _check(A, B):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd
    add = SpAdd(DeviceCsr.from_host(A), DeviceCsr.from_host(B))
    rp, _ = add.symbolic()
    orp, ocol, oval, _ = oracle.spadd(A, B, 3.0, -2.0)
    np.testing.assert_array_equal(rp.cpu().numpy().astype(np.int64), orp)
    for _ in range(2):
        col, val = add.numeric(3.0, -2.0)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(col.cpu().numpy(), ocol)
        np.testing.assert_array_equal(val.cpu().numpy().astype(np.float64), oval)  # integers: exact


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("order", ["sorted", "unsorted", "repeats"])
@pytest.mark.parametrize("longest", [512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8193, 16384])
def test_longest_row(longest, order, dtype):
    rng = np.random.default_rng(longest)
    n = 20000
    a, b = [], []
    for c in (longest, 65, longest - 1, 130, longest // 2 + 1, 512, 3, 0):
        cols = np.sort(rng.choice(n, size=c, replace=False))
        split = rng.random(c) < 0.5
        ra, rb = cols[split], cols[~split]
        if c + 40 <= 16384 and c > 40:
            rb = np.sort(np.concatenate([rb, ra[:20]]))  # some columns in both
        if order == "repeats" and 3 * c <= 16384:
            ra = np.sort(np.concatenate([ra, ra[::2]]))  # and some twice in one
        if order == "unsorted":
            ra, rb = rng.permutation(ra), rng.permutation(rb)
        a.append(ra)
        b.append(rb)
    _check(_csr(n, a, dtype, 1), _csr(n, b, dtype, 2))


@pytest.mark.parametrize("columns", [1, 100, 512, 513])
def test_many_entries_in_few_columns(columns):
    rng = np.random.default_rng(columns)
    a = [np.concatenate([np.arange(columns), rng.integers(0, columns, size=8000 - columns)]), np.arange(3)]
    b = [rng.integers(0, columns, size=7000), np.arange(2)]
    _check(_csr(600, a, np.float64, 3), _csr(600, b, np.float64, 4))


def test_few_long_rows_among_many():
    """More rows than one look of every workgroup covers (2048 x 256)."""
    m, n = 600000, 5000
    lens = np.ones(m, dtype=np.int64)
    lens[[0, 1, 2047, 2048, 300001, 524288, 524289, m - 1]] = [600, 513, 2000, 700, 4500, 512, 900, 1500]
    at = np.arange(lens.sum()) - np.repeat(np.cumsum(lens) - lens, lens)
    ci = (np.repeat(np.arange(m) * 7 % n, lens) + at) % n
    vals = (np.arange(ci.size) % 7 - 3).astype(np.float64)
    A = gen.csr_from_rows_cols(m, n, np.repeat(np.arange(m), lens), ci, vals)
    B = gen.csr_from_rows_cols(m, n, np.arange(m), (np.arange(m) * 11) % n, np.ones(m))
    _check(A, B)
