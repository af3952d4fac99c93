"""The segment path of long numeric rows at the edges of its segments: rows of
C of exactly one, two and sixteen segments of values and one column either
side, with the row's table in LDS (a range of 200 thousand columns, 11776
values beside its table) and in the global slab (a million columns, 18048
values; beyond 78848 the row adds into C), plain and Jacobi-fused."""
import numpy as np
import pytest

import oracle
from paper_2103_11991_amd import gen
from gpu_util import compare

pytestmark = pytest.mark.gpu

FULL, W = 1999, 100  # rows of B of 100 neighbouring columns, then rows of 1, 2, ..., 100 columns behind them


def _matrices(sizes, stride, dtype):
    """A square, with a stored diagonal; its rows 2, 3, ... give rows of C of ``sizes`` columns."""
    rng = np.random.default_rng(len(sizes) + stride)
    n = FULL + W
    bl = np.concatenate([np.full(FULL, W), np.arange(1, W + 1)])
    first = np.concatenate([np.arange(FULL) * W, np.full(W, FULL * W)])
    cols = np.concatenate([rng.permutation(np.arange(f, f + l)) for f, l in zip(first, bl)]) * stride
    B = gen.csr_from_rows_cols(n, (FULL * W + W) * stride, np.repeat(np.arange(n), bl), cols,
                               rng.integers(-3, 4, size=cols.size).astype(dtype))
    rows = [np.array([i]) for i in range(n)]
    for t, c in enumerate(sizes):
        full = (c - 1) // W
        assert full > 2 + t
        rows[2 + t] = np.concatenate([rng.permutation(full), [FULL + c - W * full - 1]])
    ci = np.concatenate(rows)
    A = gen.csr_from_rows_cols(n, n, np.repeat(np.arange(n), [r.size for r in rows]), ci,
                               rng.integers(1, 4, size=ci.size).astype(dtype))
    return A, B


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("stride,sizes", [(1, [11775, 11776, 11777, 23552, 23553, 188415, 188416, 188417]),
                                          (5, [18047, 18048, 18049, 78847, 78848, 78849])])
def test_segment_edges(stride, sizes, dtype):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMM
    A, B = _matrices(sizes, stride, dtype)
    # (with the limit FP32 rows of 11775 columns are no LDS rows either)
    op = SpGEMM(DeviceCsr.from_host(A), DeviceCsr.from_host(B), tiled_global=0, lds_limit=16384)
    rp, _ = op.symbolic()
    rp = rp.cpu().numpy().astype(np.int64)
    assert list(np.diff(rp)[2:2 + len(sizes)]) == sizes
    assert op.stats()["num_rows"][9] == len(sizes)
    col, val = op.numeric()
    torch.cuda.synchronize()
    compare(A, B, rp, col.cpu().numpy(), val.cpu().numpy(), exact=True)  # integers
    dinv = np.arange(1, A.m + 1) % 5 + 1.0
    col, val = op.numeric_jacobi(2.0, torch.from_numpy(dinv.astype(dtype)).cuda())
    torch.cuda.synchronize()
    _, ocol, oval, _ = oracle.jacobi_spgemm(A, B, 2.0, dinv)
    np.testing.assert_array_equal(col.cpu().numpy(), ocol)
    np.testing.assert_array_equal(val.cpu().numpy().astype(np.float64), oval)
