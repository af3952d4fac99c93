"""Columns out of range at the first entries of B, in each of the walks that
compress B's rows (one lane, a group of lanes, a wavefront): refused, whatever
block such a column would fall in, and the handle works on afterwards."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen
from gpu_util import compare

pytestmark = pytest.mark.gpu


def _b(rows, length, k=700):
    """``rows`` rows of ``length`` consecutive columns."""
    first = (np.arange(rows) * 37) % (k - length)
    ci = (first[:, None] + np.arange(length)[None, :]).reshape(-1)
    return gen.csr_from_rows_cols(rows, k, np.repeat(np.arange(rows), length), ci, np.ones(ci.size))


@pytest.mark.parametrize("bad", [-1, -31, -32, -33, 700, 2 ** 31 - 1, -2 ** 31])
@pytest.mark.parametrize("rows,length", [((1 << 17) + 3, 5), (300, 20), (300, 8), (40, 600)])
def test_first_columns_out_of_range(rows, length, bad):
    import torch
    from paper_2103_11991_amd._lib import SpgError
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMM
    B = _b(rows, length)
    A = gen.csr_from_rows_cols(3, rows, np.array([0, 0, 1, 2]), np.array([0, rows - 1, 1, 0]), np.ones(4))
    dA = DeviceCsr.from_host(A)
    good = DeviceCsr.from_host(B)
    op = SpGEMM(dA, good)
    for count in (1, 2, length):  # the first row's first entries
        ci = B.col_idx.copy()
        ci[:count] = bad
        op.set_matrices(dA, DeviceCsr.from_host(gen.Csr(B.m, B.n, B.row_ptr, ci, B.values)))
        with pytest.raises(SpgError) as e:
            op.symbolic()
        assert e.value.status_name == "SPG_ERR_INDEX"
    op.set_matrices(dA, good)
    rp, _ = op.symbolic()
    col, val = op.numeric()
    torch.cuda.synchronize()
    compare(A, B, rp.cpu().numpy().astype(np.int64), col.cpu().numpy(), val.cpu().numpy(), exact=True)
