"""A product without rows after another on the same handle: nothing of the
earlier one's analysis is left (its missing diagonal, its column tiles)."""
import numpy as np
import pytest

from paper_2103_11991_amd import gen

pytestmark = pytest.mark.gpu


def test_jacobi_without_rows_after_a_missing_diagonal():
    from paper_2103_11991_amd._lib import SpgError
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMM
    A = DeviceCsr.from_host(gen.csr_from_rows_cols(2, 2, np.array([0]), np.array([1]), np.ones(1)))
    none = np.empty(0, dtype=np.int64)
    E = DeviceCsr.from_host(gen.csr_from_rows_cols(0, 0, none, none, np.empty(0)))
    op = SpGEMM(A, A)
    op.symbolic()
    with pytest.raises(SpgError) as e:
        op.numeric_jacobi(0.5, A.values.new_ones(2))
    assert e.value.status_name == "SPG_ERR_SHAPE"
    op.set_matrices(E, E)
    rp, nnz = op.symbolic()
    assert nnz == 0 and rp.tolist() == [0]
    col, val = op.numeric_jacobi(0.5, A.values.new_ones(0))
    assert col.numel() == 0 and val.numel() == 0 and op.stats()["num_tiles"] == 0
