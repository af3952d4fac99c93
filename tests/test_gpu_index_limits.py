"""Matrices of 2^31 - 1 entries, the most that int32 row pointers hold: the
last row ends where an index stepped past it no longer fits int32.  Rows of
8, 64, 512 and more entries take the walks of one lane, of a group of lanes,
of a wavefront and of several.  Needs up to 70 GB of device memory."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NNZ = 2 ** 31 - 1
PART = 1 << 28


def setup_function(_):
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 75 * 2 ** 30:
        pytest.skip("needs 75 GiB of free device memory")


def teardown_function(_):
    import torch
    torch.cuda.empty_cache()


def _full(length, k, dtype):
    """NNZ ones: rows of ``length`` entries, the last of one less, columns ascending inside each row (length divides k)."""
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr
    m = 2 ** 31 // length
    rp = torch.arange(m + 1, dtype=torch.int64, device="cuda").mul_(length)
    rp[-1] = NNZ
    ci = torch.arange(NNZ, dtype=torch.int32, device="cuda").bitwise_and_(k - 1)
    return DeviceCsr(m, k, rp.to(torch.int32), ci, torch.ones(NNZ, dtype=dtype, device="cuda"))


def _same(col, val, A, f):
    """C has A's columns, and the value f(column) at each."""
    import torch
    for s in range(0, NNZ, PART):
        c = A.col_idx[s:s + PART]
        assert torch.equal(col[s:s + PART], c)
        assert torch.equal(val[s:s + PART], f(c))


@pytest.mark.parametrize("length", [8, 64, 512])
def test_last_rows_of_b(length):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMM
    B = _full(length, 1024, torch.float32)
    n = B.m
    rows = [[(n - 1, 2.0)], [(n - 2, 3.0), (n - 1, 5.0), (0, 7.0)], [], [(n - 1, 1.0), (n - 1, 1.0)]]
    A = DeviceCsr(4, n, torch.tensor([0, 1, 4, 4, 6], dtype=torch.int32, device="cuda"),
                  torch.tensor([j for r in rows for j, _ in r], dtype=torch.int32, device="cuda"),
                  torch.tensor([x for r in rows for _, x in r], dtype=torch.float32, device="cuda"))
    op = SpGEMM(A, B)
    rp, _ = op.symbolic()
    col, val = op.numeric()
    rp, col, val = rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()
    for i, r in enumerate(rows):
        want, hit = np.zeros(1024), np.zeros(1024, dtype=bool)
        for j, x in r:
            e = np.arange(j * length, min((j + 1) * length, NNZ)) % 1024
            want[e] += x
            hit[e] = True
        s = slice(rp[i], rp[i + 1])
        np.testing.assert_array_equal(col[s], np.flatnonzero(hit))
        np.testing.assert_array_equal(val[s], want[hit])


@pytest.mark.parametrize("length,opts", [(8, {}), (64, {}), (512, {}), (4096, {}), (16384, {}),
                                         (16384, {"tiled_global": 0})])
def test_last_rows_of_a(length, opts):
    """Times a diagonal matrix of 1, 2, 3, ..."""
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpGEMM
    k = max(length, 512)
    A = _full(length, k, torch.float32)
    i = torch.arange(k + 1, dtype=torch.int32, device="cuda")
    B = DeviceCsr(k, k, i, i[:-1].clone(), i[1:].to(torch.float32))
    op = SpGEMM(A, B, **opts)
    rp, nnz = op.symbolic()
    assert nnz == NNZ and torch.equal(rp, A.row_ptr)
    col, val = op.numeric()
    _same(col, val, A, lambda c: (c + 1).to(torch.float32))


@pytest.mark.parametrize("length", [8, 64, 512, 4096])
def test_last_rows_of_an_addition(length):
    import torch
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd
    A = _full(length, 8192, torch.float32)
    none = torch.zeros(0, device="cuda")
    B = DeviceCsr(A.m, A.n, torch.zeros_like(A.row_ptr), none.to(torch.int32), none)
    for first, second in ((A, B), (B, A)):
        add = SpAdd(first, second)
        rp, nnz = add.symbolic()
        assert nnz == NNZ and torch.equal(rp, A.row_ptr)
        col, val = add.numeric(3.0, 3.0)
        _same(col, val, A, lambda c: torch.full(c.shape, 3.0, device="cuda"))
        del add, rp, col, val


@pytest.mark.parametrize("la,lb", [(2 ** 30, 2 ** 30 + 5), (NNZ, 2), (2 ** 30, 16)])
def test_row_pair_of_more_than_int32_entries_is_refused(la, lb):
    import torch
    from paper_2103_11991_amd._lib import SpgError
    from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd
    def row(count):
        return DeviceCsr(1, 8, torch.tensor([0, count], dtype=torch.int32, device="cuda"),
                         torch.zeros(count, dtype=torch.int32, device="cuda"), torch.ones(count, device="cuda"))
    with pytest.raises(SpgError) as e:
        SpAdd(row(la), row(lb)).symbolic()
    assert e.value.status_name == "SPG_ERR_UNSUPPORTED"
