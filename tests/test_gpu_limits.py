"""Calls at the limits of the index types: entry counts next to 2^31, where a
step's positions no longer fit an int, and launches next to 2^32 threads."""
import pytest
import torch

pytestmark = pytest.mark.gpu

mls = pytest.importorskip("paper_1804_00695_amd")

LIMIT = (1 << 31) - 1   # entry counts stay below


def need(gib):
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip(f"needs {gib} GiB of free device memory")


@pytest.fixture(autouse=True)
def give_back():
    yield
    mls._default_ws.clear()
    torch.cuda.empty_cache()


def full_rows(nnz, ncols):
    """Rows of columns 0 .. 32767, the last one shorter: nnz entries in all."""
    ci = torch.arange(nnz, dtype=torch.int32, device="cuda").bitwise_and_(32767)
    rp = torch.arange(0, nnz + 32768, 32768, dtype=torch.int64, device="cuda").clamp_(max=nnz).to(torch.int32)
    return mls.DeviceCsr(rp.numel() - 1, ncols, rp, ci, None)


# the entry streams (validation, compression, row sizes) at a run that ends
# within a tile (512 entries) of the limit
def test_entry_streams_near_the_limit():
    need(64)
    M = full_rows(LIMIT - 299, 70000)
    tail = M.nnz - 32768 * (M.nrows - 1)
    words, count = mls.compress(M)
    assert count[:-1].eq(1024).all() and int(count[-1]) == (tail + 31) // 32
    last = words[2 * (M.nnz - tail):2 * (M.nnz - tail) + 2 * int(count[-1])].view(-1, 2)
    assert last[:, 0].eq(torch.arange(int(count[-1]), device="cuda")).all() and last[:-1, 1].eq(-1).all()
    assert int(last[-1, 1]) == (1 << (tail % 32)) - 1
    del words, count, last
    one = mls.DeviceCsr(1, M.nrows, torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                        torch.tensor([M.nrows - 1], dtype=torch.int32, device="cuda"), None)
    C = mls.symbolic(one, M, with_values=False)
    assert C.nnz == tail and C.col_idx.eq(torch.arange(tail, device="cuda")).all()
    C = None
    mls._default_ws.clear()
    eye = torch.arange(70001, dtype=torch.int32, device="cuda")
    C = mls.symbolic(M, mls.DeviceCsr(70000, 70000, eye, eye[:-1], None), with_values=False)
    assert torch.equal(C.row_ptr, M.row_ptr) and torch.equal(C.col_idx, M.col_idx)
    C = None
    M.col_idx[-1] = 70000   # the last entry is looked at
    with pytest.raises(mls.SpgemmError):
        mls.symbolic(one, M, with_values=False)


# the fixed-order adjoint with a row of B of two entries at the very end
def test_fixed_order_adjoint_near_the_limit():
    need(80)
    B = full_rows(LIMIT - 1, 32768)
    n = B.nrows
    rp = torch.cat([B.row_ptr[:-1], B.row_ptr[-1:] - 2, B.row_ptr[-1:]])
    B.col_idx[-2:] = torch.tensor([5, 9], dtype=torch.int32, device="cuda")
    v = torch.zeros(B.nnz, dtype=torch.float64, device="cuda")
    v[-2:] = torch.tensor([3.0, 7.0])
    B = mls.DeviceCsr(n + 1, 32768, rp, B.col_idx, v)
    i32 = dict(dtype=torch.int32, device="cuda")
    f64 = dict(dtype=torch.float64, device="cuda")
    A = mls.DeviceCsr(1, n + 1, torch.tensor([0, 1], **i32), torch.tensor([n], **i32), torch.tensor([2.0], **f64))
    W = mls.DeviceCsr(1, 32768, torch.tensor([0, 2], **i32), torch.tensor([5, 9], **i32),
                      torch.tensor([10.0, 100.0], **f64))
    gA, gB = mls.backward(A, B, W, deterministic=True)
    assert gA.tolist() == [730.0] and gB[-2:].tolist() == [20.0, 200.0]
    assert int(torch.count_nonzero(gB)) == 2


# several lanes per row (scatter) and per column (sort): 2^32 threads and more
@pytest.mark.parametrize("nrows,ncols", [(4000, (1 << 28) + 3), ((1 << 29) + 3, 7)])
def test_transpose_of_many_rows(nrows, ncols):
    need(48)
    i32 = dict(dtype=torch.int32, device="cuda")
    k = 3000   # the first k rows and the last one end in the last column
    rp = torch.full((nrows + 1,), k, **i32)
    rp[:k], rp[nrows:] = torch.arange(k, **i32), k + 2
    ci = torch.full((k + 2,), ncols - 1, **i32)
    ci[k] = 0
    v = torch.arange(k + 2, dtype=torch.float64, device="cuda")
    T = mls.transpose(mls.DeviceCsr(nrows, ncols, rp, ci, v))
    assert T.row_ptr[0] == 0 and T.row_ptr[1:ncols].eq(1).all() and T.row_ptr[ncols] == k + 2
    assert T.col_idx.tolist() == [nrows - 1] + list(range(k)) + [nrows - 1]
    assert T.values.tolist() == [float(k)] + [float(x) for x in range(k)] + [k + 1.0]
