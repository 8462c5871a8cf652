"""SpMV on unordered entries by bins of rows (unordered COO, CSC) at the edges of its tiles, bins and scratch.
Operands are built on the GPU; the reference is the definition, its products and sums in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FROM, MOST, STEP = 3 << 17, 3 << 18, 512 * 2048  # half of the line; binned from here on; entries that a vector a thread is


def _entries(order, N, M, nnz, dtype, misalign, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    row = torch.randint(0, N, (nnz,), generator=g, device="cuda")
    if order == "heavy":  # a row with nearly half of them, at random places; no entry in the upper half of the rows
        row = torch.where(torch.rand(nnz, generator=g, device="cuda") < 0.45, N // 3, row // 2)
    elif order == "sorted":
        row = row.sort().values
    elif order == "edges":  # the first and the last row of the matrix only
        row = (row % 2) * (N - 1)
    col = torch.randint(0, M, (nnz,), generator=g, device="cuda")
    vals = torch.rand(nnz, generator=g, device="cuda", dtype=dtype) * 2 - 1

    def place(t):  # at the start of its allocation, or one element further
        out = torch.empty(len(t) + 1, dtype=t.dtype, device="cuda")[int(misalign):][:len(t)]
        out.copy_(t)
        return out

    return row, col, place(row.int()), place(col.int()), place(vals)


def _operand(form, N, M, row, col, row32, col32, vals):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    one = np.ones(1, np.float64 if vals.dtype == torch.float64 else np.float32)
    nnz = len(vals)
    if form == "csc":
        at = col.argsort(stable=True)
        row32, vals = row32[at].contiguous(), vals[at].contiguous()
        pos = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
        pos[1:] = torch.bincount(col, minlength=M).cumsum(0)
        A = spt.DeviceTensor(wl.csr_spec(1, N, [0, 1], [0], one))
        A.c.level[0].N, A.c.level[1].M, A.c.level[1].N = M, M, N
        A.c.level[0].mode, A.c.level[1].mode = 1, 0
        A.c.level[1].pos, A.c.level[1].crd, A.c.level[1].max_children = pos.data_ptr(), row32.data_ptr(), 0
    else:
        A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], one, ordered=False))
        pos = torch.tensor([0, nnz], dtype=torch.int32, device="cuda")
        A.c.level[0].pos = pos.data_ptr()
        A.c.level[0].crd, A.c.level[1].crd = row32.data_ptr(), col32.data_ptr()
    A.c.vals, A.c.nvals = vals.data_ptr(), nnz
    return A, (pos, row32, col32, vals)


@pytest.mark.parametrize("form,order,N,M,nnz,dtype,misalign,ws_of", [
    # a thread has 2 to 8 vectors; whole tiles, tails of a vector and of a tile
    ("coo", "random", 40_000, 30_000, FROM, "float64", False, "query"),
    ("coo", "random", 40_000, 30_000, 2 * STEP + 1, "float32", False, "query"),
    ("coo", "random", 200_000, 30_000, 4 * STEP - 3, "float64", True, "query"),
    ("coo", "sorted", 200_000, 30_000, 4 * STEP + 5, "float32", True, "query"),
    ("coo", "random", 70_001, 50_000, 6 * STEP, "float64", False, "query"),
    ("coo", "heavy", 70_001, 50_000, 7 * STEP - 1, "float32", False, "query"),
    ("coo", "random", 70_001, 50_000, 8 * STEP + 2, "float64", False, "query"),
    # few rows; the first and the last of a bin; rows in one bin or two
    ("coo", "random", 1, 30_000, FROM + 1, "float64", False, "query"),
    ("coo", "random", 255, 30_000, MOST, "float32", False, "query"),
    ("coo", "edges", 257, 30_000, 900_001, "float64", False, "query"),
    ("coo", "sorted", 1_000_003, 30_000, 900_001, "float64", True, "query"),
    ("coo", "heavy", 100_000, 30_000, 3_000_001, "float64", True, "query"),
    # several sub-ranges of a bin; 32-bit rows within a bin
    ("coo", "random", (1 << 22) + 1, 30_000, 1_000_000, "float32", False, "query"),
    ("coo", "edges", (1 << 24) + 1000, 30_000, 500_000, "float64", False, "query"),
    ("coo", "heavy", (1 << 24) + 1000, 30_000, 1_000_000, "float32", True, "query"),
    # x slice by slice
    ("coo", "random", 300_000, 800_001, 1 << 22, "float64", False, "query"),
    ("coo", "sorted", 300_000, 1_600_000, (1 << 22) + 4099, "float32", True, "query"),
    ("coo", "heavy", (1 << 24) + 1000, 800_001, (1 << 22) + 2, "float64", True, "query"),
    ("coo", "random", 300_000, 800_001, (1 << 22) - 1, "float64", False, "query"),
    # without the workspace of the bins: the scatter below the line
    ("coo", "random", 40_000, 30_000, FROM, "float64", False, "none"),
    ("coo", "random", 40_000, 30_000, MOST - 1, "float32", False, "none"),
    ("coo", "random", 40_000, 30_000, MOST, "float64", False, "refused"),
    ("csc", "random", 40_000, 30_000, 500_000, "float64", False, "query"),
    ("csc", "heavy", 300_000, 900_000, (1 << 22) + 3, "float32", False, "query"),
    ("csc", "random", 40_000, 30_000, MOST - 1, "float64", False, "none"),
    ("csc", "random", 40_000, 30_000, MOST, "float32", False, "refused"),
])
def test_binned_spmv(form, order, N, M, nnz, dtype, misalign, ws_of):
    import torch
    import paper_1804_10112_amd as spt
    dt = getattr(torch, dtype)
    row, col, row32, col32, vals = _entries(order, N, M, nnz, dt, misalign, nnz % 97)
    A, keep = _operand(form, N, M, row, col, row32, col32, vals)
    x = torch.rand(M, device="cuda", dtype=dt) * 2 - 1
    y = torch.full((N,), float("nan"), device="cuda", dtype=dt)
    columns = (nnz * 4 + 255) // 256 * 256 if form == "csc" else 0
    size = spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A)
    ws = torch.empty(size if ws_of == "query" else columns + 256, dtype=torch.uint8, device="cuda")
    if ws_of == "refused":
        with pytest.raises(spt.SptError):
            spt.spt_spmv(A, x, y, ws)
        return
    spt.spt_spmv(A, x, y, ws)
    got = y.cpu().numpy()
    t = (vals.double() * x.double()[col]).cpu().numpy()
    at = row.cpu().numpy()
    ref, mag = np.bincount(at, t, N), np.bincount(at, np.abs(t), N)
    count = np.bincount(at, minlength=N)
    # a rounding per product, one per addition in any order (of the scatter; the bins have fewer), and one of the result
    eps = np.finfo(got.dtype).eps
    assert np.all(np.abs(got - ref) <= eps * (count + 2) * mag), np.max(np.abs(got - ref) - eps * (count + 2) * mag)
