"""SpMV with x gathered slice by slice: CSR of 2^25 entries or more and ordered COO of more than 2^24, x beyond
6 MB. Operands are built on the GPU; the reference is the definition, its products and sums in float64."""
import numpy as np
import pytest

from gpu_util import assert_close_where_finite

pytestmark = pytest.mark.gpu

CSR_FROM, COO_FROM, SEGMENT = 1 << 25, (1 << 24) + 1, 256


def _lengths(kind, N, nnz, g):
    """Row lengths that add up to nnz: runs of empty rows at both ends and (one segment's worth of them and more)
    in the middle; `heavy` adds rows of many segments (`declared`: and a bound on them), `one row` leaves nearly all
    entries to one, `some empty` leaves a third of all rows without entries. `level`: all rows alike."""
    import torch
    if kind == "level":
        return nnz // N + (torch.arange(N, device="cuda") < nnz % N).long()
    L = torch.randint(0, 2 * (nnz // N) + 2, (N,), generator=g, device="cuda")
    if kind == "one row":
        L = torch.randint(0, 2, (N,), generator=g, device="cuda")
    elif kind == "some empty":
        L = torch.randint(0, 3, (N,), generator=g, device="cuda")
    L[:700] = 0
    L[N // 2:N // 2 + 3000] = 0
    L[-900:] = 0
    L[N // 3] = 5000
    if kind in ("heavy", "declared"):
        L[N // 4] = nnz // 60
        L[N // 5:N // 5 + 40] = 4097
    at = 2 * N // 3
    L[at] = 0
    over = int(L.sum()) - nnz
    if over > 0:  # thin out from the end, keeping the empty rows
        c = L.flip(0).cumsum(0)
        k = int(torch.searchsorted(c, torch.tensor(over, device="cuda")))
        L[N - k:] = 0
        L[N - 1 - k] -= over - (int(c[k - 1]) if k else 0)
    else:
        L[at] = -over
    assert int(L.sum()) == nnz and int(L.min()) >= 0
    return L


def _matrix(form, kind, cols, N, M, nnz, dtype, misalign, seed):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    g = torch.Generator(device="cuda").manual_seed(seed)
    L = _lengths(kind, N, nnz, g)
    row = torch.repeat_interleave(torch.arange(N, device="cuda"), L)
    if cols == "scattered":
        col = torch.randint(0, M, (nnz,), generator=g, device="cuda")
        col = (row * M + col).sort().values % M
    elif cols == "third":  # anywhere in a third of x that moves on with the row
        col = (row * M // N + torch.randint(0, M // 3, (nnz,), generator=g, device="cuda")) % M
        col = (row * M + col).sort().values % M
    else:
        col = (row * M // N + torch.randint(-60, 61, (nnz,), generator=g, device="cuda")).clamp_(0, M - 1)
        col = (row * M + col).sort().values % M
    vals = torch.rand(nnz, generator=g, device="cuda", dtype=dtype) * 2 - 1

    def place(t):  # at the start of its allocation, or one element further
        out = torch.empty(len(t) + 1, dtype=t.dtype, device="cuda")[int(misalign):][:len(t)]
        out.copy_(t)
        return out

    row32, col32, vals = place(row.int()), place(col.int()), place(vals)
    one = np.ones(1, np.float64 if dtype == torch.float64 else np.float32)
    if form == "csr":
        pos = place(torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), L.cumsum(0)]).int())
        A = spt.DeviceTensor(wl.csr_spec(1, M, [0, 1], [0], one))
        A.c.level[1].max_children = nnz // 60 if kind == "declared" else 0
        A.c.level[0].N = A.c.level[1].M = N
        A.c.level[1].pos, A.c.level[1].crd = pos.data_ptr(), col32.data_ptr()
        keep = (pos, col32, vals)
    else:
        A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], one, ordered=True))
        pos = torch.tensor([0, nnz], dtype=torch.int32, device="cuda")
        A.c.level[0].pos = pos.data_ptr()
        A.c.level[0].crd, A.c.level[1].crd = row32.data_ptr(), col32.data_ptr()
        keep = (pos, row32, col32, vals)
    A.c.vals, A.c.nvals = vals.data_ptr(), nnz
    return A, keep, row, col, vals


def _reference(row, col, vals, x, N):
    t = (vals.double() * x.double()[col]).cpu().numpy()
    first = np.flatnonzero(np.diff(row.cpu().numpy(), prepend=-1))
    ref, mag = np.zeros(N), np.zeros(N)
    at = row.cpu().numpy()[first]
    with np.errstate(invalid="ignore", over="ignore"):
        ref[at], mag[at] = np.add.reduceat(t, first), np.add.reduceat(np.abs(t), first)
    return ref, mag


def _check(A, row, col, vals, x, N, ws, what):
    import torch
    import paper_1804_10112_amd as spt
    y = torch.full((N,), float("nan"), dtype=x.dtype, device="cuda")
    spt.spt_spmv(A, x, y, ws)
    again = torch.full_like(y, float("nan"))
    spt.spt_spmv(A, x, again, ws)
    assert torch.equal(y.nan_to_num(7.0), again.nan_to_num(7.0)), f"{what}: two calls differ"
    ref, mag = _reference(row, col, vals, x, N)
    assert_close_where_finite(y.cpu().numpy(), ref, mag, np.float64 if x.dtype == torch.float64 else np.float32, what)


# x of just over 6 MB (two or three slices, the last shorter), and of 16 MB; entries that fill the last segment, that leave
# one entry to it, and that end inside a vector; lanes, waves and workgroups without a segment occur in all of them
@pytest.mark.parametrize("form,kind,cols,dtype,M,extra,misalign", [
    ("csr", "even", "scattered", "float64", 750_003, 1, False),
    ("csr", "even", "scattered", "float32", 1_500_007, 0, True),
    ("csr", "heavy", "scattered", "float64", 2_000_003, 255, True),
    ("csr", "heavy", "local", "float32", 4_000_001, 3, False),
    ("csr", "heavy", "local", "float64", 750_003, 2, True),
    ("csr", "even", "local", "float64", 1_000_003, 1, False),
    ("csr", "declared", "scattered", "float32", 1_500_007, 254, False),
    ("csr", "declared", "local", "float64", 750_003, 1, False),
    ("csr", "one row", "scattered", "float32", 1_500_007, 1, False),
    # rows of a segment about as many as its entries: a wave enters those of some segments row by row (up to 256) and
    # looks those of others up, into the same stretch of LDS
    ("csr", "some empty", "scattered", "float64", 750_003, 7, False),
    ("csr", "some empty", "scattered", "float32", 1_500_007, 2, True),
    # columns that do not lie scattered, segments in order: rows looked up and entered, a row of most segments
    ("csr", "one row", "local", "float64", 750_003, 255, True),
    ("csr", "one row", "local", "float32", 1_500_007, 0, False),
    ("coo", "one row", "local", "float32", 1_500_007, 255, True),
    ("coo", "some empty", "local", "float64", 750_003, 0, False),
    ("coo", "even", "scattered", "float64", 750_003, 0, True),
    ("coo", "heavy", "scattered", "float32", 1_500_007, 255, False),
    ("coo", "heavy", "local", "float64", 2_000_003, 2, False),
    ("coo", "even", "local", "float32", 1_500_007, 3, True),
    ("coo", "one row", "scattered", "float64", 750_003, 1, False),
])
def test_against_the_definition(form, kind, cols, dtype, M, extra, misalign):
    import torch
    dt = getattr(torch, dtype)
    nnz = (CSR_FROM if form == "csr" else COO_FROM + SEGMENT - 1) + extra
    N = nnz + 100_000 if kind == "some empty" else 1_200_007 if form == "csr" else 700_003
    A, keep, row, col, vals = _matrix(form, kind, cols, N, M, nnz, dt, misalign, 5)
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.rand(M, generator=g, device="cuda", dtype=dt) * 2 - 1
    x[col[nnz // 2]] = float("inf")  # stays in its rows, as do a NaN and the largest value
    x[col[nnz // 3]] = float("nan")
    x[col[nnz // 7]] = torch.finfo(dt).max
    import paper_1804_10112_amd as spt
    _check(A, row, col, vals, x, N, A.workspace(spt.SPT_OP_SPMV), f"{form} {kind} {cols} {dtype}")
    del A, keep, row, col, vals
    torch.cuda.empty_cache()


@pytest.mark.parametrize("form", ["csr", "coo"])
def test_least_workspace_and_replayed_graph(form):
    """A workspace that holds the carries of 2048 entries each, as smaller x take it, is enough; a captured call
    replays to the eager result, and the entry point with its own scratch memory gives the same."""
    import torch
    import paper_1804_10112_amd as spt
    nnz = CSR_FROM + 9 if form == "csr" else COO_FROM + 9
    N, M = 1_200_007, 1_000_003
    A, keep, row, col, vals = _matrix(form, "heavy", "scattered", N, M, nnz, torch.float64, False, 8)
    x = torch.rand(M, device="cuda", dtype=torch.float64)
    query = spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A)
    chunks = -(-nnz // 2048)
    least = -(-4 * chunks // 256) * 256 + -(-8 * chunks // 256) * 256 + 256
    assert least < query <= nnz // 15
    _check(A, row, col, vals, x, N, torch.empty(least, dtype=torch.uint8, device="cuda"), f"{form}, least workspace")
    ws = torch.empty(query, dtype=torch.uint8, device="cuda")
    _check(A, row, col, vals, x, N, ws, form)
    y = torch.zeros(N, dtype=torch.float64, device="cuda")
    spt.spt_spmv(A, x, y, ws)
    eager = y.clone()
    static = torch.full_like(y, float("nan"))
    spt.spt_spmv_static(A, x, static)
    assert torch.equal(static, eager)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        spt.spt_spmv(A, x, y, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        spt.spt_spmv(A, x, y, ws)
    for _ in range(3):
        y.fill_(float("nan"))
        ws.fill_(0xFF)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager)
        spt.spt_spmv(A, x, static, ws)
        assert torch.equal(static, eager)


BY_ROWS, BY_ENTRIES, BY_SLICES = range(3)


def _choice(ws):
    """What the flags of the device's choice, the first 256 bytes of the workspace, amount to."""
    f = ws[:256].cpu().numpy()
    heavy, scattered, tells = ((f & bit) != 0 for bit in (1, 2, 4))
    return BY_SLICES if 2 * scattered.sum() > tells.sum() else BY_ENTRIES if heavy.any() else BY_ROWS


# What is chosen, and that it is done: rows cut by segments leave carries in the workspace, the row kernel does not touch
# it. x of 8 MB: a third of it stays in an L2; of 24 MB: not. In a row of nearly all entries columns ascend, which tells nothing.
@pytest.mark.parametrize("form,kind,cols,dtype,M,want", [
    ("csr", "level", "local", "float64", 1_000_003, BY_ROWS),
    ("csr", "level", "third", "float64", 1_000_003, BY_ROWS),
    ("csr", "level", "third", "float32", 2_000_003, BY_ROWS),
    ("csr", "heavy", "local", "float32", 2_000_003, BY_ENTRIES),
    ("csr", "heavy", "third", "float32", 2_000_003, BY_ENTRIES),
    ("csr", "level", "third", "float64", 3_000_001, BY_SLICES),
    ("csr", "level", "scattered", "float32", 1_500_007, BY_SLICES),
    ("csr", "heavy", "scattered", "float64", 16_000_000, BY_SLICES),
    ("coo", "level", "local", "float32", 2_000_003, BY_ROWS),
    ("coo", "level", "third", "float32", 2_000_003, BY_ROWS),
    ("coo", "level", "scattered", "float64", 750_003, BY_SLICES),
])
def test_device_choice(form, kind, cols, dtype, M, want):
    import torch
    import paper_1804_10112_amd as spt
    nnz, dt = (CSR_FROM if form == "csr" else COO_FROM) + 7, getattr(torch, dtype)
    N = 1_200_007
    A, keep, row, col, vals = _matrix(form, kind, cols, N, M, nnz, dt, False, 9)
    x = torch.rand(M, device="cuda", dtype=dt)
    y = torch.empty(N, device="cuda", dtype=dt)
    ws = torch.full((spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A),), 0x7F, dtype=torch.uint8, device="cuda")
    spt.spt_spmv(A, x, y, ws)
    assert _choice(ws) == want
    segments = -(-nnz // SEGMENT)
    carries = 256 + -(-4 * (segments + 1) // 256) * 256  # their rows, behind the flags and the first row of each segment
    unused = (ws[carries:carries + 4 * segments].view(torch.int32) == 0x7F7F7F7F).all().item()
    assert unused == (form == "csr" and want == BY_ROWS)
    del A, keep, row, col, vals
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_declared_short_rows_are_spared_the_choice(dtype):
    """No look at the columns, no flags or carries, whatever workspace is handed over; the same sums."""
    import torch
    import paper_1804_10112_amd as spt
    nnz, N, M, dt = CSR_FROM + 7, 1_200_007, 2_000_003, getattr(torch, dtype)
    A, keep, row, col, vals = _matrix("csr", "level", "local", N, M, nnz, dt, False, 9)
    ws = torch.full((spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A),), 0x7F, dtype=torch.uint8, device="cuda")
    A.c.level[1].max_children = nnz // N + 1
    assert spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A) < ws.numel()
    x = torch.rand(M, device="cuda", dtype=dt)
    y = torch.full((N,), float("nan"), device="cuda", dtype=dt)
    spt.spt_spmv(A, x, y, ws)
    assert (ws == 0x7F).all().item()
    A.c.level[1].max_children = 0
    chosen = torch.full_like(y, float("nan"))
    spt.spt_spmv(A, x, chosen, ws)
    assert _choice(ws) == BY_ROWS and torch.equal(y, chosen)
    del A, keep, row, col, vals
    torch.cuda.empty_cache()


@pytest.mark.parametrize("form", ["csr", "coo"])
def test_beyond_the_static_scratch(form):
    """Where the library's own scratch memory no longer holds what the slices take, the call without a workspace runs
    the kernel that does with less, as spt_spmv does with a workspace of that size."""
    import torch
    import paper_1804_10112_amd as spt
    nnz = (spt.SPT_STATIC_SCRATCH_BYTES // 16 + 1) * SEGMENT
    N, M = 2_400_007, 1_000_003
    A, keep, row, col, vals = _matrix(form, "level", "scattered", N, M, nnz, torch.float64, False, 8)
    query = spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A)
    assert query > spt.SPT_STATIC_SCRATCH_BYTES
    x = torch.rand(M, device="cuda", dtype=torch.float64)
    y, least = (torch.full((N,), float("nan"), device="cuda", dtype=torch.float64) for _ in range(2))
    spt.spt_spmv_static(A, x, y)
    ref, mag = _reference(row, col, vals, x, N)
    assert_close_where_finite(y.cpu().numpy(), ref, mag, np.float64, f"{form}, static")
    spt.spt_spmv(A, x, least, torch.empty(spt.SPT_STATIC_SCRATCH_BYTES, dtype=torch.uint8, device="cuda"))
    assert torch.equal(least, y)
    _check(A, row, col, vals, x, N, torch.empty(query, dtype=torch.uint8, device="cuda"), f"{form}, workspace of the query")
    del A, keep, row, col, vals
    torch.cuda.empty_cache()
