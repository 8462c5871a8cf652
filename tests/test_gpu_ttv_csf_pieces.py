"""CSF tensor times vector by pieces of 256 entries with c in global memory: entry counts at the rules' edges (2^19 and
2^20 entries; a c of which less than a quarter is held; 32 768 pieces), ends of a piece, empty fibres before, between and
after the others, arrays that are not 16-byte aligned, and a workspace that only the reduction by rows can do with. The
reference is the definition, its products and sums in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS, STAGED = 1 << 19, 1 << 20


@pytest.mark.parametrize("fibres,K,nnz,dtype,misalign,small", [
    ("short", 9000, ROWS - 1, "float32", False, False),
    ("short", 9000, ROWS, "float32", False, False),
    ("empty", 9000, ROWS + 1, "float64", True, False),
    ("one", 9000, ROWS + 255, "float32", False, False),
    ("each", 30_000, STAGED - 1, "float32", True, False),
    ("empty", 30_000, STAGED, "float32", False, False),
    ("empty", 70_000, ROWS + 257, "float64", False, False),
    ("each", 70_000, STAGED + 3, "float64", True, False),
    ("mixed", 130_000, STAGED + 256, "float32", True, False),
    ("mixed", 70_000, STAGED + 5, "float64", False, True),
    ("mixed", 70_000, 32767 * 256 + 1, "float64", False, False),
    ("empty", 70_000, 32768 * 256 + 1, "float64", False, False),
])
def test_ttv_csf_pieces(fibres, K, nnz, dtype, misalign, small):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    from paper_1804_10112_amd.binding import SptTensor
    g = torch.Generator(device="cuda").manual_seed(nnz)
    head = torch.rand(nnz, generator=g, device="cuda") < {"short": 0.4, "mixed": 0.01, "empty": 0.1, "one": 0.0, "each": 1.0}[fibres]
    if fibres == "mixed":  # long fibres, and a stretch in which every entry is one
        head[nnz // 3:nnz // 3 + 5000] = True
    head[0] = True
    at = torch.nonzero(head).flatten()
    copies = torch.ones(len(at), dtype=torch.int64, device="cuda")
    if fibres == "empty":  # a fibre begins here after as many empty ones
        copies += (torch.rand(len(at), generator=g, device="cuda") < 0.2) * torch.randint(1, 300, (len(at),), generator=g, device="cuda")
        copies[0] += 777
    owner = copies.cumsum(0) - 1  # the fibre that holds the entries, last of those that begin there
    pos = torch.cat([at.repeat_interleave(copies), torch.full((600 if fibres == "empty" else 1,), nnz, device="cuda")])
    n = len(pos) - 1
    dt = getattr(torch, dtype)
    k = torch.randint(0, K, (nnz,), generator=g, device="cuda")
    vals = torch.rand(nnz, generator=g, device="cuda", dtype=dt) * 2 - 1
    c = torch.rand(K, generator=g, device="cuda", dtype=dt) * 2 - 1

    def place(t):  # at the start of its allocation, or one element further
        out = torch.empty(len(t) + 1, dtype=t.dtype, device="cuda")[int(misalign):][:len(t)]
        out.copy_(t)
        return out

    ints = [place(t.int()) for t in (torch.tensor([0, 1]), torch.tensor([0]), torch.tensor([0, n]), torch.arange(n), pos, k)]
    v = place(vals)
    B = SptTensor()
    B.order, B.nlevels = 3, 3
    B.dtype = spt.SPT_F64 if dtype == "float64" else spt.SPT_F32
    B.vals, B.nvals = v.data_ptr(), nnz
    for level, (N, M) in enumerate([(1, 1), (n, 1), (K, n)]):
        lv = B.level[level]
        lv.kind, lv.mode, lv.N, lv.M, lv.crd_stride = wl.COMPRESSED, level, N, M, 1
        lv.flags = spt.SPT_ORDERED | spt.SPT_UNIQUE
        lv.pos, lv.crd = ints[2 * level].data_ptr(), ints[2 * level + 1].data_ptr()
    out, count = torch.full((n,), -1, dtype=dt, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    need = spt.spt_workspace_bytes(spt.SPT_OP_TTV, B)
    ws = torch.empty(need // 4 if small else need, dtype=torch.uint8, device="cuda")
    spt.spt_ttv(B, c, None, None, out, count, ws)
    assert int(count[0]) == n
    t = (vals.double() * c.double()[k]).cpu().numpy()
    at = at.cpu().numpy()
    ref, mag = np.add.reduceat(t, at), np.add.reduceat(np.abs(t), at)
    length = np.diff(np.append(at, nnz))
    eps = np.finfo(np.float64 if dtype == "float64" else np.float32).eps
    got = out.cpu().numpy().astype(np.float64)
    owner = owner.cpu().numpy()
    # a rounding per product and one per addition, in any order
    assert np.all(np.abs(got[owner] - ref) <= eps * (length + 1) * mag)
    got[owner] = 0
    assert not got.any()
