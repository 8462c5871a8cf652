"""COO tensor times vector where the offsets of the results come from groups of pieces: entry counts at the edges of
pieces (256 entries), groups (16 and 32 pieces) and of the rules (6144 pieces, 10752 and 12288 where little or nothing of c is held; 98304). Built on the
GPU; the reference is the definition, its products and sums in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FROM, PIECE = 6144 * 256, 256


@pytest.mark.parametrize("fibres,K,nnz,dtype,misalign", [
    ("short", 9000, FROM, "float32", False),
    ("short", 9000, FROM + 1, "float32", False),
    ("mixed", 25_000, FROM + PIECE, "float64", True),
    ("mixed", 40_000, FROM + PIECE, "float64", True),
    ("short", 40_000, FROM // 4 * 7, "float64", False),
    ("mixed", 40_000, FROM // 4 * 7 + 1, "float64", True),
    ("mixed", 9000, FROM + 15 * PIECE + 3, "float64", False),
    ("one", 9000, FROM + 16 * PIECE, "float32", False),
    ("each", 50_000, FROM + 17 * PIECE - 1, "float32", True),
    ("mixed", 200_000, 2 * FROM, "float64", False),
    ("short", 200_000, 2 * FROM + 5, "float32", False),
    ("mixed", 9000, 16 * FROM - 1, "float32", False),
    ("mixed", 9000, 16 * FROM + 31 * PIECE + 7, "float32", True),
])
def test_ttv_groups(fibres, K, nnz, dtype, misalign):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    g = torch.Generator(device="cuda").manual_seed(nnz)
    I, J = 3000, nnz
    start = {"short": 0.4, "mixed": 0.01, "one": 0.0, "each": 1.0}[fibres]
    head = torch.rand(nnz, generator=g, device="cuda") < start
    if fibres == "mixed":  # long fibres, and a stretch in which every entry is one
        head[nnz // 3:nnz // 3 + 5000] = True
    head[0] = True
    fibre = head.cumsum(0) - 1
    n = int(fibre[-1]) + 1
    i, j = fibre * I // n, fibre  # ascending
    k = torch.randint(0, K, (nnz,), generator=g, device="cuda")
    dt = getattr(torch, dtype)
    vals = torch.rand(nnz, generator=g, device="cuda", dtype=dt) * 2 - 1
    c = torch.rand(K, generator=g, device="cuda", dtype=dt) * 2 - 1

    def place(t):  # at the start of its allocation, or one element further
        out = torch.empty(len(t) + 1, dtype=t.dtype, device="cuda")[int(misalign):][:len(t)]
        out.copy_(t)
        return out

    arrays = [place(t.int()) for t in (i, j, k)] + [place(vals)]
    one = np.ones(1, np.float64 if dtype == "float64" else np.float32)
    B = spt.DeviceTensor(wl.coo3_spec((I, J, K), [0], [0], [0], one))
    pos = torch.tensor([0, nnz], dtype=torch.int32, device="cuda")
    B.c.level[0].pos = pos.data_ptr()
    for level in range(3):
        B.c.level[level].crd = arrays[level].data_ptr()
    B.c.vals, B.c.nvals = arrays[3].data_ptr(), nnz
    oi, oj = (torch.full((nnz,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ov, count = torch.full((nnz,), -1, dtype=dt, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_TTV, B), dtype=torch.uint8, device="cuda")
    spt.spt_ttv(B, c, oi, oj, ov, count, ws)
    at = torch.nonzero(head).flatten()
    assert int(count[0]) == n
    assert torch.equal(oi[:n].long(), i[at]) and torch.equal(oj[:n].long(), j[at])
    t = (vals.double() * c.double()[k]).cpu().numpy()
    at = at.cpu().numpy()
    ref, mag = np.add.reduceat(t, at), np.add.reduceat(np.abs(t), at)
    length = np.diff(np.append(at, nnz))
    eps = np.finfo(np.float64 if dtype == "float64" else np.float32).eps
    got = ov[:n].cpu().numpy().astype(np.float64)
    # a rounding per product and one per addition, in any order
    assert np.all(np.abs(got - ref) <= eps * (length + 1) * mag)
