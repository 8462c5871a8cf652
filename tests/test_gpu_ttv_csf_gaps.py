"""CSF tensor times vector by pieces of 256 entries, fibres without entries in long gaps: lengths at the edges of the groups
of 1024 that are zeroed apart and of the 4096 up to which a piece walks through its fibres, several gaps in one piece,
gaps before the first and after the last entry. The reference is the definition, its products and sums in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def tensor(K, length, dtype):
    """One slice of fibres of the given lengths (a tensor of 64-bit integers on the GPU): descriptor, arrays, c."""
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    from paper_1804_10112_amd.binding import SptTensor
    n, nnz, dt = len(length), int(length.sum()), getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(nnz + n)
    pos = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), length.cumsum(0)])
    k = torch.randint(0, K, (nnz,), generator=g, device="cuda")
    v = torch.rand(nnz, generator=g, device="cuda", dtype=dt) * 2 - 1
    c = torch.rand(K, generator=g, device="cuda", dtype=dt) * 2 - 1
    keep = [t.int().cuda() for t in (torch.tensor([0, 1]), torch.tensor([0]), torch.tensor([0, n]), torch.arange(n), pos, k)]
    B = SptTensor()
    B.order, B.nlevels = 3, 3
    B.dtype = spt.SPT_F64 if dtype == "float64" else spt.SPT_F32
    B.vals, B.nvals = v.data_ptr(), nnz
    for level, (N, M) in enumerate([(1, 1), (n, 1), (K, n)]):
        lv = B.level[level]
        lv.kind, lv.mode, lv.N, lv.M, lv.crd_stride = wl.COMPRESSED, level, N, M, 1
        lv.flags = spt.SPT_ORDERED | spt.SPT_UNIQUE
        lv.pos, lv.crd = keep[2 * level].data_ptr(), keep[2 * level + 1].data_ptr()
    return B, keep + [v], k, v, c, pos


def call(B, c, out, ws):
    import torch
    import paper_1804_10112_amd as spt
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    spt.spt_ttv(B, c, None, None, out, count, ws)
    return count


ROWS, STAGED = 1 << 19, 1 << 20
GAPS = {
    "edges": [1, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 5119, 5120, 5121, 6000],
    "long": [300_000, 1, 0, 0, 70_001, 1 << 16, (1 << 20) + 3],
    "spread": [99] * 400 + [1200] * 100 + [3] * 2000 + [1000, 1024, 1100] * 60,
}


@pytest.mark.parametrize("gaps", sorted(GAPS))
@pytest.mark.parametrize("K,nnz,dtype", [
    (30_000, ROWS + 3, "float32"),     # c in global memory
    (90_000, STAGED + 77, "float64"),
    (9_000, STAGED + 255, "float64"),  # c staged
    (9_000, STAGED + 1, "float32"),
])
def test_gaps(gaps, K, nnz, dtype):
    import torch
    import paper_1804_10112_amd as spt
    gap = torch.tensor(GAPS[gaps], device="cuda")
    # an entry after each gap, and so in the middle and at both ends of the other fibres, of one to six entries
    alone = torch.zeros(int(gap.sum()) + len(gap), dtype=torch.int64, device="cuda")
    alone[(gap + 1).cumsum(0) - 1] = 1
    rest = torch.arange((nnz - 3 * len(gap)) // 7 * 2, device="cuda") % 2 * 5 + 1
    half = len(rest) // 2
    length = torch.cat([alone, rest[:half], alone, rest[half:], alone.flip(0)])
    length[half] += nnz - int(length.sum())
    B, keep, k, v, c, pos = tensor(K, length, dtype)
    out = torch.full((len(length),), -1, dtype=v.dtype, device="cuda")
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_TTV, B), dtype=torch.uint8, device="cuda")
    count = call(B, c, out, ws)
    assert int(count[0]) == len(length)
    t = (v.double() * c.double()[k]).cpu().numpy()
    full = torch.nonzero(length).flatten()
    at = pos[full].cpu().numpy()
    ref, mag = np.add.reduceat(t, at), np.add.reduceat(np.abs(t), at)
    eps = np.finfo(np.float64 if dtype == "float64" else np.float32).eps
    got, full, n = out.cpu().numpy().astype(np.float64), full.cpu().numpy(), length.cpu().numpy()
    # a rounding per product and one per addition, in any order
    assert np.all(np.abs(got[full] - ref) <= eps * (n[full] + 1) * mag)
    got[full] = 0
    assert not got.any()


@pytest.mark.parametrize("K", [9_000, 100_000])
def test_a_gap_is_not_the_work_of_one_wave(K):
    """8M fibres without entries between two others: fibre after fibre, a wave needs 34 ms for them; all compute units, 0.1."""
    import torch
    import paper_1804_10112_amd as spt
    length = torch.full((STAGED // 4 + (8 << 20),), 4, device="cuda")
    length[STAGED // 8:STAGED // 8 + (8 << 20)] = 0
    B, keep, k, v, c, pos = tensor(K, length, "float64")
    out = torch.full((len(length),), -1, dtype=v.dtype, device="cuda")
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_TTV, B), dtype=torch.uint8, device="cuda")
    call(B, c, out, ws)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(5):
        start.record()
        call(B, c, out, ws)
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end))
    assert not out[STAGED // 8:STAGED // 8 + (8 << 20)].any()
    assert best < 3.0, best
