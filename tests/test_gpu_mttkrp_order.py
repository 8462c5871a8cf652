"""MTTKRP whose chunks are taken in the order of their rows of C: entry counts and factors on both sides of the rule, slices
that hold many chunks, a few and a part of one, a share of the order's workgroups that is full, begun and cut. Built on the
GPU with small integers, whose sums are exact in any order: the reference is the definition in float64, compared bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FROM = 8_000_000   # entries


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("I,J,K,nnz,R,dtype", [
    (37, 100_000, 60_000, FROM - 1, 16, "float64"),          # in the given order
    (37, 100_000, 60_000, FROM, 16, "float64"),
    (3000, 100_000, 60_000, FROM + 2049, 16, "float32"),
    (3, 60_000, 60_000, 8192 * 1024, 33, "float64"),         # shares that are full
    (200_000, 1_000_003, 2000, FROM + 77, 8, "float64"),     # a slice is a part of a chunk
    (40, 255, 4_000_000, FROM + 3, 8, "float64"),            # fewer rows of C than bins: given order, C is small
    (400, 47_000, 47_000, FROM + 5, 32, "float32"),
])
def test_ordered_chunks(form, I, J, K, nnz, R, dtype):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    g = torch.Generator(device="cuda").manual_seed(nnz)
    dt = getattr(torch, dtype)

    def ints(n, top):
        return torch.randint(-top, top + 1, (n,), generator=g, device="cuda")

    # slices of uneven size; a third of the entries in the middle rows of C; fibres by chance
    i = (torch.rand(nnz, generator=g, device="cuda", dtype=torch.float64).square() * I).long()
    j = torch.randint(0, J, (nnz,), generator=g, device="cuda")
    j = torch.where(torch.rand(nnz, generator=g, device="cuda") < 1 / 3, j // 16 + J // 2, j)
    key = torch.sort((i * J + j) * K + torch.randint(0, K, (nnz,), generator=g, device="cuda")).values
    i, j, k = key // (J * K), key // K % J, key % K
    del key
    vals, C, D = ints(nnz, 1).to(dt), ints(J * R, 2).to(dt), ints(K * R, 2).to(dt)
    one = np.ones(1, np.float64 if dtype == "float64" else np.float32)
    i32, j32, k32 = i.int(), j.int(), k.int()
    end = torch.tensor([0, nnz], dtype=torch.int32, device="cuda")
    if form == "coo":
        B = spt.DeviceTensor(wl.coo3_spec((I, J, K), [0], [0], [0], one))
        keep = [end, i32, j32, k32]
        B.c.level[0].pos, B.c.level[0].crd, B.c.level[1].crd, B.c.level[2].crd = (t.data_ptr() for t in keep)
    else:
        B = spt.DeviceTensor(wl.csf3_spec((I, J, K), [0, 1], [0], [0, 1], [0], [0, 1], [0], one))
        fibre, length = torch.unique_consecutive(i * J + j, return_counts=True)
        slices, fibres = torch.unique_consecutive(fibre // J, return_counts=True)
        zero = torch.zeros(1, dtype=torch.int64, device="cuda")
        keep = [torch.tensor([0, len(slices)], dtype=torch.int32, device="cuda"), slices.int(),
                torch.cat([zero, fibres.cumsum(0)]).int(), (fibre % J).int(), torch.cat([zero, length.cumsum(0)]).int(), k32]
        for level in range(3):
            B.c.level[level].pos, B.c.level[level].crd = keep[2 * level].data_ptr(), keep[2 * level + 1].data_ptr()
        B.c.level[1].M, B.c.level[2].M = len(slices), len(fibre)
    B.c.vals, B.c.nvals = vals.data_ptr(), nnz
    A = torch.full((I, R), float("nan"), dtype=dt, device="cuda")
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_MTTKRP, B, R), dtype=torch.uint8, device="cuda")
    spt.spt_mttkrp(B, C, D, R, A, ws)
    want = torch.zeros(I, R, dtype=torch.float64, device="cuda")
    Cd, Dd = C.view(J, R).double(), D.view(K, R).double()
    for a in range(0, nnz, 1 << 20):
        e = slice(a, a + (1 << 20))
        rows, n = torch.unique_consecutive(i[e], return_counts=True)
        upto = (vals[e].double()[:, None] * Cd[j[e]] * Dd[k[e]]).cumsum(0)[n.cumsum(0) - 1]
        want[rows] += torch.diff(upto, dim=0, prepend=torch.zeros_like(upto[:1]))
    assert float(want.abs().max()) < 2 ** (53 if dtype == "float64" else 24)   # (and so are the partial sums: |term| <= 4)
    assert torch.equal(A.double(), want)
