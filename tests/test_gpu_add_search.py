"""Addition of COO operands, numbers of tiles at which the search for their ends changes: by a wave, by 16 lanes, and with
the last coordinate fetched only where the others are the same. Rows long enough that most comparisons need it, and rows of
a few entries; half of the coordinates in both operands. Bit for bit against the definition."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STEP = 2047  # places of a tile


@pytest.mark.parametrize("places", [128 * STEP, 128 * STEP + 1, 400 * STEP, 400 * STEP + 1, 401 * STEP + 7])
@pytest.mark.parametrize("dims", [(3, 4_000_000), (90_000, 90_000), (3, 40, 100_000), (100, 300, 300)])
def test_union(places, dims):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    g = torch.Generator(device="cuda").manual_seed(places + len(dims))
    size = int(np.prod(dims))
    keys = torch.randperm(size, generator=g, device="cuda") if size < 20_000_000 else torch.unique(
        torch.randint(0, size, (2 * places,), generator=g, device="cuda"))
    keys = keys[torch.randperm(len(keys), generator=g, device="cuda")][: places - places // 3]
    kb = keys[: places - places // 2].sort().values              # the two overlap in a sixth of the places
    kc = keys[len(keys) - places // 2:].sort().values
    assert len(kb) + len(kc) == places

    def operand(k):
        one = np.ones(1, np.float64)
        spec = wl.coo_spec(*dims, [0], [0], one) if len(dims) == 2 else wl.coo3_spec(dims, [0], [0], [0], one)
        A = spt.DeviceTensor(spec)
        crd, rest = [], k
        for n in reversed(dims):
            crd.insert(0, (rest % n).int())
            rest = rest // n
        v = torch.rand(len(k), generator=g, device="cuda", dtype=torch.float64)
        end = torch.tensor([0, len(k)], dtype=torch.int32, device="cuda")
        A.c.level[0].pos = end.data_ptr()
        for level, c in enumerate(crd):
            A.c.level[level].crd = c.data_ptr()
        A.c.vals, A.c.nvals = v.data_ptr(), len(k)
        return A, [end, v] + crd, v

    (B, keep_b, vb), (C, keep_c, vc) = operand(kb), operand(kc)
    out = [torch.full((places,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
    vals, count = torch.zeros(places, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = torch.empty(spt.spt_add_workspace_bytes(B, C), dtype=torch.uint8, device="cuda")
    spt.spt_add(B, C, None, out[0], out[1], out[2] if len(dims) == 3 else None, vals, count, ws)
    want = torch.unique(torch.cat([kb, kc]))
    n = len(want)
    assert int(count[0]) == n and n < places
    got = out[0][:n].long()
    for level in range(1, len(dims)):
        got = got * dims[level] + out[level][:n]
    assert torch.equal(got, want)
    sums = torch.zeros(n, dtype=torch.float64, device="cuda")
    sums[torch.searchsorted(want, kb)] = vb
    sums[torch.searchsorted(want, kc)] += vc
    assert torch.equal(vals[:n], sums)
