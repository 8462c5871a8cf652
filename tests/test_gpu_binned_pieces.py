"""SpMV on unordered entries by bins: stretches of a bin in a tile that are a piece of 64 entries long, one less, one more,
several of them; tiles that end with a part of a vector. Small integers, whose sums are exact in any order, bit for bit."""
import pytest

from test_gpu_binned import _operand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("length,N,nnz", [
    (63, 2560, 786_432), (64, 2560, 800_001), (65, 256, 800_003), (127, 2560, 900_000), (128, 25_600, 1_100_007),
    (129, 25_600, 1_500_001), (500, 700_000, 4_000_001), (4096, 700_000, 2_000_003),
])
def test_pieces(length, N, nnz, dtype):
    import torch
    import paper_1804_10112_amd as spt
    g = torch.Generator(device="cuda").manual_seed(nnz + length)
    dt = getattr(torch, dtype)
    at = torch.arange(nnz, device="cuda")
    # `length` entries in a row go to one bin, the next ones to another
    row = (at // length * 97 % 256) * (N // 256) + torch.randint(0, N // 256, (nnz,), generator=g, device="cuda")
    col = torch.randint(0, 5000, (nnz,), generator=g, device="cuda")
    vals = torch.randint(-2, 3, (nnz,), generator=g, device="cuda").to(dt)
    x = torch.randint(-3, 4, (5000,), generator=g, device="cuda").to(dt)
    A, keep = _operand("coo", N, 5000, row, col, row.int(), col.int(), vals)
    y = torch.full((N,), float("nan"), device="cuda", dtype=dt)
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A), dtype=torch.uint8, device="cuda")
    spt.spt_spmv(A, x, y, ws)
    want = torch.bincount(row, (vals * x[col]).double(), N)
    assert torch.equal(y.double(), want)
