"""COO -> CSR by two partitions: buckets whose keys take 32 bits from their lower bound on, and buckets whose keys do not
(a segment has records of 4 or 8 bytes of key). Up to 3M records whose keys and positions take 64 bits that is the sort with less
workspace than the query's; both run. Built on the GPU; the reference is a stable sort, bit for bit."""
import numpy as np
import pytest

from gpu_util import conversion_workspaces

pytestmark = pytest.mark.gpu


def convert_and_check(N, M, row, col, by_col, dtype):
    """row, col: 64-bit integers on the GPU."""
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    n = len(row)
    vals = torch.arange(n, device="cuda").to(getattr(torch, dtype))  # (the place in the input, as far as 24 bits go)
    one = np.ones(1, np.float64 if dtype == "float64" else np.float32)
    A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], one, ordered=False))
    row32, col32, end = row.int(), col.int(), torch.tensor([0, n], dtype=torch.int32, device="cuda")
    A.c.level[0].pos, A.c.level[0].crd, A.c.level[1].crd = end.data_ptr(), row32.data_ptr(), col32.data_ptr()
    A.c.vals, A.c.nvals = vals.data_ptr(), n
    at = torch.sort(row * M + col if by_col else row, stable=True).indices
    want = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    want[1:] = torch.bincount(row, minlength=N).cumsum(0)
    for ws in conversion_workspaces(A, n):
        pos = torch.full((N + 1,), -1, dtype=torch.int32, device="cuda")
        crd, out = torch.full((n,), -1, dtype=torch.int32, device="cuda"), torch.full_like(vals, -1)
        spt.spt_coo_to_csr(A, spt.SPT_ORDER_ROW_COL if by_col else spt.SPT_ORDER_ROW_STABLE, pos, crd, out, ws)
        assert torch.equal(pos.long(), want)
        assert torch.equal(crd, col32[at])
        assert torch.equal(out, vals[at])


@pytest.mark.parametrize("what,by_col,N,M,n", [
    ("narrow", True, 50_000, 1 << 20, 400_001),
    ("wide", True, 5_000_011, (1 << 31) - 1, 400_001),       # 2^42 places to a bucket
    ("around", True, 250_007, 1 << 22, 500_003),             # some 0.7 x 2^32 to a bucket: segments of either kind
    ("around", True, 2_000_003, 1 << 22, 4_000_001),         # the same with tiles of 4096
    ("cluster", True, 3_000_017, (1 << 31) - 1, 900_001),    # half of the records in few rows and columns
    ("one bit short", False, 80_021, 1 << 24, 500_003),      # by row: 24 bits of column leave 256 rows to a narrow bucket
    ("wide", False, 80_021, (1 << 31) - 1, 500_003),         # 31 leave one
    ("two rows", False, 70_001, (1 << 31) - 1, 500_003),     # nearly all records in two rows: equal keys
])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_narrow_and_wide(what, by_col, N, M, n, dtype):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    row = torch.randint(0, N, (n,), generator=g, device="cuda")
    col = torch.randint(0, M, (n,), generator=g, device="cuda")
    half = torch.rand(n, generator=g, device="cuda") < 0.5
    if what == "cluster":
        row, col = torch.where(half, row % 1000 + N // 2, row), torch.where(half, col % 5000, col)
    elif what == "two rows":
        row = torch.where(torch.rand(n, generator=g, device="cuda") < 0.99, N // 3 + half.long(), row)
    row[0], col[0], row[1], col[1] = 0, 0, N - 1, M - 1
    convert_and_check(N, M, row, col, by_col, dtype)
