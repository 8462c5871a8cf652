"""COO -> CSR at the sizes where the sample sort's plan changes (up to 3M records with less workspace than the query's, too, with
which the sort by reserved regions runs): tiles of 1024, 2048 and 4096 records, one partition or two, samples of
1024 to 4096, buckets that take four, six, eight and sixteen words of a thread, and counts whose rows end off 16 bytes.
Built on the GPU; the reference is a stable sort, bit for bit."""
import numpy as np
import pytest

from gpu_util import conversion_workspaces

pytestmark = pytest.mark.gpu

SELECT, SMALL, ONE, LARGE = 64 * 1024, 128 * 1024, 256 * 1408, 11 << 18  # one launch; tiles of 1024; one partition; tiles of 4096


@pytest.mark.parametrize("keys,by_col,n,dtype", [
    # one launch: the picked records lie in a few words of a bit set (input in order), or in all of them
    ("sorted", True, 385, "float64"),
    ("random", True, 769, "float32"),
    ("random", False, 3000, "float64"),
    ("sorted", False, 20_000, "float32"),
    ("equal", True, 33_001, "float64"),
    ("skewed", True, 50_021, "float32"),
    ("sorted", True, SELECT, "float64"),
    ("random", True, SELECT, "float64"),
    ("random", True, SELECT + 1, "float64"),
    ("random", False, SMALL, "float32"),
    ("random", True, SMALL + 1, "float64"),
    ("equal", True, SMALL + 2049, "float64"),
    ("random", True, ONE, "float32"),
    ("skewed", True, ONE + 1, "float64"),
    ("sorted", True, 64 * 16 * 1408 + 1, "float64"),
    ("skewed", False, 128 * 16 * 1408 + 77, "float32"),
    ("random", True, LARGE, "float64"),
    ("skewed", True, LARGE + 1, "float64"),
    ("equal", False, LARGE + 4097, "float32"),
    ("random", True, 6_000_011, "float32"),
])
def test_sizes(keys, by_col, n, dtype):
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    N, M = n // 9 + 3, 3_000_017
    g = torch.Generator(device="cuda").manual_seed(n)
    row = torch.randint(0, N, (n,), generator=g, device="cuda")
    col = torch.randint(0, M, (n,), generator=g, device="cuda")
    if keys == "skewed":  # a third in one row, an eighth at one place
        row = torch.where(torch.rand(n, generator=g, device="cuda") < 1 / 3, N // 2, row)
        same = torch.rand(n, generator=g, device="cuda") < 1 / 8
        row, col = torch.where(same, N - 2, row), torch.where(same, M // 3, col)
    elif keys == "equal":
        row, col = torch.full_like(row, N - 1), torch.full_like(col, 5)
    elif keys == "sorted":
        row = row.sort().values
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
