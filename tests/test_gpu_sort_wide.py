"""COO -> CSR by two partitions, inputs whose first sample sees none of most records: all those lie in one segment, whose
buckets are then larger than the last sort's arrays or than its LDS, with records of 64-bit keys and of 32-bit ones, with
different keys and with equal ones; and entry counts at which the rows' radix passes take over. Bit for bit against a
stable sort."""
import numpy as np
import pytest

import test_gpu_sort_records as records

pytestmark = pytest.mark.gpu

TARGET = 1408  # records that a bucket aims at


def sampled(n):
    """Positions that the first level samples out of n records."""
    nb = min(256, -(-n // (16 * TARGET)))
    S = next(s for s in (1024, 2048, 4096) if 16 * nb <= s or s == 4096)
    t = np.arange(S, dtype=np.uint64)
    jitter = (t * np.uint64(2654435769) % np.uint64(1 << 32)) >> np.uint64(16)
    return (((t << np.uint64(16)) | jitter) * np.uint64(n) // np.uint64(S) >> np.uint64(16)).astype(np.int64)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("keys,by_col,M,n", [
    ("any", True, (1 << 31) - 1, 640_003),       # 64-bit keys, buckets of some 2500 records: beyond 2048
    ("any", True, (1 << 31) - 1, 1_200_007),     # of 4700: split once more (beyond 3072)
    ("equal", True, (1 << 31) - 1, 1_200_007),
    ("few", True, (1 << 31) - 1, 1_000_003),
    ("any", True, 4000, 1_200_007),              # 32-bit keys: beyond 3584
    ("equal", True, 4000, 880_001),
    ("any", False, (1 << 31) - 1, 1_200_007),    # rows alone
])
def test_buckets_that_do_not_fit(keys, by_col, M, n, dtype):
    import torch
    N = 3_000_017
    g = torch.Generator(device="cuda").manual_seed(n + M)
    row = torch.randint(0, N // 2, (n,), generator=g, device="cuda")
    col = torch.randint(0, M, (n,), generator=g, device="cuda")
    if keys == "equal":
        row, col = torch.full_like(row, 77), torch.full_like(col, M // 3)
    elif keys == "few":  # three hundred places
        row, col = row % 300 * 5000, torch.full_like(col, M - 2)
    at = torch.from_numpy(sampled(n)).cuda()
    row[at] = torch.randint(N // 2, N, (len(at),), generator=g, device="cuda")
    records.convert_and_check(N, M, row, col, by_col, dtype)


@pytest.mark.parametrize("n", [3 << 19, (3 << 19) + 1, 7 << 18, (7 << 18) + 1])
@pytest.mark.parametrize("by_col,N,M", [(False, 70_001, 1 << 22), (False, 16_000_000, 1 << 22), (True, 65_536, 256)])
def test_where_three_passes_take_over(by_col, N, M, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n + N)
    row = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64).square() * N).long()
    records.convert_and_check(N, M, row, torch.randint(0, M, (n,), generator=g, device="cuda"), by_col, "float64")
