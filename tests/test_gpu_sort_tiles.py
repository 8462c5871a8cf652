"""COO -> CSR by two partitions, at the edges of the sizes of tiles: 1024 records up to 15 * 2^17, 2048 up to 11 * 2^18,
4096 beyond. Bit for bit against a stable sort."""
import pytest

from test_gpu_sort_records import convert_and_check

pytestmark = pytest.mark.gpu

LEAST, SMALL = 15 << 17, 11 << 18


@pytest.mark.parametrize("n,rows,skewed", [
    (LEAST, 130_000, False), (LEAST + 1, 130_000, True), (LEAST + 2047, 1_000_003, False), (2_500_009, 70_001, True),
    (SMALL, 190_000, True), (SMALL + 1, 190_000, False),
])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_tiles(n, rows, skewed, dtype):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    row = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    row = ((row ** 6 if skewed else row) * rows).long().clamp_(max=rows - 1)
    convert_and_check(rows, 1 << 20, row, torch.randint(0, 1 << 20, (n,), generator=g, device="cuda"), True, dtype)
