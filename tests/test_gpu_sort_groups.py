"""COO -> CSR by two partitions: the counts of tiles by workgroups of one tile, four, and four by twice the threads (from 2048 tiles
of 4096 records on, up to 4096), and the edges of the sizes of tiles where rows are short. Bit for bit against a stable sort."""
import pytest

from test_gpu_sort_records import convert_and_check

pytestmark = pytest.mark.gpu

ONE, WIDE = 2047 * 4096, 4095 * 4096
LEAST, SMALL = 15 << 17, 11 << 18


@pytest.mark.parametrize("n,rows,skewed", [
    (ONE, 700_001, False), (ONE + 1, 700_001, True), (ONE + 4097, 3_000_017, False), (WIDE, 1_000_003, True), (WIDE + 1, 1_000_003, False),
    (9_000_011, 40_003, True), (LEAST, 900_001, True), (LEAST + 1, 900_001, False), (SMALL, 900_001, False), (SMALL + 1, 900_001, True),
])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_groups_of_tiles(n, rows, skewed, dtype):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    row = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    row = ((row ** 6 if skewed else row) * rows).long().clamp_(max=rows - 1)
    convert_and_check(rows, 1 << 22, row, torch.randint(0, 1 << 22, (n,), generator=g, device="cuda"), True, dtype)
