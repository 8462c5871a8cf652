"""SpMV with x gathered slice by slice, at the edges of the rule that gives a lane 32 entries or 40 (fp64) and 64 (fp32): by
the rounds that the chip makes over x, and by the size of x where they look at about as many registers."""
import pytest

import test_gpu_slices_many as many

pytestmark = pytest.mark.gpu

ROUND = 1024 * 256 * 32  # entries of all lanes, 32 to each


@pytest.mark.parametrize("form,kind,dtype,N,M,nnz", [
    ("coo", "heavy", "float64", 900_000, 1_600_001, 3 * ROUND),           # three rounds with either
    ("coo", "heavy", "float64", 900_000, 1_600_001, 3 * ROUND + 1),       # four, or three of 40
    ("coo", "even", "float64", 900_000, 1_000_003, 3 * ROUND + 257),      # the same with a small x
    ("coo", "even", "float64", 900_000, 1_000_003, 2 * ROUND + 300),      # three, or two of 40: x is too small
    ("coo", "one row", "float64", 900_000, 5_100_000, 4 * ROUND),         # four with either
    ("coo", "one row", "float64", 900_000, 5_100_000, 4 * ROUND + 3),     # five of 32 look at as much as four of 40: by x
    ("coo", "some empty", "float64", 900_000, 4_900_000, 4 * ROUND + 3),
    ("coo", "some empty", "float32", 900_000, 9_100_000, 2 * ROUND + 300),
    ("coo", "heavy", "float32", 900_000, 8_900_000, 3 * ROUND),           # three, or two of 64
    ("coo", "heavy", "float32", 900_000, 8_900_000, 3 * ROUND + 2),       # four
    ("csr", "heavy", "float64", 900_000, 1_400_001, 4 * ROUND + 5),
    ("csr", "heavy", "float64", 900_000, 1_600_001, 4 * ROUND + 5),
])
def test_edges(form, kind, dtype, N, M, nnz):
    many.test_many_entries_to_a_lane(form, kind, dtype, N, M, nnz, False)
