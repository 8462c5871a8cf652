"""MTTKRP of rows that take 16 lanes: entry counts where groups go from 16 entries to 48 and from 48 to 64 (a batch of the
coordinates that the lanes hold is 64)."""
import pytest

import test_gpu_mttkrp_order as order

pytestmark = pytest.mark.gpu

CSF, COO, TWO = 4 * 256 * 256, 5 * 256 * 256, 2 * 256 * 16 * 48


@pytest.mark.parametrize("form,nnz", [("csf", CSF), ("csf", CSF + 1), ("csf", TWO), ("csf", TWO + 1),
                                      ("coo", COO), ("coo", COO + 1), ("coo", TWO), ("coo", TWO + 1), ("coo", 450 * 768 + 47)])
@pytest.mark.parametrize("R,dtype", [(32, "float64"), (64, "float32"), (31, "float64")])
def test_groups(form, nnz, R, dtype):
    order.test_ordered_chunks(form, 97, 5003, 7001, nnz, R, dtype)
