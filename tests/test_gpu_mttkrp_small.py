"""MTTKRP where the entries of a group change with the size: 4, 8, 16 and 32 of them, one batch of the coordinates that its lanes
hold, rows of four or eight entries in flight together, carries added up in one launch or two; and with the least workspace, which
holds the carries of 16 entries to a group."""
import re

import pytest

import test_gpu_mttkrp_order as order

pytestmark = pytest.mark.gpu

# two workgroups to a compute unit with 4 entries to a group, three with 8, three with 16 (16 lanes: four)
EDGES = {lanes: (512 * 4 * (256 // lanes), 768 * 8 * (256 // lanes), (1024 if lanes == 16 else 768) * 16 * (256 // lanes)) for lanes in (2, 4, 8, 16, 32)}


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("R,dtype,lanes", [(8, "float32", 2), (5, "float32", 2), (4, "float64", 2), (16, "float32", 4), (3, "float32", 4),
                                           (32, "float32", 8), (16, "float64", 8), (33, "float32", 16), (33, "float64", 32)])
@pytest.mark.parametrize("edge", [0, 1, 2])
@pytest.mark.parametrize("more", [0, 1])
def test_entries_of_a_group(form, R, dtype, lanes, edge, more):
    order.test_ordered_chunks(form, 97, 503, 701, EDGES[lanes][edge] + more, R, dtype)


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("I,J,K,nnz,R,dtype", [
    (3, 11, 13, 1, 16, "float64"), (3, 11, 13, 7, 8, "float32"), (5, 17, 19, 130, 70, "float64"),
    (40_011, 503, 701, 50_021, 32, "float32"),              # rows of one entry
    (1, 503, 701, 300_007, 16, "float64"),                  # one row of all carries
    (3, 503, 701, 60_001, 200, "float64"),                  # four workgroups side by side
    (3, 5003, 701, 4096 * 1024, 8, "float32"), (3, 5003, 701, 4096 * 1024 + 1, 8, "float32"),  # one launch for the carries of COO, two
    (3, 5003, 701, 4096 * 2048 + 1, 8, "float32"),          # (of CSF)
    (3, 5003, 701, 2560 * 2048, 32, "float32"), (3, 5003, 701, 2560 * 2048 + 1, 32, "float32"),
])
def test_few_and_many(form, I, J, K, nnz, R, dtype):
    order.test_ordered_chunks(form, I, J, K, nnz, R, dtype)


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("J,K,nnz,R,dtype", [(503, 701, 50_021, 16, "float64"), (503, 701, 150_001, 8, "float32"), (5003, 701, 1_500_001, 8, "float32"),
                                             (503, 701, 40_001, 33, "float64"), (20_011, 16_001, 400_003, 32, "float64")])
def test_least_workspace(form, J, K, nnz, R, dtype):
    """Small integers, whose sums are exact in any order."""
    import numpy as np
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    I = 97
    rng = np.random.default_rng(5)
    key = np.unique(rng.integers(0, I * J * K, nnz))
    i, j, k = (x.astype(np.int32) for x in (key // (J * K), key // K % J, key % K))
    v = rng.integers(-1, 2, len(key)).astype(dtype)
    B = spt.DeviceTensor((wl.coo3_spec if form == "coo" else wl.csf3_from_sorted_coo)((I, J, K), i, j, k, v))
    C, D = (torch.from_numpy(rng.integers(-2, 3, n * R).astype(dtype)).cuda() for n in (J, K))
    with pytest.raises(Exception) as refused:
        spt.spt_mttkrp(B, C, D, R, torch.empty(I, R, dtype=C.dtype, device="cuda"), torch.empty(256, dtype=torch.uint8, device="cuda"))
    least = int(re.search(r"workspace of (\d+) bytes", str(refused.value)).group(1))
    asked = spt.spt_workspace_bytes(spt.SPT_OP_MTTKRP, B, R)
    assert 256 < least <= asked and (least < asked or nnz > 150_001)   # (more entries: the best plan may be one of few carries)
    got = []
    for room in (asked, max(asked - 1, least), least):
        A = torch.full((I, R), float("nan"), dtype=C.dtype, device="cuda")
        spt.spt_mttkrp(B, C, D, R, A, torch.empty(room, dtype=torch.uint8, device="cuda"))
        got.append(A)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    assert bool(got[0].abs().sum() > 0)
    with pytest.raises(Exception):
        spt.spt_mttkrp(B, C, D, R, got[0], torch.empty(least - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("more", [0, 1, 20_000])
def test_offsets_of_rows(form, more):
    """Factors of 4 GiB, whose rows are found at offsets of 32 bits, and of more."""
    order.test_ordered_chunks(form, 97, (1 << 23) + more, 503, 30_011, 64, "float64")


@pytest.mark.parametrize("R,dtype", [(32, "float32"), (16, "float64"), (8, "float32"), (33, "float64")])
@pytest.mark.parametrize("nnz", [9_001, 150_001, 700_003])
def test_empty_segments(R, dtype, nnz):
    """CSF whose slices and fibres are empty here and there, first fibres of a slice among them, against the same entries in COO."""
    import numpy as np
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    I, J, K = 211, 503, 701
    rng = np.random.default_rng(nnz)
    key = np.unique(rng.integers(0, I * J * K, nnz))
    i, j, k = (x.astype(np.int32) for x in (key // (J * K), key // K % J, key % K))
    v = rng.integers(-1, 2, len(key)).astype(dtype)
    C, D = (torch.from_numpy(rng.integers(-2, 3, n * R).astype(dtype)).cuda() for n in (J, K))
    got = []
    for spec in (wl.coo3_spec((I, J, K), i, j, k, v), wl.csf3_with_empty_segments((I, J, K), i, j, k, v, 7, 400, 40)):
        B = spt.DeviceTensor(spec)
        A = torch.full((I, R), float("nan"), dtype=C.dtype, device="cuda")
        spt.spt_mttkrp(B, C, D, R, A, B.workspace(spt.SPT_OP_MTTKRP, R))
        got.append(A)
    assert torch.equal(*got) and bool(got[0].abs().sum() > 0)
