"""MTTKRP whose columns are split into parts of whole lines: entry counts on both sides of the rule, two, four and eight parts,
parts of more than a line and of lines that leave lanes idle, chunks in the order of their rows of C, rows that cannot be split, factors that do not lie on lines."""
import pytest

import test_gpu_mttkrp_order as order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["coo", "csf"])
@pytest.mark.parametrize("I,J,K,nnz,R,dtype", [
    (97, 20_011, 16_001, 195_312, 32, "float64"),       # too few entries
    (97, 20_011, 16_001, 195_313, 32, "float64"),       # two parts
    (30_011, 20_011, 16_001, 400_003, 64, "float32"),
    (3, 20_011, 16_001, 1_000_003, 32, "float64"),      # rows of many chunks of each part
    (97, 20_011, 16_001, 97_657, 64, "float64"),        # four
    (97, 9_001, 9_001, 97_657, 128, "float32"),
    (97, 5_003, 5_001, 100_003, 256, "float32"),        # eight
    (97, 3_001, 2_003, 100_003, 512, "float32"),        # eight of two lines
    (97, 9_001, 9_001, 97_657, 96, "float32"),          # three lines: one part
    (97, 9_001, 9_001, 97_657, 96, "float64"),          # two of three lines, lanes idle
    (97, 4_001, 4_003, 97_657, 192, "float64"),         # (factors too small for that)
    (97, 9_001, 9_001, 97_657, 192, "float64"),         # four
    (97, 9_001, 9_001, 97_657, 160, "float64"),         # two would be of five lines: one part
    (97, 9_001, 9_001, 97_657, 320, "float64"),         # two of ten lines
    (97, 4_001, 4_003, 50_021, 384, "float64"),         # two of twelve lines
    (97, 9_001, 9_001, 50_021, 384, "float64"),         # eight of three lines
    (3, 9_001, 9_001, 50_021, 640, "float64"),          # four of ten lines
    (97, 9_001, 9_001, 97_657, 384, "float32"),
    (97, 9_001, 9_001, 50_021, 768, "float32"),
    (97, 20_011, 16_001, 400_003, 33, "float64"),
    (400, 47_000, 47_000, 8_000_005, 32, "float64"),    # ordered
])
def test_parts(form, I, J, K, nnz, R, dtype):
    order.test_ordered_chunks(form, I, J, K, nnz, R, dtype)


@pytest.mark.parametrize("shift_c,shift_d", [(1, 0), (0, 1), (16, 0), (0, 8)])
def test_factors_off_the_lines(shift_c, shift_d):
    """A factor that begins between two lines is not split; small integers, whose sums are exact in any order."""
    import numpy as np
    import torch
    import paper_1804_10112_amd as spt
    import workloads as wl
    I, J, K, nnz, R = 97, 20_011, 16_001, 400_003, 32
    rng = np.random.default_rng(5)
    key = np.sort(rng.integers(0, I * J * K, nnz))
    i, j, k = (x.astype(np.int32) for x in (key // (J * K), key // K % J, key % K))
    B = spt.DeviceTensor(wl.coo3_spec((I, J, K), i, j, k, rng.integers(-1, 2, nnz).astype(np.float64)))
    C, D = (torch.from_numpy(rng.integers(-2, 3, n * R).astype(np.float64)).cuda() for n in (J, K))
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_MTTKRP, B, R), dtype=torch.uint8, device="cuda")
    got = []
    for sc, sd in ((0, 0), (shift_c, shift_d)):
        Cs, Ds = (torch.cat([torch.zeros(k, device="cuda", dtype=torch.float64), f])[k:] for k, f in ((sc, C), (sd, D)))
        A = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
        spt.spt_mttkrp(B, Cs, Ds, R, A, ws)
        got.append(A)
    assert torch.equal(*got)
    assert bool(got[0].abs().sum() > 0)
