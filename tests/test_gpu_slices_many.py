"""SpMV with x gathered slice by slice where lanes hold 40 (fp64) and 64 (fp32) entries, the offsets and then the values in
the same registers: slices of 3.2 to 5.6 MB (the edges of the rule: test_gpu_slices_rounds.py), last rounds that few workgroups have; x holds values
whose first half looks like an offset. The reference is the definition, its products and sums in float64."""
import pytest

from test_gpu_slices import _check, _matrix

pytestmark = pytest.mark.gpu

COO_FROM, MANY = (1 << 24) + 256, 32_000_000


@pytest.mark.parametrize("form,kind,dtype,N,M,nnz,misalign", [
    ("coo", "even", "float64", 900_000, 2_621_000, COO_FROM + 1, False),
    ("coo", "heavy", "float64", 900_000, 2_622_000, COO_FROM, True),
    ("coo", "even", "float32", 900_000, 8_389_000, COO_FROM + 255, False),
    ("coo", "some empty", "float64", 15_000_000, 15_900_000, COO_FROM + 3, False),
    ("coo", "heavy", "float32", 900_000, 2_000_003, MANY - 1, True),
    ("coo", "even", "float32", 900_000, 2_000_003, MANY, False),
    ("coo", "one row", "float64", 900_000, 2_000_003, MANY + 2, False),
    ("csr", "some empty", "float64", 30_000_000, 2_000_003, 34_000_001, True),
    ("csr", "heavy", "float32", 900_000, 31_000_000, 34_000_000, False),
    ("csr", "declared", "float64", 900_000, 9_000_001, 41_943_041, False),   # a segment more than four rounds of all workgroups
    ("csr", "one row", "float32", 900_000, 2_000_003, 67_108_865, False),
])
def test_many_entries_to_a_lane(form, kind, dtype, N, M, nnz, misalign):
    import torch
    import paper_1804_10112_amd as spt
    dt = getattr(torch, dtype)
    A, keep, row, col, vals = _matrix(form, kind, "scattered", N, M, nnz, dt, misalign, nnz % 89)
    g = torch.Generator(device="cuda").manual_seed(nnz % 83)
    x = torch.rand(M, generator=g, device="cuda", dtype=dt) * 2 - 1
    if dt == torch.float64:  # first halves below 128 MB, as offsets are
        x = (x.view(torch.int64) & ~0xFFFFFFFF | torch.randint(0, 8 * M, (M,), generator=g, device="cuda")).view(torch.float64)
    else:                    # the smallest floats, whose bits are such numbers, among others
        x = torch.where(torch.rand(M, generator=g, device="cuda") < 0.5, torch.randint(0, 4 * M, (M,), generator=g, device="cuda", dtype=torch.int32).view(torch.float32), x)
    ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_SPMV, A), dtype=torch.uint8, device="cuda")
    _check(A, row, col, vals, x, N, ws, f"{form} {kind} {dtype}")
