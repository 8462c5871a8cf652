"""COO -> CSR by reserved regions: the lines of its plan, buckets that a workgroup or a region does not hold, keys that do
not fit, and workspaces below the query, against a stable sort on the host."""
import numpy as np
import pytest
import torch

import paper_1804_10112_amd as spt
from paper_1804_10112_amd.binding import SptTensor

pytestmark = pytest.mark.gpu


def _coo(row, col, vals, N, M):
    dev = [torch.from_numpy(a).cuda() for a in (np.array([0, len(row)], np.int32), row, col, vals)]
    t = SptTensor()
    t.order, t.nlevels, t.dtype = 2, 2, spt.SPT_F64 if vals.dtype == np.float64 else spt.SPT_F32
    t.vals, t.nvals = dev[3].data_ptr(), len(row)
    for k, (kind, n) in enumerate(((1, N), (2, M))):
        lv = t.level[k]
        lv.kind, lv.mode, lv.N, lv.M, lv.flags, lv.crd_stride = kind, k, n, 1 - k, 0, 1
        lv.crd = dev[1 + k].data_ptr()
    t.level[0].pos = dev[0].data_ptr()
    return t, dev


def _check(row, col, vals, N, M, order=spt.SPT_ORDER_ROW_COL, ws_bytes=None):
    A, keep = _coo(row, col, vals, N, M)
    n = len(row)
    pos = torch.full((N + 1,), -1, dtype=torch.int32, device="cuda")
    crd = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    out = torch.zeros(n, dtype=keep[3].dtype, device="cuda")
    ws = torch.empty(ws_bytes or spt.spt_workspace_bytes(spt.SPT_OP_COO_TO_CSR, A), dtype=torch.uint8, device="cuda")
    ws.fill_(0xEE)
    at = np.lexsort((col, row)) if order == spt.SPT_ORDER_ROW_COL else np.argsort(row, kind="stable")
    want = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=N))])
    for _ in range(2):
        spt.spt_coo_to_csr(A, order, pos, crd, out, ws)
        assert np.array_equal(pos.cpu().numpy(), want)
        assert np.array_equal(crd.cpu().numpy(), col[at])
        assert np.array_equal(out.cpu().numpy(), vals[at])


def _sampled(n, S):
    """The positions that the splitters are drawn from."""
    t = np.arange(S, dtype=np.uint64)
    jitter = ((t * np.uint64(2654435769)) & np.uint64(0xFFFFFFFF)) >> np.uint64(16)
    return ((((t << np.uint64(16)) | jitter) * np.uint64(n) // np.uint64(S)) >> np.uint64(16)).astype(np.int64)


@pytest.mark.parametrize("order", [spt.SPT_ORDER_ROW_COL, spt.SPT_ORDER_ROW_STABLE])
@pytest.mark.parametrize("n", [16384, 16385, 81920, 81921, 294912, 294913, 655360, 655361, 1310720, 1310721, 1572864, 1572865,
                               1835008, 1835009])
def test_lines_of_the_plan(n, order):
    rng = np.random.default_rng(n)
    N, M = n // 9, n // 7
    row = np.where(rng.random(n) < 0.8, rng.integers(0, N, n), N // 3).astype(np.int32)  # a long row
    col = rng.integers(0, M, n).astype(np.int32)
    _check(row, col, rng.random(n).astype(np.float64 if n & 1 else np.float32), N, M, order)


@pytest.mark.parametrize("order", [spt.SPT_ORDER_ROW_COL, spt.SPT_ORDER_ROW_STABLE])
@pytest.mark.parametrize("n,mean", [(7 << 18, 3), ((7 << 18) + 1, 3), (2 << 20, 4), ((2 << 20) + 1, 4), (2 << 20, 11), (5 << 19, 12), ((5 << 19) + 1, 12),
                                    (3 << 20, 15), ((3 << 20) + 1, 15)])
def test_where_the_sample_sort_takes_over(n, mean, order):
    rng = np.random.default_rng(n)
    N = n // mean
    row = np.where(rng.random(n) < 0.9, rng.integers(0, N, n), N // 3).astype(np.int32)
    _check(row, rng.integers(0, N, n).astype(np.int32), rng.random(n).astype(np.float64 if mean & 1 else np.float32), N, N, order)


@pytest.mark.parametrize("n", [20000, 400003, 2_500_003])
@pytest.mark.parametrize("kind", ["one place", "in order", "backwards", "few rows"])
def test_orders_and_duplicates(n, kind):
    rng = np.random.default_rng(n)
    N = M = 50021
    row, col = (np.full(n, 7), np.arange(n) % 3) if kind == "one place" else (rng.integers(0, 3, n), rng.integers(0, M, n)) \
        if kind == "few rows" else (np.arange(n) * N // n, np.arange(n) % M)
    step = -1 if kind == "backwards" else 1
    _check(row[::step].astype(np.int32), col[::step].astype(np.int32), rng.random(n), N, M)


def test_a_bucket_beyond_a_workgroup():
    # 256 buckets of 1152 records on average, one of 4300 more, none of them a sample
    n, N = 294912, 200000
    rng = np.random.default_rng(1)
    row = rng.integers(0, N, n).astype(np.int32)
    others = np.setdiff1d(np.arange(n), _sampled(n, 2048))
    row[rng.permutation(others)[:4300]] = 77777
    _check(row, rng.integers(0, N, n).astype(np.int32), rng.random(n), N, N)


@pytest.mark.parametrize("rows", ["the last", "any"])
def test_a_bucket_beyond_its_region(rows):
    # the samples lie in the first ten rows, all other records beyond
    n, N = 20011, 5000
    rng = np.random.default_rng(2)
    row = np.full(n, N - 1) if rows == "the last" else rng.integers(10, N, n)
    at = _sampled(n, 1024)
    row[at] = rng.integers(0, 10, len(at))
    _check(row.astype(np.int32), rng.integers(0, 900, n).astype(np.int32), rng.random(n).astype(np.float32), N, 900)


@pytest.mark.parametrize("n,N,M", [(100_000, 1 << 20, 1 << 27), (100_000, 1 << 20, (1 << 27) + 1), (30_000, 1 << 24, (1 << 31) - 2)])
def test_keys_of_64_bits_and_more(n, N, M):
    rng = np.random.default_rng(3)
    row, col = rng.integers(0, N, n).astype(np.int32), rng.integers(0, M, n).astype(np.int32)
    row[:2], col[:2] = N - 1, M - 1
    _check(row, col, rng.random(n), N, M)


@pytest.mark.parametrize("n,ws_bytes", [(65_536, 256), (65_537, 40 * 65_537), (500_000, 40 * 500_000)])
def test_less_workspace_than_the_query(n, ws_bytes):
    rng = np.random.default_rng(4)
    row, col = rng.integers(0, 10_000, n).astype(np.int32), rng.integers(0, 10_000, n).astype(np.int32)
    vals = rng.random(n)
    A, _ = _coo(row, col, vals, 10_000, 10_000)
    assert ws_bytes < spt.spt_workspace_bytes(spt.SPT_OP_COO_TO_CSR, A)
    _check(row, col, vals, 10_000, 10_000, ws_bytes=ws_bytes)
