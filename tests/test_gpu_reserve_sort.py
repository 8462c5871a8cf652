"""COO -> CSR by reserved regions: the lines of its plan, buckets that a workgroup or a region does not hold, keys that do
not fit, and workspaces below the query, against a stable sort on the host."""
import numpy as np
import pytest
import torch

import paper_1804_10112_amd as spt
from paper_1804_10112_amd.binding import SptTensor

pytestmark = pytest.mark.gpu


def _coo(row, col, vals, N, M, shift=0):
    # shift: rows and columns begin that many elements beyond a boundary of 16 bytes
    dev = [torch.from_numpy(np.concatenate([np.zeros(s, a.dtype), a])).cuda()[s:]
           for a, s in ((np.array([0, len(row)], np.int32), 0), (row, shift), (col, shift and 4 - shift), (vals, 0))]
    t = SptTensor()
    t.order, t.nlevels, t.dtype = 2, 2, spt.SPT_F64 if vals.dtype == np.float64 else spt.SPT_F32
    t.vals, t.nvals = dev[3].data_ptr(), len(row)
    for k, (kind, n) in enumerate(((1, N), (2, M))):
        lv = t.level[k]
        lv.kind, lv.mode, lv.N, lv.M, lv.flags, lv.crd_stride = kind, k, n, 1 - k, 0, 1
        lv.crd = dev[1 + k].data_ptr()
    t.level[0].pos = dev[0].data_ptr()
    return t, dev


def _check(row, col, vals, N, M, order=spt.SPT_ORDER_ROW_COL, ws_bytes=None, shift=0):
    A, keep = _coo(row, col, vals, N, M, shift)
    n = len(row)
    pos, crd = (torch.empty(k, dtype=torch.int32, device="cuda") for k in (N + 1, n))
    out = torch.empty(n, dtype=keep[3].dtype, device="cuda")
    ws = torch.empty(ws_bytes or spt.spt_workspace_bytes(spt.SPT_OP_COO_TO_CSR, A), dtype=torch.uint8, device="cuda")
    ws.fill_(0xEE)
    at = np.lexsort((col, row)) if order == spt.SPT_ORDER_ROW_COL else np.argsort(row, kind="stable")
    want = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=N))])
    for _ in range(2):
        pos.fill_(-1), crd.fill_(-1), out.fill_(-1)
        spt.spt_coo_to_csr(A, order, pos, crd, out, ws)
        assert np.array_equal(pos.cpu().numpy(), want)
        assert np.array_equal(crd.cpu().numpy(), col[at])
        assert np.array_equal(out.cpu().numpy(), vals[at])


def _sampled(n, S, mix=2654435769):
    """The positions that the splitters are drawn from (and, of another mix, the parts of a bucket beyond its region)."""
    t = np.arange(S, dtype=np.uint64)
    jitter = ((t * np.uint64(mix)) & np.uint64(0xFFFFFFFF)) >> np.uint64(16)
    return ((((t << np.uint64(16)) | jitter) * np.uint64(n) // np.uint64(S)) >> np.uint64(16)).astype(np.int64)


def _plan(n):
    """Buckets, samples, threads of a workgroup that sorts a bucket, records of a region."""
    nb, S, threads = next(p[1:] for p in ((5 << 14, 128, 1024, 512), (9 << 15, 256, 2048, 512), (5 << 17, 512, 4096, 512), (5 << 18, 512, 4096, 1024),
                                          (3 << 19, 1024, 16384, 512), (3 << 20, 1024, 16384, 1024)) if n <= p[0])
    mean = -(-n // nb)
    return nb, S, threads, 5 * mean if S == 8 * nb else (16 * mean + 4) // 5


def _buckets(row, col, order=spt.SPT_ORDER_ROW_COL):
    """Records of each bucket."""
    n = len(row)
    nb, S, _, _ = _plan(n)
    at = np.lexsort((col, row)) if order == spt.SPT_ORDER_ROW_COL else np.argsort(row, kind="stable")
    rank = np.empty(n, np.int64)
    rank[at] = np.arange(n)
    cuts = np.sort(rank[_sampled(n, S)])[:: S // nb]
    return np.diff(np.concatenate([[0], cuts[1:], [n]]))


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


@pytest.mark.parametrize("n", [294_912, 1_048_577, 1_500_000, 3_000_000])
@pytest.mark.parametrize("order", [spt.SPT_ORDER_ROW_COL, spt.SPT_ORDER_ROW_STABLE])
def test_a_bucket_beyond_a_workgroup(n, order):
    # a bucket with many records that are no samples: more than nine words of a thread, and no more than its region
    N = 200_000
    nb, S, threads, room = _plan(n)
    rng = np.random.default_rng(1)
    row, col = rng.integers(0, N, n).astype(np.int32), rng.integers(0, N, n).astype(np.int32)
    free = rng.permutation(np.setdiff1d(np.arange(n), _sampled(n, S)))
    many = 9 * threads - n // nb
    row[free[:many]] = 77_777
    row[free[many : many + (9 * threads + room) // 2 - _buckets(row, col, order).max()]] = 77_777
    assert 9 * threads < _buckets(row, col, order).max() <= room
    _check(row, col, rng.random(n), N, N, order)


@pytest.mark.parametrize("order", [spt.SPT_ORDER_ROW_COL, spt.SPT_ORDER_ROW_STABLE])
@pytest.mark.parametrize("n,N,M", [(20_011, 5000, 900), (200_003, 5000, 900), (1_000_003, 70_000, 900), (1_000_003, 1_000_003, 1 << 22), (1_500_000, 90_000, 50_000),
                                   (2_500_000, 200_000, 50_000)])
@pytest.mark.parametrize("rows", ["the last", "any", "two", "a line"])
def test_buckets_beyond_their_regions(n, N, M, rows, order):
    # the samples lie in the first ten rows, all other records, or those of two rows, or a few more than a region holds, beyond
    nb, S, threads, room = _plan(n)
    rng = np.random.default_rng(2)
    row, col = rng.integers(10, N, n), rng.integers(0, M, n)
    at = _sampled(n, S)
    if rows == "two":  # two buckets, others in order between and around them
        some = rng.permutation(np.setdiff1d(np.arange(n), at))[: 4 * room]
        row[some] = np.where(np.arange(len(some)) % 2, N // 3, N // 2)
    elif rows == "a line":
        row[rng.permutation(np.setdiff1d(np.arange(n), at))[: room + 1 - n // nb]] = N // 3
        free = np.setdiff1d(np.flatnonzero(row != N // 3), at)
        row[free[: 3 * (n // nb)]] = N // 3
    else:
        if rows == "the last":
            row[:] = N - 1
        row[at] = rng.integers(0, 10, len(at))
    row, col = row.astype(np.int32), col.astype(np.int32)
    assert np.sort(_buckets(row, col, order))[-2 if rows == "two" else -1] > room
    _check(row, col, rng.random(n).astype(np.float32 if n & 1 else np.float64), N, M, order, shift=n % 4)


@pytest.mark.parametrize("n,clustered", [(20_011, False), (20_011, True), (100_003, False), (100_003, True), (300_000, True)])
def test_records_that_both_draws_miss(n, clustered):
    # one bucket, not cut into parts: its records lie anywhere, or in a few stretches of neighbours far apart
    nb, S, threads, room = _plan(n)
    N, M = 1 << 20, 1 << 22
    rng = np.random.default_rng(3)
    row, col = rng.integers(10, N, n), rng.integers(0, M, n)
    if clustered:
        row, col = np.array([11, 12, N // 7, N // 2, N - 1])[rng.integers(0, 5, n)], M // 3 + rng.integers(0, 2000, n) // 1000
    at = np.union1d(_sampled(n, S), _sampled(n, 8 * threads, 3266489917))
    row[at] = rng.integers(0, 10, len(at))
    row, col = row.astype(np.int32), col.astype(np.int32)
    assert _buckets(row, col).max() > room
    _check(row, col, rng.random(n), N, M)


@pytest.mark.parametrize("n", [20_011, 100_003, 300_007, 1_000_003, 1_500_000, 3_000_000])
def test_what_the_sample_misses_costs_little(n):
    """All records but the samples in one bucket: by one workgroup, which read all of the input for each 2048 or 4096 of them, 1M took 2500 times
    as long as in even order."""
    nb, S, threads, room = _plan(n)
    N, M = n // 15, 100_000
    rng = np.random.default_rng(46)
    times = []
    for missed in (False, True):
        row, col = rng.integers(10, N, n).astype(np.int32), rng.integers(0, M, n).astype(np.int32)
        if missed:
            row[_sampled(n, S)] = np.arange(S) % 10
            assert _buckets(row, col).max() > n - 2 * S
        A, keep = _coo(row, col, np.zeros(n), N, M)
        pos, crd = (torch.empty(k, dtype=torch.int32, device="cuda") for k in (N + 1, n))
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        ws = torch.empty(spt.spt_workspace_bytes(spt.SPT_OP_COO_TO_CSR, A), dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(4):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            spt.spt_coo_to_csr(A, spt.SPT_ORDER_ROW_COL, pos, crd, out, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        times.append(best)
    print(f"{n}: {times[0] * 1e3:.1f} us, {times[1] * 1e3:.0f} us where the sample misses them")
    assert times[1] < 40 * times[0], f"{times[1]:.2f} ms where the sample misses them, {times[0]:.3f} otherwise"


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
