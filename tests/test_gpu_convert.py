"""GPU parity: spt_coo_to_csr vs the oracle -- every output bit-exact."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import gpu_coo_to_csr

pytestmark = pytest.mark.gpu

TILE = 4096  # records of a tile of a large partition, and the most that are sorted in LDS


def _check(N, M, r, c, v, order, ordered=False, what=""):
    spec = wl.coo_spec(N, M, r, c, v, ordered=ordered)
    pos, crd, vout = gpu_coo_to_csr(spec, order)
    rpos, rcrd, rv, _ = oracle.coo_to_csr(N, r, c, v, order)
    assert np.array_equal(pos, rpos), f"{what}: pos differs"
    assert np.array_equal(crd, rcrd), f"{what}: crd differs"
    assert np.array_equal(vout.view(np.uint8), rv.view(np.uint8)), f"{what}: vals differ"
    assert pos[0] == 0 and pos[-1] == len(v) and np.all(np.diff(pos) >= 0)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [0, 1, 255, 256, 4095, 4096, 4097, 3 * 4096 + 5, 100_003])
def test_random_unsorted(order, dtype, nnz):
    N, M = 1500, 70_000
    r, c, v = wl.random_coo_entries(N, M, nnz, seed=200 + nnz, dtype=dtype, sort=False)
    _check(N, M, r, c, v, order, what=f"nnz={nnz}")


@pytest.mark.parametrize("order", [0, 1])
def test_duplicates_keep_input_order(order):
    N, M = 37, 19
    r, c, v = wl.random_coo_entries(N, M, 20_000, seed=5, duplicates=True, sort=False)
    v = np.arange(len(v), dtype=np.float64)   # values identify the input position
    _check(N, M, r, c, v, order, what="duplicates")


@pytest.mark.parametrize("order", [0, 1])
def test_degenerate_shapes(order):
    rng = np.random.default_rng(1)
    n = 2 * TILE + 9
    v = rng.uniform(-1, 1, n)
    _check(1, 1, np.zeros(n, int), np.zeros(n, int), v, order, what="1x1")
    _check(1, 300, np.zeros(n, int), rng.integers(0, 300, n), v, order, what="one row")
    _check(300, 1, rng.integers(0, 300, n), np.zeros(n, int), v, order, what="one col")
    _check(100_000, 3, np.array([99_999, 0, 50_000, 0]), np.array([2, 1, 0, 0]),
           np.array([1., 2., 3., 4.]), order, what="rows >> entries")
    # runs of empty rows of every length next to a dense cluster (long runs are written by a whole wave)
    rr = np.concatenate([rng.integers(0, 1_000_000, 5000), rng.integers(400_000, 400_300, 6000)])
    _check(1_000_000, 50, rr, rng.integers(0, 50, rr.size), rng.uniform(-1, 1, rr.size), order,
           what="sparse rows with a dense cluster")
    big = 2**31 - 10                           # maximum dimension sizes: all 31 key bits used
    r = np.array([big - 1, 0, big - 1, 12345, 2**30])
    c = np.array([big - 2, 5, 0, 2**30 + 1, 7])
    spec = wl.coo_spec(5, big, [0, 1, 2, 3, 4], c, np.arange(5.0), ordered=False)
    pos, crd, vout = gpu_coo_to_csr(spec, order)
    assert list(pos) == [0, 1, 2, 3, 4, 5] and np.array_equal(crd, c)


@pytest.mark.parametrize("order", [0, 1])
def test_buffers_that_are_not_16_byte_aligned(order):
    N, M = 700, 900
    r, c, v = wl.random_coo_entries(N, M, 20_000, seed=12, sort=False)
    spec = wl.coo_spec(N, M, r, c, v, ordered=False)
    pos, crd, vout = gpu_coo_to_csr(spec, order, misalign=True)
    rpos, rcrd, rv, _ = oracle.coo_to_csr(N, r, c, v, order)
    assert np.array_equal(pos, rpos) and np.array_equal(crd, rcrd) and np.array_equal(vout, rv)


def test_sorted_flagged_input_skips_the_sort():
    N, M = 800, 900
    r, c, v = wl.random_coo_entries(N, M, 30_000, seed=6)
    _check(N, M, r, c, v, 0, ordered=True, what="flagged sorted")
    _check(N, M, r, c, v, 1, ordered=True, what="flagged sorted, stable")


def test_csr_to_coo_to_csr_is_a_fixed_point():
    N, M = 500, 600
    r, c, v = wl.random_coo_entries(N, M, 9000, seed=7, sort=False)
    pos, crd, vout = gpu_coo_to_csr(wl.coo_spec(N, M, r, c, v, ordered=False), 0)
    rows = np.repeat(np.arange(N), np.diff(pos))
    pos2, crd2, v2 = gpu_coo_to_csr(wl.coo_spec(N, M, rows, crd, vout, ordered=False), 0)
    assert np.array_equal(pos, pos2) and np.array_equal(crd, crd2) and np.array_equal(vout, v2)
    # the multiset of (row, col, value) is preserved
    a = np.lexsort((v, c, r))
    b = np.lexsort((vout, crd, rows))
    assert np.array_equal(r[a], rows[b]) and np.array_equal(c[a], crd[b]) and np.array_equal(v[a], vout[b])


@pytest.mark.parametrize("order", [0, 1])
def test_power_law_scaled_config4(order):
    c4 = wl.config4(N=50_000, nnz_target=700_000, max_row=30_000)
    coo = c4["coo"]
    _check(50_000, 50_000, coo.levels[0].crd, coo.levels[1].crd, coo.vals, order, what="c4 scaled")


# ---- sizes, input orders and duplicate patterns that stress any sort implementation ----

@pytest.mark.parametrize("nnz", [6143, 6144, 6145, 20_000, 524_288, 524_289, 1_300_000])
def test_sizes_from_thousands_to_a_million(nnz):
    N, M = 90_000, 70_000
    r, c, v = wl.random_coo_entries(N, M, nnz, seed=300 + nnz % 97, dtype=np.float64, sort=False)
    _check(N, M, r, c, v, 0, what=f"nnz={nnz}")


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("kind", ["sorted", "reversed", "by_column", "interleaved"])
def test_unordered_flagged_input_in_special_orders(kind, order):
    """Input flagged unordered that is in fact sorted, reversed, column-major, or a regular
    interleaving of 170 sorted runs."""
    N, M, nnz = 3000, 5000, 700_000
    r, c, v = wl.random_coo_entries(N, M, nnz, seed=41, dtype=np.float32, sort=True)
    if kind == "reversed":
        r, c, v = r[::-1].copy(), c[::-1].copy(), v[::-1].copy()
    elif kind == "by_column":
        o = np.lexsort((r, c))
        r, c, v = r[o], c[o], v[o]
    elif kind == "interleaved":
        stride = len(v) // 4096
        o = np.concatenate([np.arange(len(v))[i::stride] for i in range(stride)])
        r, c, v = r[o], c[o], v[o]
    _check(N, M, r, c, v, order, what=kind)


@pytest.mark.parametrize("order", [0, 1])
def test_many_copies_of_one_coordinate_keep_their_input_order(order):
    """20 000 entries share one (row, col) pair and 9 000 another, scattered through the input."""
    N, M = 4000, 4000
    r, c, v = wl.random_coo_entries(N, M, 300_000, seed=43, dtype=np.float64, sort=False)
    rng = np.random.default_rng(44)
    r = np.concatenate([r, np.full(20_000, 1234), np.full(9_000, 77)])
    c = np.concatenate([c, np.full(20_000, 999), np.full(9_000, 3)])
    p = rng.permutation(len(r))
    r, c = r[p], c[p]
    v = np.arange(len(r), dtype=np.float64)            # values identify the input position
    _check(N, M, r, c, v, order, what="heavy duplicates")
    keep = slice(0, 200_000)
    _check(N, M, r[keep], c[keep], v[keep].astype(np.float32), order, what="heavy duplicates, fp32")


@pytest.mark.parametrize("order", [0, 1])
def test_one_row_holds_most_entries_and_columns_use_31_bits(order):
    rng = np.random.default_rng(45)
    M = 2**31 - 10
    n = 900_000
    r = rng.integers(0, 5000, n)
    r[: 2 * n // 3] = 4321                               # one row with 600 000 entries
    c = rng.integers(0, M, n)
    p = rng.permutation(n)
    _check(5000, M, r[p], c[p], rng.uniform(-1, 1, n), order, what="heavy row, 31-bit columns")


# ---- the sample sort's own boundaries ----

@pytest.mark.parametrize("nnz", [384, 385, 1025, 65_536, 65_537, 131_072, 131_073, 360_448, 360_449, 4_194_304, 4_194_305])
def test_sizes_at_which_the_sample_sort_changes_its_plan(nnz):
    """One workgroup / several; one launch / one partition / two partitions."""
    N, M = 50_000, 60_000
    r, c, v = wl.random_coo_entries(N, M, nnz, seed=500 + nnz % 89, dtype=np.float32, sort=False)
    _check(N, M, r, c, v, nnz % 2, what=f"nnz={nnz}")


def _sampled(m, S):
    t = np.arange(S, dtype=np.uint64)
    jitter = ((t * np.uint64(2654435769)) & np.uint64(0xFFFFFFFF)) >> np.uint64(16)
    return ((((t << np.uint64(16)) | jitter) * np.uint64(m) // np.uint64(S)) >> np.uint64(16)).astype(np.int64)


@pytest.mark.parametrize("nnz, S", [(6000, 1024), (4_200_000, 4096)])
def test_input_that_defeats_the_sampling(nnz, S):
    """Small keys exactly at the sampled positions: all other records end in one bucket. Of 6000, it is
    ranked by counting; of 4.2M, the second partition leaves buckets of 16 000, which are split once more."""
    N, M = 100_000, 4000
    rng = np.random.default_rng(46)
    r, c = rng.integers(1000, N, nnz), rng.integers(0, M, nnz)
    at = _sampled(nnz, S)
    r[at], c[at] = np.arange(S) % 7, np.arange(S) % M
    _check(N, M, r, c, np.arange(nnz, dtype=np.float64), 0, what="sampling defeated")


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("many", [4097, 6000, 20_000])
@pytest.mark.parametrize("same", [False, True])
def test_a_bucket_that_the_sample_got_wrong(order, many, same):
    """Among 200 000 records `many` neighbours in the order (or copies of one coordinate) at positions that
    are not sampled: one bucket of at least that many."""
    N, M, nnz = 50_000, 60_000, 200_000
    rng = np.random.default_rng(many)
    r, c = rng.integers(0, N, nnz), rng.integers(0, M, nnz)
    free = np.setdiff1d(np.arange(nnz), _sampled(nnz, 2048))        # 14 samples for each of 143 buckets
    at = rng.choice(free, many, replace=False)
    r[at], c[at] = (30_000, 7) if same else (rng.integers(30_000, 30_003, many), rng.integers(0, M, many))
    _check(N, M, r, c, np.arange(nnz, dtype=np.float64), order, what=f"bucket of {many}")


def test_a_bucket_that_the_sample_got_wrong_costs_little():
    """4.2M records of which all but the sampled ones share a bucket of the first partition, so that all buckets
    of the second hold four times what fits: counting their ranks took 1.1 s, split once more they take 2 ms (0.2 otherwise)."""
    import torch
    import paper_1804_10112_amd as spt
    N, M, nnz = 100_000, 4000, 4_200_000
    rng = np.random.default_rng(46)
    times = []
    for defeat in (False, True):
        r, c = rng.integers(1000, N, nnz), rng.integers(0, M, nnz)
        if defeat:
            at = _sampled(nnz, 4096)
            r[at], c[at] = np.arange(4096) % 7, np.arange(4096) % M
        A = spt.DeviceTensor(wl.coo_spec(N, M, r, c, np.zeros(nnz, np.float32), ordered=False))
        pos = torch.empty(N + 1, dtype=torch.int32, device="cuda")
        crd, vals = torch.empty(nnz, dtype=torch.int32, device="cuda"), torch.empty(nnz, device="cuda")
        ws = A.workspace(spt.SPT_OP_COO_TO_CSR)
        best = 1e9
        for _ in range(4):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            spt.spt_coo_to_csr(A, 0, pos, crd, vals, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        times.append(best)
    assert times[1] < 40 * times[0], f"{times[1]:.2f} ms with all buckets too large, {times[0]:.2f} otherwise"


def _clustered(nnz, width, M, rng):
    """Rows of `width` neighbouring columns anywhere in M, in random order."""
    N = -(-nnz // width)
    r = np.repeat(np.arange(N), width)[:nnz]
    c = (rng.integers(0, M - width, N)[:, None] + np.arange(width)).reshape(-1)[:nnz]
    p = rng.permutation(nnz)
    return N, r[p], c[p]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("nnz", [300, 5000, 60_000, 200_000, 700_000])
@pytest.mark.parametrize("width", [7, 8, 9, 15, 16, 17, 100, 1000])
def test_clustered_columns(nnz, width, order):
    """Stretches of records that 20 bits of a bucket's key range do not tell apart, around the length from
    which all are sorted again by 20 bits at a time."""
    M = 2**31 - 10
    rng = np.random.default_rng(nnz + width)
    N, r, c = _clustered(nnz, width, M, rng)
    _check(N, M, r, c, np.arange(nnz, dtype=np.float64), order, what=f"rows of {width} neighbours")


def test_clustered_columns_take_no_longer():
    """Rows of 1000 neighbours in 2^31 columns: with every record compared with its whole stretch, the
    conversion took twelve times as long as with columns anywhere."""
    import torch
    import paper_1804_10112_amd as spt
    nnz, M = 3_000_000, 2**31 - 10
    rng = np.random.default_rng(5)
    times = []
    for clustered in (False, True):
        N, r, c = _clustered(nnz, 1000, M, rng) if clustered else (200_000, rng.integers(0, 200_000, nnz), rng.integers(0, M, nnz))
        A = spt.DeviceTensor(wl.coo_spec(N, M, r, c, np.zeros(nnz, np.float32), ordered=False))
        pos = torch.empty(N + 1, dtype=torch.int32, device="cuda")
        crd, vals = torch.empty(nnz, dtype=torch.int32, device="cuda"), torch.empty(nnz, device="cuda")
        ws = A.workspace(spt.SPT_OP_COO_TO_CSR)
        best = 1e9
        for _ in range(4):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            spt.spt_coo_to_csr(A, 0, pos, crd, vals, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        times.append(best)
    assert times[1] < 3 * times[0], f"{times[1]:.2f} ms clustered, {times[0]:.2f} with columns anywhere"


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N,M,order,at", [
    (200, 4_000_000, 1, 1 << 16),                                       # one pass
    (60_000, 900, 1, 256 * 1408), (256, 129, 0, 256 * 1408),            # two
    (3_000_000, 70_000, 1, 3 << 19), (60_000, 250, 0, 3 << 19),         # three
])
def test_short_keys_where_radix_passes_take_over(N, M, order, at, dtype):
    """Both sides of the record counts from which one to three radix passes replace the sample sort, and 8M;
    every third record in one row. The reference is torch's stable sort."""
    import torch
    import paper_1804_10112_amd as spt
    g = torch.Generator(device="cuda").manual_seed(N + order)
    np_dt, t_dt = (np.float64, torch.int64) if dtype == "f64" else (np.float32, torch.int32)
    i32 = dict(dtype=torch.int32, device="cuda")
    for nnz in (at, at + 1, 8_000_003):
        r = torch.randint(0, N, (nnz,), generator=g, **i32)
        r[::3] = N // 2
        c = torch.randint(0, M, (nnz,), generator=g, **i32)
        v = torch.arange(nnz, dtype=t_dt, device="cuda")                # bits that tell the position
        A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], np.zeros(1, np_dt), ordered=False))
        A.c.level[0].crd, A.c.level[1].crd, A.c.vals, A.c.nvals = r.data_ptr(), c.data_ptr(), v.data_ptr(), nnz
        pos, crd, vals = torch.empty(N + 1, **i32), torch.empty_like(c), torch.empty_like(v)
        spt.spt_coo_to_csr(A, order, pos, crd, vals, A.workspace(spt.SPT_OP_COO_TO_CSR))
        perm = torch.sort(r.long() * M + c if order == 0 else r, stable=True).indices
        assert torch.equal(crd, c[perm]) and torch.equal(vals, perm.to(t_dt))
        assert torch.equal(pos[1:].long(), torch.bincount(r, minlength=N).cumsum(0)) and int(pos[0]) == 0


def test_more_records_than_the_sample_sort_takes():
    import torch
    import paper_1804_10112_amd as spt
    N, M, nnz = 3_000_000, 5_000_000, (1 << 26) + 3
    g = torch.Generator(device="cuda:0").manual_seed(1)
    r = torch.randint(0, N, (nnz,), generator=g, device="cuda:0", dtype=torch.int32)
    c = torch.randint(0, M, (nnz,), generator=g, device="cuda:0", dtype=torch.int32)
    v = torch.arange(nnz, dtype=torch.int32, device="cuda:0").view(torch.float32)
    A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], np.zeros(1, np.float32), ordered=False))
    A.c.level[0].crd, A.c.level[1].crd, A.c.vals, A.c.nvals = r.data_ptr(), c.data_ptr(), v.data_ptr(), nnz
    pos = torch.empty(N + 1, dtype=torch.int32, device="cuda:0")
    crd, vals = torch.empty_like(c), torch.empty_like(v)
    spt.spt_coo_to_csr(A, spt.SPT_ORDER_ROW_COL, pos, crd, vals, A.workspace(spt.SPT_OP_COO_TO_CSR))
    order = torch.sort(r.long() * M + c, stable=True).indices
    assert torch.equal(crd, c[order]) and torch.equal(vals.view(torch.int32), order.int())
    assert torch.equal(pos[1:].long(), torch.bincount(r, minlength=N).cumsum(0)) and int(pos[0]) == 0
