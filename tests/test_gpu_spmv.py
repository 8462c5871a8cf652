"""GPU parity: spt_spmv through the C ABI vs the CPU oracle, element by element."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_util import assert_close, assert_close_where_finite, gpu_spmv, gpu_spmv_sparse_x

pytestmark = pytest.mark.gpu

CHUNK = 2048  # entries per workgroup of the entry-balanced kernel: sizes below straddle it


def _check(spec, x, what):
    ref, mag = oracle.spmv(spec, x)
    got = gpu_spmv(spec, x)
    assert_close(got, ref, mag, spec.vals.dtype, what)
    return got


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [0, 1, 63, 64, 65, 2047, 2048, 2049, 4096, 5000, 70001])
def test_csr_coo_random_sizes(dtype, nnz):
    N, M = 997, 1201
    r, c, v = wl.random_coo_entries(N, M, nnz, seed=100 + nnz, dtype=dtype)
    x = wl.dense_vector(M, 7, dtype)
    _check(wl.csr_from_sorted_coo(N, M, r, c, v), x, f"csr nnz={nnz}")
    _check(wl.coo_spec(N, M, r, c, v), x, f"coo nnz={nnz}")
    p = np.random.default_rng(1).permutation(len(v))
    _check(wl.coo_spec(N, M, r[p], c[p], v[p], ordered=False), x, f"coo-unsorted nnz={nnz}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_csr_coo_degenerate_structures(dtype):
    x = wl.dense_vector(50, 3, dtype)
    # one row holds everything (spans several chunks), all other rows empty
    n = 3 * CHUNK + 17
    rng = np.random.default_rng(5)
    c = rng.integers(0, 50, n)
    v = rng.uniform(-1, 1, n).astype(dtype)
    for row in (0, 5, 9):
        r = np.full(n, row)
        _check(wl.csr_from_sorted_coo(10, 50, r, c, v), x, f"csr single row {row}")
        _check(wl.coo_spec(10, 50, r, c, v), x, f"coo single row {row}")
    # many empty rows between few entries, rows >> entries
    r = np.array([3, 3, 40000, 99999])
    c4 = np.array([1, 2, 3, 4])
    v4 = np.array([1, 2, 3, 4], dtype)
    _check(wl.csr_from_sorted_coo(100000, 50, r, c4, v4), x, "csr mostly empty")
    _check(wl.coo_spec(100000, 50, r, c4, v4), x, "coo mostly empty")
    # more than 2^20 rows: few entries still go in pieces (fill + carries)
    _check(wl.coo_spec(3_000_000, 50, np.array([3, 3, 40000, 2_999_999]), c4, v4), x, "coo, 3M rows, 4 entries")
    # row boundaries exactly on chunk boundaries
    r = np.repeat(np.arange(4), CHUNK)
    c = rng.integers(0, 50, 4 * CHUNK)
    v = rng.uniform(-1, 1, 4 * CHUNK).astype(dtype)
    _check(wl.csr_from_sorted_coo(4, 50, r, c, v), x, "csr aligned rows")
    _check(wl.coo_spec(4, 50, r, c, v), x, "coo aligned rows")
    # duplicates are summed by SpMV
    r, c, v = wl.random_coo_entries(20, 50, 6000, seed=8, dtype=dtype, duplicates=True)
    _check(wl.csr_from_sorted_coo(20, 50, r, c, v), x, "csr duplicates")
    _check(wl.coo_spec(20, 50, r, c, v), x, "coo duplicates")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [255, 257, 1023, 65_535, 65_536, 65_537, 200_000])
def test_sorted_coo_on_both_sides_of_the_single_launch_limit(dtype, nnz):
    """Up to 65 536 entries sorted COO runs in one launch (a wave per 256 entries, the owner of
    a row reads on past its piece); above, in pieces with carries. Rows of 1 to 3000
    entries, runs of empty rows, the last rows empty, an infinite x value under the last entry."""
    N, M = 9000, 700
    rng = np.random.default_rng(nnz)
    lens = np.minimum(rng.zipf(1.4, 4000), min(3000, nnz // 3))
    lens = lens[np.cumsum(lens) <= nnz]
    rows = np.sort(rng.choice(N - 50, len(lens), replace=False))      # the last 50 rows stay empty
    r = np.repeat(rows, lens)
    r = np.concatenate([r, np.full(nnz - len(r), rows[-1] + 1)])      # fill up with one more long row
    c = rng.integers(0, M, nnz)
    c = c[np.lexsort((c, r))]                                         # columns ascend inside every row
    v = rng.uniform(-1, 1, nnz).astype(dtype)
    x = wl.dense_vector(M, 11, dtype)
    _check(wl.coo_spec(N, M, r, c, v), x, f"sorted coo nnz={nnz}")
    x2 = x.copy()
    x2[c[-1]] = np.inf
    v[c == c[-1]] = 1.0
    spec = wl.coo_spec(N, M, r, c, v)
    ref, _ = oracle.spmv(spec, x2)
    got = gpu_spmv(spec, x2)
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and not np.isnan(got).any()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_buffers_that_are_not_16_byte_aligned(dtype):
    """Arrays one element past an aligned address take the scalar-load paths."""
    N, M = 1000, 1200
    r, c, v = wl.random_coo_entries(N, M, 9000, seed=77, dtype=dtype)
    x = wl.dense_vector(M, 7, dtype)
    c2 = wl.config2(N=1000, dtype=dtype)
    c3 = wl.config3(N=1000, dtype=dtype)
    for spec, xx in ((wl.csr_from_sorted_coo(N, M, r, c, v), x), (wl.coo_spec(N, M, r, c, v), x),
                     (c2["dia"], c2["x"]), (c3["ell"], c3["x"])):
        ref, mag = oracle.spmv(spec, xx)
        assert_close(gpu_spmv(spec, xx, misalign=True), ref, mag, dtype, spec.name + " misaligned")


def test_config1_full_and_deterministic():
    c1 = wl.config1()
    for fmt in ("csr", "coo"):
        ref, mag = oracle.spmv(c1[fmt], c1["x"])
        a, b = gpu_spmv(c1[fmt], c1["x"], repeat=2)
        assert_close(a, ref, mag, np.float64, f"c1 {fmt}")
        assert np.array_equal(a, b), "run-to-run bits differ"


def test_power_law_rows_scaled_config4():
    c4 = wl.config4(N=40_000, nnz_target=600_000, max_row=20_000)
    coo = c4["coo"]
    r, c = coo.levels[0].crd, coo.levels[1].crd
    _check(coo, c4["x"], "c4 unsorted coo")
    o = np.lexsort((c, r))
    rs, cs, vs = r[o], c[o], coo.vals[o]
    a = _check(wl.coo_spec(40_000, 40_000, rs, cs, vs), c4["x"], "c4 sorted coo")
    csr = wl.csr_from_sorted_coo(40_000, 40_000, rs, cs, vs)
    b = _check(csr, c4["x"], "c4 csr, kernel chosen by the mean row length")
    lv = csr.levels[1]
    _check(wl.csr_spec(40_000, 40_000, lv.pos, lv.crd, csr.vals, max_row=20_000), c4["x"],
           "c4 csr, declared long rows: entry-balanced kernel")
    assert np.bincount(r).max() > 2 * CHUNK      # a row really spans several chunks


@pytest.mark.parametrize("dtype,N", [(np.float64, 6_000_000), (np.float32, 20_000_000)])
def test_unordered_coo_with_more_rows_than_one_lds_window(dtype, N):
    """Row count so large that a bin's rows need several LDS sub-ranges, and a row so long
    that its bin is cut into several slices, which a last kernel adds up."""
    rng = np.random.default_rng(4)
    n = 900_000                                 # binned from 786 432 entries on
    row = rng.integers(0, N, n)
    row[: n // 2] = N - 7                       # one heavy row: half of all entries in one bin
    col = rng.integers(0, 1000, n)
    v = rng.uniform(-1, 1, n).astype(dtype)
    p = rng.permutation(n)
    spec = wl.coo_spec(N, 1000, row[p], col[p], v[p], ordered=False)
    x = wl.dense_vector(1000, 5, dtype)
    _check(spec, x, f"unordered coo N={N}")


def test_exact_integer_data_is_bit_exact():
    N, M = 3000, 2000
    r, c, v = wl.random_coo_entries(N, M, 50_000, seed=9, dtype=np.float32, dist="int")
    x = wl.dense_vector(M, 10, np.float32, "int")
    ref, _ = oracle.spmv(wl.coo_spec(N, M, r, c, v), x)
    for spec in (wl.csr_from_sorted_coo(N, M, r, c, v), wl.coo_spec(N, M, r, c, v),
                 wl.coo_spec(N, M, r[::-1].copy(), c[::-1].copy(), v[::-1].copy(), ordered=False)):
        assert np.array_equal(gpu_spmv(spec, x).astype(np.float64), ref)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("N", [1, 255, 256, 257, 100_003])
def test_dia_scaled_config2_with_poison(dtype, N):
    c2 = wl.config2(N=max(N, 8), poison=True, dtype=dtype)
    got = _check(c2["dia"], c2["x"], f"dia N={N}")
    assert np.isfinite(got).all()
    _check(c2["csr"], c2["x"], f"c2 csr N={N}")


def test_dia_rectangular_and_outside_diagonals():
    rng = np.random.default_rng(3)
    for (N, M) in ((700, 1000), (1000, 700)):
        off = np.array([-1200, -699, -3, 0, 1, 250, 999, 5000])
        diag = rng.uniform(-1, 1, (len(off), N))
        i = np.arange(N)
        for d, o in enumerate(off):
            diag[d, ~((i + o >= 0) & (i + o < M))] = np.nan
        _check(wl.dia_spec(N, M, off, diag), wl.dense_vector(M, 4), f"dia {N}x{M}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("N", [1, 300, 100_001])
def test_ell_scaled_config3_with_poisoned_padding(dtype, N):
    c3 = wl.config3(N=max(N, 40), dtype=dtype)
    ell = c3["ell"]
    v = ell.vals.copy()
    v[ell.levels[2].crd < 0] = np.nan
    got = _check(wl.TensorSpec(ell.dims, ell.levels, v), c3["x"], f"ell N={N}")
    assert np.isfinite(got).all()
    _check(c3["csr"], c3["x"], f"c3 csr N={N}")
    # a matrix whose rows are all empty: every slot is padding
    z = wl.config3(N=50, lo=0, hi=0, dtype=dtype)
    assert z["W"] == 0 or np.all(z["ell"].levels[2].crd < 0)
    _check(z["ell"], z["x"], "ell all padding")


def _with_hint(spec, bound):
    lv = spec.levels[1]
    return wl.csr_spec(spec.dims[0], spec.dims[1], lv.pos, lv.crd, spec.vals, max_row=bound)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("lo,hi", [(0, 3), (1, 7), (0, 12), (9, 16), (8, 32)])
def test_csr_kernel_choice_by_mean_row_length_and_by_hint(dtype, lo, hi):
    """Plain (pos, crd) CSR with a short mean row runs the row kernel (a group of lanes per row)
    with no hint at all; a declared bound <= 32 selects the same
    kernel (same bits), a larger one the entry-balanced kernel; all match the oracle."""
    c3 = wl.config3(N=5003, lo=lo, hi=hi, dtype=dtype)
    hinted = c3["csr"]
    assert hinted.levels[1].max_children == c3["W"] <= 32
    plain = _with_hint(hinted, 0)
    ref, mag = oracle.spmv(hinted, c3["x"])
    a, b = gpu_spmv(plain, c3["x"], repeat=2)
    assert_close(a, ref, mag, dtype, f"no hint, rows {lo}..{hi}")
    assert np.array_equal(a, b), "run-to-run bits differ"
    assert np.array_equal(gpu_spmv(hinted, c3["x"]), a), "the hint selects the same kernel"
    assert_close(gpu_spmv(_with_hint(hinted, 100_000), c3["x"]), ref, mag, dtype,
                 f"entry-balanced kernel rows {lo}..{hi}")
    assert_close(gpu_spmv(plain, c3["x"], misalign=True), ref, mag, dtype, "row kernel, unaligned")


@pytest.mark.parametrize("which", ["c2", "c3"])
def test_unhinted_csr_of_configs_2_and_3_is_bit_reproducible(which):
    cfg = wl.config2(N=300_001) if which == "c2" else wl.config3(N=100_003)
    plain = _with_hint(cfg["csr"], 0)
    dt = plain.vals.dtype
    ref, mag = oracle.spmv(plain, cfg["x"])
    a, b = gpu_spmv(plain, cfg["x"], repeat=2)
    assert_close(a, ref, mag, dt, f"unhinted {which} csr")
    assert np.array_equal(a, b)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz_mod", [0, 1, 2, 3])
def test_csr_long_rows_among_short_ones(dtype, nnz_mod):
    """Mean row length 8, so the row kernel runs, but single rows hold 60, 3000, 9000 and
    40 000 entries: they are added up by a wave, or above 4096 entries by the workgroup. The entry
    count takes every remainder modulo 4 (the last vector of the arrays is moved back)."""
    N, M = 12_000, 50_000
    r, c, v = wl.random_coo_entries(N, M, 40_000 + nnz_mod, seed=70 + nnz_mod, dtype=dtype)
    rng = np.random.default_rng(71)
    rows, cols, vals = [r], [c], [v]
    for row, n in ((3, 60), (700, 3000), (701, 9000), (5000, 40_000), (N - 1, 5000)):
        keep = rows[0] != row
        rows[0], cols[0], vals[0] = rows[0][keep], cols[0][keep], vals[0][keep]
        rows.append(np.full(n, row))
        cols.append(np.sort(rng.choice(M, n, replace=False)))
        vals.append(rng.uniform(-1, 1, n).astype(dtype))
    r, c, v = np.concatenate(rows), np.concatenate(cols), np.concatenate(vals)
    r, c, v = r[: len(r) - (len(r) - nnz_mod) % 4], c[: len(r) - (len(r) - nnz_mod) % 4], v[: len(r) - (len(r) - nnz_mod) % 4]
    order = np.lexsort((c, r))
    spec = wl.csr_from_sorted_coo(N, M, r[order], c[order], v[order])
    assert len(spec.vals) % 4 == nnz_mod and len(spec.vals) <= 32 * N
    x = wl.dense_vector(M, 72, dtype)
    ref, mag = oracle.spmv(spec, x)
    a, b = gpu_spmv(spec, x, repeat=2)
    assert_close(a, ref, mag, dtype, "long rows, by rows")
    assert np.array_equal(a, b)
    assert_close(gpu_spmv(spec, x, misalign=True), ref, mag, dtype, "long rows, by rows, unaligned")
    assert_close(gpu_spmv(_with_hint(spec, 40_000), x), ref, mag, dtype, "long rows, entry-balanced")


@pytest.mark.parametrize("heavy_row", [0, 150_000])
def test_large_unhinted_csr_picks_its_kernel_on_the_device(heavy_row):
    """From 2^25 entries on, a CSR matrix without a declared row bound has the entry counts of
    its 256-row blocks inspected on the device: even blocks keep the row kernel (same bits
    as with a declared bound of 16), one block holding a 150 000-entry row switches to the
    entry-balanced kernel (same bits as with a declared bound of 150 000)."""
    N = M = 2_100_000
    K = 16
    rng = np.random.default_rng(90 + (heavy_row > 0))
    # near the diagonal: columns anywhere in an x of 8 MB would be gathered slice by slice, whatever the rows
    cols = (np.arange(N, dtype=np.int64)[:, None] + rng.integers(0, 7, (N, K)) + np.arange(K, dtype=np.int64)[None, :] * 7) % M
    cols.sort(axis=1)
    lens = np.full(N, K, dtype=np.int64)
    crd = cols.reshape(-1)
    if heavy_row:
        at = 1_234_567
        extra = np.sort(rng.choice(M, heavy_row, replace=False))
        crd = np.concatenate([crd[: at * K], extra, crd[(at + 1) * K:]])
        lens[at] = heavy_row
    del cols
    pos = np.concatenate([[0], np.cumsum(lens)])
    nnz = int(pos[-1])
    assert nnz >= 2**25 and nnz <= 32 * N
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    plain = wl.csr_spec(N, M, pos, crd, vals)
    x = wl.dense_vector(M, 92, np.float32)
    ref, mag = oracle.spmv(plain, x)
    a, b = gpu_spmv(plain, x, repeat=2)
    assert_close(a, ref, mag, np.float32, f"large unhinted csr, heavy row {heavy_row}")
    assert np.array_equal(a, b), "run-to-run bits differ"
    same = gpu_spmv(_with_hint(plain, heavy_row if heavy_row else K), x)
    assert np.array_equal(a, same), "the device-side choice differs from the expected kernel"
    other = gpu_spmv(_with_hint(plain, K if heavy_row else 100_000), x)
    assert_close(other, ref, mag, np.float32, "the kernel not chosen")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_csr_hint_that_the_data_violates_stays_correct(dtype):
    """A declared bound of 8 on a matrix with one row of 9000 entries: the row kernel gives
    the long row to its workgroup; slower, never wrong."""
    N, M = 3000, 10_000
    r, c, v = wl.random_coo_entries(N, M, 20_000, seed=77, dtype=dtype)
    rng = np.random.default_rng(78)
    long_cols = np.sort(rng.choice(M, 9000, replace=False))
    keep = r != 7
    r = np.concatenate([r[keep], np.full(9000, 7)])
    c = np.concatenate([c[keep], long_cols])
    v = np.concatenate([v[keep], rng.uniform(-1, 1, 9000).astype(dtype)])
    order = np.lexsort((c, r))
    lying = wl.csr_from_sorted_coo(N, M, r[order], c[order], v[order])
    lying.levels[1].max_children = 8
    x = wl.dense_vector(M, 79, dtype)
    ref, mag = oracle.spmv(lying, x)
    assert_close(gpu_spmv(lying, x), ref, mag, dtype, "violated hint")


def test_unsupported_and_invalid_descriptors_report_errors():
    import paper_1804_10112_amd as spt
    import torch
    c1 = wl.config1(N=64, nnz=100)
    c1["csr"].levels[1].max_children = 5000     # declared long rows: the kernel that needs a workspace
    A = spt.DeviceTensor(c1["csr"])
    x = torch.zeros(64, dtype=torch.float64, device="cuda")
    y = torch.zeros(64, dtype=torch.float64, device="cuda")
    with pytest.raises(spt.SptError) as e:
        spt.spt_spmv(A, x, y, None)          # workspace missing
    assert e.value.status == 3
    with pytest.raises(spt.SptError) as e:
        spt.spt_spmv(A, None, y, A.workspace(spt.SPT_OP_SPMV))
    assert e.value.status == 1


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("lengths", [
    [4], [0, 0, 4, 0], [1, 3], [3, 1, 0],                       # the fewest entries a vector load needs
    [7] * 1000, [0, 1, 2, 3, 4, 5] * 300, [33, 31] * 500,        # groups of every width
    [40] * 70 + [64, 65, 127, 128, 129, 255, 256, 257] * 3,      # lane group / wave boundary
    [2] * 50 + [4095, 4096, 4097, 9001] + [1] * 50 + [20_000],   # wave / workgroup boundary
], ids=lambda l: f"{len(l)}rows{sum(l)}")
def test_csr_row_lengths_at_the_edges_of_the_row_kernel(lengths, dtype):
    rng = np.random.default_rng(len(lengths))
    M = 30_000
    pos = np.concatenate([[0], np.cumsum(lengths)])
    crd = np.concatenate([np.sort(rng.choice(M, n, replace=False)) for n in lengths]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(crd)).astype(dtype)
    x = rng.uniform(-1, 1, M).astype(dtype)
    # a declared bound of 32 (violated here and there) takes the matrix by rows whatever its mean row
    spec = _with_hint(wl.csr_spec(len(lengths), M, pos, crd, vals), 32)
    _check(spec, x, "csr rows")
    ref, mag = oracle.spmv(spec, x)
    assert_close(gpu_spmv(spec, x, misalign=True), ref, mag, spec.vals.dtype, "csr rows, unaligned arrays")
    assert_close(gpu_spmv(_with_hint(spec, 0), x), ref, mag, spec.vals.dtype, "csr by the mean row")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("lengths", [
    [2, 0, 2, 2], [0, 1, 2, 3, 4, 5] * 50, [7, 0, 9] * 200, [31, 0, 33, 1] * 50,
    [16, 17, 32, 33, 64, 65, 127, 0, 128, 129, 255, 256, 257, 0] * 2 + [1] * 400,
    [4095, 0, 4096, 4097, 1, 9001, 0] + [3] * 1500,
], ids=lambda l: f"{len(l)}rows{sum(l)}")
def test_csr_infinities_and_nans_stay_in_their_rows(lengths, dtype):
    """A vector load reaches into the rows before and after: what it finds there is not multiplied.
    Every third row with entries holds one Inf or NaN, at its start, its end or its middle."""
    rng = np.random.default_rng(len(lengths))
    M = 12_000
    pos = np.concatenate([[0], np.cumsum(lengths)])
    crd = np.concatenate([np.sort(rng.choice(M, n, replace=False)) for n in lengths]).astype(np.int32)
    vals = rng.uniform(0.5, 1, len(crd)).astype(dtype)
    for q, r in enumerate(np.flatnonzero(lengths)[1::3]):
        at = (pos[r], pos[r + 1] - 1, (pos[r] + pos[r + 1]) // 2)[q % 3]
        vals[at] = (np.inf, np.nan, -np.inf, np.inf)[q % 4]
    x = rng.uniform(0.5, 1, M).astype(dtype)
    rows = np.repeat(np.arange(len(lengths)), lengths)
    plain = wl.csr_spec(len(lengths), M, pos, crd, vals)
    ref, mag = oracle.spmv(plain, x)
    assert np.isfinite(ref).any() and not np.isfinite(ref).all()
    dcsr = wl.dcsr_from_sorted_coo(len(lengths), M, rows, crd, vals)
    for spec, what in ((plain, "csr"), (_with_hint(plain, 32), "csr by rows"),
                       (_with_hint(plain, 100_000), "csr by entries"), (dcsr, "dcsr")):
        assert_close_where_finite(gpu_spmv(spec, x), ref, mag, dtype, what)
    every = np.arange(M)
    for xs in (wl.sparse_vector_spec(M, every, x), wl.hash_vector_spec(M, every, x, 2 * M)):
        for spec in (plain, _with_hint(plain, 32)):
            assert_close_where_finite(gpu_spmv_sparse_x(spec, xs), ref, mag, dtype, xs.name)


@pytest.mark.parametrize("case", ["even", "long rows", "ends on a vector", "x beyond an L2"])
def test_csr_fp32_streamed_through_lds(case):
    """fp32 matrices of more than 12M entries, 8 to 32 per row, whose x fits an L2: rows of 0 to 32 entries,
    some of 49 to 60 000 (a wave's, several pieces', a block that goes by rows), an infinity and a NaN."""
    rng = np.random.default_rng(11)
    N = 620_000 if case != "x beyond an L2" else 800_000
    M = 700_000 if case != "x beyond an L2" else 1_700_000
    lens = rng.integers(8, 33, N)
    lens[rng.integers(0, N, 2000)] = 0
    if case == "long rows":
        for row, n in ((5, 49), (6, 2048), (300, 5000), (9_999, 12_000), (10_001, 30_000), (40_000, 60_000), (N - 1, 700)):
            lens[row] = n
    pos = np.concatenate([[0], np.cumsum(lens)])
    if case == "ends on a vector":
        lens[-1] += -pos[-1] % 4
        pos[-1] = pos[-2] + lens[-1]
    nnz = int(pos[-1])
    assert 96e6 < 8 * nnz and 8 * N <= nnz <= 32 * N
    crd = rng.integers(0, M, nnz, dtype=np.int32)
    vals = rng.uniform(-1, 1, nnz).astype(np.float32)
    vals[pos[1000]], vals[pos[5001] - 1] = np.inf, np.nan
    x = rng.uniform(0.5, 1, M).astype(np.float32)
    spec = wl.csr_spec(N, M, pos, crd, vals)
    ref, mag = oracle.spmv(spec, x)
    a, b = gpu_spmv(spec, x, repeat=2)
    assert_close_where_finite(a, ref, mag, np.float32, case)
    assert np.array_equal(a, b, equal_nan=True), "run-to-run bits differ"
    assert_close_where_finite(gpu_spmv(spec, x, misalign=True), ref, mag, np.float32, f"{case}, unaligned arrays")


def _device_matrix(rows, nnz, dcsr):
    """nnz entries dealt out evenly to the rows, anywhere in 10^6 columns; arrays on the GPU."""
    import torch
    import paper_1804_10112_amd as spt
    M = 1_000_000
    A = spt.DeviceTensor((wl.dcsr_from_sorted_coo if dcsr else wl.csr_from_sorted_coo)(
        rows, M, np.arange(rows), np.zeros(rows, np.int64), np.ones(rows, np.float32)))
    pos = (torch.arange(rows + 1, device="cuda") * nnz // rows).int()
    crd = torch.randint(0, M, (nnz,), device="cuda", dtype=torch.int32)
    vals = torch.rand(nnz, device="cuda")
    A.c.level[1].pos, A.c.level[1].crd, A.c.vals, A.c.nvals = pos.data_ptr(), crd.data_ptr(), vals.data_ptr(), nnz
    return A, (pos, crd, vals)


@pytest.mark.parametrize("nnz,rows", [(20_000_000, 1), (10_000_000, 100), (500_000, 3)])
@pytest.mark.parametrize("form", ["csr", "dcsr", "sparse x", "hashed x", "ttv csf"])
def test_few_long_rows_do_not_wait_for_one_workgroup(nnz, rows, form):
    """The same entries in few rows and in rows of 16 take about the same time: by rows, a workgroup
    per long row, they took 10 to 100 times as long. And the sums are right."""
    import torch
    import paper_1804_10112_amd as spt
    M = 1_000_000
    xd = torch.rand(M, device="cuda")
    X = {"sparse x": wl.sparse_vector_spec(M, np.arange(64) * 15_000, np.ones(64, np.float32)),
         "hashed x": wl.hash_vector_spec(M, np.arange(64) * 15_000, np.ones(64, np.float32), 128)}.get(form)
    if X is not None:
        xd = torch.zeros(M, device="cuda")
        xd[torch.arange(64, device="cuda") * 15_000] = 1
        X = spt.DeviceTensor(X)
    if form == "ttv csf":
        nnz = min(nnz, (1 << 19) - 1)   # above, TTV walks over entries anyway

    def best(n_rows):
        A, keep = _device_matrix(n_rows, nnz, form == "dcsr")
        y = torch.empty(n_rows, device="cuda")
        ws = A.workspace(spt.SPT_OP_SPMV)
        if form == "ttv csf":
            B = spt.DeviceTensor(wl.csf3_from_sorted_coo((1, n_rows, M), np.zeros(n_rows, np.int64), np.arange(n_rows),
                                                         np.zeros(n_rows, np.int64), np.ones(n_rows, np.float32)))
            B.c.level[2].pos, B.c.level[2].crd, B.c.vals, B.c.nvals = A.c.level[1].pos, A.c.level[1].crd, A.c.vals, nnz
            count = torch.zeros(1, dtype=torch.int64, device="cuda")
            ws = B.workspace(spt.SPT_OP_TTV)
        times = []
        for _ in range(4):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            if form == "ttv csf":
                spt.spt_ttv(B, xd, None, None, y, count, ws)
            elif X is not None:
                spt.spt_spmv_sparse_x(A, X, y, ws)
            else:
                spt.spt_spmv(A, xd, y, ws)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        pos, crd, vals = keep
        terms = vals.double() * xd[crd.long()].double()
        before = torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64), terms.cumsum(0)])
        ref = (before[pos[1:].long()] - before[pos[:-1].long()]).cpu().numpy()
        # no term is negative; ref itself, a difference of running sums up to 10^7, is right to 1e-8
        assert_close(y.cpu().numpy(), ref, ref + 1e-3, np.float32, f"{form} {n_rows} rows")
        return min(times)

    long, short = best(rows), best(nnz // 16)
    assert long < 3 * short + 0.05, f"{form}: {long:.3f} ms in {rows} rows, {short:.3f} ms in rows of 16"


@pytest.mark.parametrize("nnz,rows", [(1000, 2), (40_000, 5)])
def test_csr_long_rows_without_a_workspace_are_walked(nnz, rows):
    import torch
    import paper_1804_10112_amd as spt
    A, (pos, crd, vals) = _device_matrix(rows, nnz, False)
    x, y = torch.rand(1_000_000, device="cuda"), torch.empty(rows, device="cuda")
    spt.spt_spmv(A, x, y, None)
    ref = (vals.double() * x[crd.long()].double()).reshape(rows, -1).sum(1).cpu().numpy()
    assert_close(y.cpu().numpy(), ref, ref, np.float32, "no workspace")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_csr_two_rows_per_group(dtype):
    """Above 2^20 entries with short rows a group of lanes takes two rows at once."""
    c2 = wl.config2(N=180_001, dtype=dtype)
    _check(c2["csr"], c2["x"], "csr short rows")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 127, 129, 255, 257, 511, 513, 1027])
def test_dia_and_ell_at_any_row_count(N, dtype):
    """Row counts around the vectors, waves and workgroups; fewer and more slots than one batch."""
    c2 = wl.config2(N=N, poison=True, dtype=dtype) if N >= 127 else None
    if c2:
        _check(c2["dia"], c2["x"], f"dia N={N}")
    for lo, hi in ((0, 3), (2, 9), (1, min(33, N + 1))):
        c3 = wl.config3(N=N, lo=min(lo, N), hi=min(hi, N), dtype=dtype, seed=N + hi)
        _check(c3["ell"], c3["x"], f"ell N={N} W={c3['W']}")
    M = 3 * N + 5                                   # rectangular, diagonals that leave the matrix early
    off = np.array([-(N - 1), -1, 0, 2, N, M - 1]) if N > 1 else np.array([0, M - 1])
    vals = np.random.default_rng(N).uniform(-1, 1, (len(off), N)).astype(dtype)
    _check(wl.dia_spec(N, M, off, vals), wl.dense_vector(M, 5, dtype), f"dia N={N} M={M}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [1, 255, 256, 1023, 1024, 1025, 30_001])
def test_unordered_coo_and_csc_by_atomics(nnz, dtype):
    """Around the 1024 entries of a workgroup; one row, few rows, and more rows than the table has slots."""
    rng = np.random.default_rng(nnz)
    M = 700
    for N in (1, 3, 900, 5000, 3_000_000):
        r, c = rng.integers(0, N, nnz), rng.integers(0, M, nnz)
        v = rng.uniform(-1, 1, nnz).astype(dtype)
        v[nnz // 2] = np.inf
        x = rng.uniform(0.5, 1, M).astype(dtype)
        ref, mag = oracle.spmv(wl.coo_spec(N, M, r, c, v, ordered=False), x)
        for spec in (wl.coo_spec(N, M, r, c, v, ordered=False), wl.csc_from_coo(N, M, r, c, v)):
            assert_close_where_finite(gpu_spmv(spec, x), ref, mag, dtype, f"{spec.name} nnz={nnz} N={N}")


def test_unordered_coo_with_a_heavy_row_takes_no_longer():
    """Half of 400 000 entries in one row: with an atomic for each, 2.4 ms instead of 0.02."""
    import torch
    import paper_1804_10112_amd as spt
    n, N, M = 400_000, 25_000, 25_000
    rng = np.random.default_rng(2)
    times = []
    for heavy in (0, n // 2):
        r = rng.integers(0, N, n)
        r[:heavy] = N // 3
        A = spt.DeviceTensor(wl.coo_spec(N, M, rng.permutation(r), rng.integers(0, M, n), np.ones(n), ordered=False))
        x, y = torch.ones(M, dtype=torch.float64, device="cuda"), torch.empty(N, dtype=torch.float64, device="cuda")
        ws = A.workspace(spt.SPT_OP_SPMV)
        best = 1e9
        for _ in range(5):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            spt.spt_spmv(A, x, y, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        times.append(best)
        assert np.array_equal(y.cpu().numpy(), np.bincount(r, minlength=N))
    assert times[1] < 3 * times[0] + 0.05, f"{times[1]:.3f} ms with a heavy row, {times[0]:.3f} without"


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [786_431, 786_432, 786_433, 1_100_003])
def test_unordered_coo_where_binning_begins(nnz, dtype):
    rng = np.random.default_rng(nnz)
    for N, M, heavy in ((30_000, 20_000, 0), (5, 7000, 0), (100_000, 9000, 400_000)):
        r, c = rng.integers(0, N, nnz), rng.integers(0, M, nnz)
        r[:heavy] = N // 3                              # one row: its bin has several slices
        p = rng.permutation(nnz)
        _check(wl.coo_spec(N, M, r[p], c[p], rng.uniform(-1, 1, nnz).astype(dtype), ordered=False),
               wl.dense_vector(M, 5, dtype), f"unordered nnz={nnz} N={N} heavy={heavy}")


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nnz", [65_537, 65_792, 200_001, 1_000_000])
def test_ordered_coo_in_pieces(nnz, dtype):
    """Pieces of 256 entries: long gaps of rows without entries (zeroed by the pieces up to 2^18 rows, by
    a fill beyond), a row of many pieces, rows that start and end with a piece."""
    rng = np.random.default_rng(nnz)
    for N in (262_144, 262_145, 3):
        r = rng.integers(0, N, nnz)
        if N > 3:
            r[r < N // 3] = N // 3                      # one row of a third of the entries after a gap
            r[(r > N // 2) & (r < N - 20_000)] = N // 2
        r = np.sort(r)
        r[: 1024] = np.repeat(r[0], 1024)
        c = rng.integers(0, 5000, nnz)
        _check(wl.coo_spec(N, 5000, r, c, rng.uniform(-1, 1, nnz).astype(dtype)), wl.dense_vector(5000, 5, dtype),
               f"ordered coo nnz={nnz} N={N}")


def test_ordered_coo_on_both_sides_of_the_largest_in_pieces():
    rng = np.random.default_rng(3)
    n = (1 << 24) + 1
    r, c, v = np.sort(rng.integers(0, 400_000, n)), rng.integers(0, 9000, n), rng.uniform(-1, 1, n)
    for m in (n, n - 1):
        _check(wl.coo_spec(400_000, 9000, r[:m], c[:m], v[:m]), wl.dense_vector(9000, 5, np.float64), f"nnz={m}")


@pytest.mark.parametrize("form", ["unordered coo", "csr", "csr, long rows"])
def test_entries_up_to_the_largest_index(form):
    """As many entries as each path takes: what its loops look ahead passes 2^31. All values and x are
    one, so that every sum is the (exact) length of its row."""
    import torch
    import paper_1804_10112_amd as spt
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    N, M = 700_001, 1000
    n = (1 << 31) - 4098 if form == "unordered coo" else (1 << 31) - 2
    i32 = dict(dtype=torch.int32, device="cuda")
    col = torch.arange(n, **i32).remainder_(M)
    vals, x = torch.ones(n, device="cuda"), torch.ones(M, device="cuda")
    if form == "unordered coo":
        row = torch.arange(n, **i32).remainder_(N)
        A = spt.DeviceTensor(wl.coo_spec(N, M, [0], [0], np.ones(1, np.float32), ordered=False))
        A.c.level[0].crd, A.c.level[1].crd = row.data_ptr(), col.data_ptr()
        length = n // N + (torch.arange(N, device="cuda") < n % N)
    else:
        N = n // 16 if form == "csr" else 400_000
        length = torch.full((N,), n // N, device="cuda")
        length[-1] += n % N                                # the last row is the longest, and ends the arrays
        pos = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), length.cumsum(0)]).int()
        A = spt.DeviceTensor(wl.csr_spec(1, M, [0, 1], [0], np.ones(1, np.float32), max_row=16))
        A.c.level[0].N = A.c.level[1].M = N
        A.c.level[1].pos, A.c.level[1].crd = pos.data_ptr(), col.data_ptr()
    A.c.vals, A.c.nvals = vals.data_ptr(), n
    y = torch.full((N,), -1.0, device="cuda")
    spt.spt_spmv(A, x, y, A.workspace(spt.SPT_OP_SPMV))
    assert torch.equal(y, length.float())
    del col, vals, y, length
    torch.cuda.empty_cache()
