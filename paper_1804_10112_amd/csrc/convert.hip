// COO -> CSR (paper Section 5.4, Figure 14) on gfx950.
//
//   1. reorder (Section 4.3 "reordering"): from 16 385 records to 3M, fewer where rows are short, by
//      reserved regions (reserve_sort.hip), else up to 2^26 by sample sort (sample_sort.hip), which
//      both assemble pos, too; beyond, and where few passes do, a stable
//      least-significant-digit radix sort of the (row, col, value) records, 8 bits per pass, over the
//      significant bits of the column (ROW_COL order only) and then of the row.
//      Every pass is histogram -> exclusive scan -> stable scatter; the records
//      themselves travel, so no gather through a permutation is needed.
//   2. assemble pos. Table 3 prescribes, for a compressed level, per-row counts
//      (append_edges) followed by a running sum (append_finalize); on sorted rows
//      that sum is the position of the first entry of each row and is stored
//      directly at the row boundaries (see pos_from_sorted_rows_kernel).
// Everything is integer or bit-copy work: results are exact and deterministic.
#include "common.hpp"
#include "radix.hpp"
#include "rows.hpp"
#include "scan.hpp"

namespace spt {

// Stable scatter of one pass. Element order inside a tile is (wave, item, lane);
// a lane's rank among equal digits comes from a ballot-based match inside the
// wave plus per-wave running digit counters in LDS, so equal keys keep their
// input order. The tile is then sorted by digit inside LDS (one array at a time
// through the same buffer) so that consecutive lanes store to consecutive
// addresses of each digit's run: scattered single-lane stores cost one memory
// transaction each, exactly like random gathers. off[d * ntiles + tile] is the
// exclusive scan of hist.
template <typename VT>
__global__ __launch_bounds__(kBlock) void radix_scatter_kernel(
    int n, int shift, int key_is_row, int ntiles, const int32_t* __restrict__ off,
    const int32_t* __restrict__ row_in, const int32_t* __restrict__ col_in,
    const VT* __restrict__ val_in, int32_t* __restrict__ row_out, int32_t* __restrict__ col_out,
    VT* __restrict__ val_out) {
  __shared__ int s_cnt[kWaves][kRadix];
  __shared__ int s_gdelta[kRadix];
  __shared__ VT s_buf[kSortTile];
  int32_t* s_buf32 = reinterpret_cast<int32_t*>(s_buf);
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  // neighbouring tiles store to neighbouring addresses of every digit's run: keep them on
  // one XCD so that partially written cache lines meet in the same L2
  const int tile = xcd_contiguous_block_id();
  for (int q = tid; q < kWaves * kRadix; q += kBlock) (&s_cnt[0][0])[q] = 0;
  __syncthreads();

  const int32_t* __restrict__ key_in = key_is_row ? row_in : col_in;
  const int32_t* __restrict__ oth_in = key_is_row ? col_in : row_in;
  int32_t* __restrict__ key_out = key_is_row ? row_out : col_out;
  int32_t* __restrict__ oth_out = key_is_row ? col_out : row_out;
  const int tile_base = tile * kSortTile;
  const int tile_n = min(kSortTile, n - tile_base);
  const int wave_base = tile_base + w * (kWave * kSortIPT);
  const uint64_t lanes_below = ((uint64_t)1 << lane) - 1;
  // (Volatile, so flat operations instead of LDS ones: with those the ranks are done sooner, and what more is then under
  // way of the 256 x 3 interleaved streams costs more than that: by rows, 60M records fp64 1.58 -> 1.79 ms, fp32
  // 1.40 -> 1.59, 30M 858 -> 904 and 741 -> 787 us; 8M 276 -> 268. Two workgroups on a compute unit: 60M 1.61, 8M 287.)
  volatile int* cnt = s_cnt[w];

  int32_t key[kSortIPT], oth[kSortIPT];
  VT val[kSortIPT];
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {  // all loads of the tile are issued up front
    const int i = wave_base + k * kWave + lane;
    const bool valid = i < n;
    key[k] = valid ? key_in[i] : 0;
    oth[k] = valid ? oth_in[i] : 0;
    val[k] = valid ? val_in[i] : VT(0);
  }
  int lpos[kSortIPT];  // first the rank inside (wave, digit), later the slot in the sorted tile
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const bool valid = wave_base + k * kWave + lane < n;
    const int d = digit_of(key[k], shift);
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t vote = __ballot(valid && bit);
      same &= bit ? vote : ~vote;
    }
    const int before = __popcll(same & lanes_below);
    int basecnt = 0;
    if (valid) basecnt = cnt[d];
    __builtin_amdgcn_wave_barrier();
    if (valid && before == 0) cnt[d] = basecnt + __popcll(same);
    __builtin_amdgcn_wave_barrier();
    lpos[k] = basecnt + before;
  }
  __syncthreads();
  {  // thread d: where digit d starts inside the sorted tile and in global memory
    const int d = tid;
    int c[kWaves], tot = 0;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      c[u] = s_cnt[u][d];
      tot += c[u];
    }
    int all;
    int start = block_inclusive_sum(tot, &all) - tot;
    s_gdelta[d] = off[(int64_t)d * ntiles + tile] - start;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      s_cnt[u][d] = start;
      start += c[u];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    if (wave_base + k * kWave + lane < n) {
      lpos[k] += s_cnt[w][digit_of(key[k], shift)];
      s_buf32[lpos[k]] = key[k];
    }
  }
  __syncthreads();
  int dst[kSortIPT];
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const int j = k * kBlock + tid;
    if (j < tile_n) {
      const int32_t kk = s_buf32[j];
      dst[k] = j + s_gdelta[digit_of(kk, shift)];
      key_out[dst[k]] = kk;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k)
    if (wave_base + k * kWave + lane < n) s_buf32[lpos[k]] = oth[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const int j = k * kBlock + tid;
    if (j < tile_n) oth_out[dst[k]] = s_buf32[j];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k)
    if (wave_base + k * kWave + lane < n) s_buf[lpos[k]] = val[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const int j = k * kBlock + tid;
    if (j < tile_n) val_out[dst[k]] = s_buf[j];
  }
}

template <typename VT>
__global__ __launch_bounds__(kBlock) void copy_entries_kernel(int n, const int32_t* __restrict__ col_in,
                                                              const VT* __restrict__ val_in,
                                                              int32_t* __restrict__ col_out,
                                                              VT* __restrict__ val_out) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p < n) {
    col_out[p] = col_in[p];
    val_out[p] = val_in[p];
  }
}

__global__ __launch_bounds__(kBlock) void zero_i32_kernel(int32_t* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) out[i] = 0;
}

struct SortPlan {
  int passes_col, passes_row, ntiles;
  size_t rec_bytes, hist_bytes, scan_bytes, total;
};

static SortPlan plan(const spt_tensor* A, int32_t order) {
  SortPlan P;
  const int64_t nnz = A->nvals;
  const size_t vsz = A->dtype == SPT_F64 ? 8 : 4;
  P.passes_col = order == SPT_ORDER_ROW_COL ? (bits_for(A->level[1].N) + kRadixBits - 1) / kRadixBits : 0;
  P.passes_row = (bits_for(A->level[0].N) + kRadixBits - 1) / kRadixBits;
  P.ntiles = (int)((nnz + kSortTile - 1) / kSortTile);
  // records between passes: the last one writes columns and values to the caller's arrays
  const int passes = P.passes_col + P.passes_row;
  const size_t row = align_up((size_t)nnz * 4, 256), rest = row + align_up((size_t)nnz * vsz, 256);
  P.rec_bytes = std::min(passes, 2) * row + std::min(passes - 1, 2) * rest;
  P.hist_bytes = align_up((size_t)kRadix * P.ntiles * 4, 256);
  const int64_t scan_n = std::max<int64_t>((int64_t)kRadix * P.ntiles, A->level[0].N + 1);
  P.scan_bytes = scan_workspace(scan_n);
  P.total = P.rec_bytes + P.hist_bytes + P.scan_bytes + 256;
  return P;
}

// sample sort (sample_sort.hip): up to 2^26 records
bool sample_sort_applies(int64_t n);
size_t sample_sort_workspace(int dtype, int64_t n);
template <typename VT>
spt_status sample_sort_convert(int64_t n, int64_t nrows, int64_t ncols, bool by_col, const int32_t* row,
                               const int32_t* col, const VT* vals, int32_t* pos_out, int32_t* crd_out,
                               VT* vals_out, void* ws, size_t ws_bytes, hipStream_t s);

// sort by reserved regions (reserve_sort.hip): a middling number of records, up to 3M
bool reserve_sort_applies(int64_t n, int64_t nrows, int64_t ncols);
size_t reserve_sort_workspace(int dtype, int64_t n);
template <typename VT>
spt_status reserve_sort_convert(int64_t n, int64_t nrows, int64_t ncols, bool by_col, const int32_t* row,
                                const int32_t* col, const VT* vals, int32_t* pos_out, int32_t* crd_out,
                                VT* vals_out, void* ws, size_t ws_bytes, hipStream_t s);

// Where the sort by reserved regions does not apply: the sample sort takes one launch, one partition or two and a finish,
// whatever the key; a radix sort a pass per 8 bits of it. Keys of few bits (a stable order of the rows, small matrices) are for
// the latter from where the sample sort needs its next step (fp64, even rows, in us, radix / sample):
//   passes            130 000     400 000     1.6M         6.4M         30M
//   1 (200 rows)       30 / 36     31 / 62     37 / 96      84 / 228    295 / 857
//   2 (60 000 rows)    61 / 35     62 / 59     70 / 93     169 / 217    586 / 791
//   3 (4M rows)       115 / 88    108 / 77    119 / 97     257 / 212    858 / 760
//   4                 144 / 93    138 / 83    152 / 97     335 / 209   1134 / 755
// Three passes: rows of power-law lengths cost the sample sort more and radix passes nothing. 1.8M fp64 104 / 104, fp32 100 /
// 97; 2M 106 / 114; 6.4M fp64 249 / 228, fp32 197 / 211; 12M 383 / 429; 30M 835 / 859; 60M 1561 / 1651 (even rows 1586 / 1483).
static bool radix_is_faster(const SortPlan& P, const spt_tensor* A) {
  const int passes = P.passes_col + P.passes_row;
  const int64_t from = passes == 1 ? 1 << 16 : passes == 2 ? 256 * 1408 : 7 << 18;
  return !sample_sort_applies(A->nvals) || (passes <= 3 && A->nvals > from);
}

// From 16 384 records on the sort by reserved regions is faster than the sample sort (its plan says by how much), up to 3M: beyond, more
// and more of its buckets take nine words of a thread, and one that a long row's neighbours crowd is sorted late. Power-law rows, reserved / sample
// sort, us: of three entries on average 1.7M 93 / 102, 1.9M fp32 99 / 103, 2.2M fp64 108 / 124, fp32 114 / 112, 3M 152 / 143; of four to eight
// 2M 88 / 108, 2.6M fp32 127 / 115; of 15 2.2M 99 / 112, 3M fp64 118 / 137, fp32 113 / 128, 4M 186 / 162 (uniform ones of
// five 137 / 153, but the host sees only the mean). Keys of three radix passes: 2.6M rows in a stable order 100 / 119, 3.1M of power-law
// lengths, fp32, 118 / 114. Radix passes (fp64, in us, reserved / radix): one pass 30.1 / 30.4 at 400 000, 37 / 31 at
// 640 000; two 47 / 67 at 1M, 73 / 70 at 1.6M.
static bool reserve_is_fastest(const SortPlan& P, const spt_tensor* A) {
  const int passes = P.passes_col + P.passes_row;
  const int64_t mean = A->nvals / std::max<int64_t>(A->level[0].N, 1);
  const int64_t most = passes == 1 ? 3 << 17 : passes == 2 ? 5 << 18 : mean < 4 ? 7 << 18 : mean < 12 ? 2 << 20 : passes == 3 ? 5 << 19 : 3 << 20;
  return A->nvals <= most && reserve_sort_applies(A->nvals, A->level[0].N, A->level[1].N);
}

// What a call needs. The query asks for more where the sort by reserved regions is the fastest.
static size_t least_workspace(const spt_tensor* A) {
  if (A->nvals == 0) return 256;  // pos is cleared
  size_t need = sample_sort_applies(A->nvals) ? sample_sort_workspace(A->dtype, A->nvals) : 0;
  for (const int32_t order : {SPT_ORDER_ROW_COL, SPT_ORDER_ROW_STABLE}) {
    const SortPlan P = plan(A, order);
    if (radix_is_faster(P, A)) need = std::max(need, P.total);
  }
  return need;
}

// Do the flags say that the entries are in this order?
static bool in_order(const spt_tensor* A, int32_t order) {
  return (A->level[0].flags & SPT_ORDERED) && (order == SPT_ORDER_ROW_STABLE || (A->level[1].flags & SPT_ORDERED));
}

size_t coo_to_csr_workspace(const spt_tensor* A) {
  const size_t need = least_workspace(A);
  const auto reserves = [&](int32_t order) { return !in_order(A, order) && reserve_is_fastest(plan(A, order), A); };
  const bool reserve = reserves(SPT_ORDER_ROW_COL) || reserves(SPT_ORDER_ROW_STABLE);
  return reserve ? std::max(need, reserve_sort_workspace(A->dtype, A->nvals)) : need;
}

template <typename VT>
static spt_status convert_typed(const spt_tensor* A, int32_t order, int32_t* pos_out,
                                int32_t* crd_out, VT* vals_out, void* ws, size_t ws_bytes,
                                hipStream_t s) {
  const int64_t nnz64 = A->nvals, N = A->level[0].N;
  if (nnz64 + kSortTile >= INT32_MAX || N + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "coo_to_csr: more than 2^31 entries or rows");
  const int nnz = (int)nnz64;
  const size_t need = least_workspace(A);
  if (!ws || ws_bytes < need)
    return fail(SPT_ERR_WORKSPACE, "coo_to_csr: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  const int32_t* row = A->level[0].crd;
  const int32_t* col = A->level[1].crd;
  const VT* vals = static_cast<const VT*>(A->vals);

  if (nnz == 0) {
    hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)((N + 1 + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, pos_out, N + 1);
    SPT_CHECK_LAUNCH("zero pos");
    return SPT_OK;
  }

  const bool sorted_in = in_order(A, order);
  const int32_t* sorted_rows = row;
  const unsigned egrid = (unsigned)((nnz + kBlock - 1) / kBlock);
  if (sorted_in) {
    hipLaunchKernelGGL(copy_entries_kernel<VT>, dim3(egrid), dim3(kBlock), 0, s, nnz, col, vals,
                       crd_out, vals_out);
    SPT_CHECK_LAUNCH("copy_entries");
  } else if (reserve_is_fastest(plan(A, order), A) && ws_bytes >= reserve_sort_workspace(A->dtype, nnz64)) {
    return reserve_sort_convert<VT>(nnz64, N, A->level[1].N, order == SPT_ORDER_ROW_COL, row, col, vals, pos_out,
                                    crd_out, vals_out, ws, ws_bytes, s);
  } else if (!radix_is_faster(plan(A, order), A)) {
    return sample_sort_convert<VT>(nnz64, N, A->level[1].N, order == SPT_ORDER_ROW_COL, row, col, vals, pos_out,
                                   crd_out, vals_out, ws, ws_bytes, s);
  } else {
    const SortPlan P = plan(A, order);
    Workspace W(ws, ws_bytes);
    const int npass = P.passes_col + P.passes_row;
    int32_t *srow[2] = {}, *scol[2] = {};
    VT* sval[2] = {};
    for (int b = 0; b < std::min(npass, 2); ++b) srow[b] = W.take<int32_t>(nnz);
    for (int b = 0; b < std::min(npass - 1, 2); ++b) {
      scol[b] = W.take<int32_t>(nnz);
      sval[b] = W.take<VT>(nnz);
    }
    int32_t* hist = W.take<int32_t>((size_t)kRadix * P.ntiles);
    int32_t* scan_tmp = reinterpret_cast<int32_t*>(W.take<char>(P.scan_bytes));
    const int32_t *rin = row, *cin = col;
    const VT* vin = vals;
    for (int i = 0; i < npass; ++i) {
      const bool is_row = i >= P.passes_col;
      const int shift = kRadixBits * (is_row ? i - P.passes_col : i);
      const bool last = i == npass - 1;
      int32_t* rout = srow[i & 1];
      int32_t* cout = last ? crd_out : scol[i & 1];
      VT* vout = last ? vals_out : sval[i & 1];
      spt_status hs = launch_radix_hist(is_row ? rin : cin, nnz, shift, P.ntiles, hist, s);
      if (hs != SPT_OK) return hs;
      spt_status st = device_scan_i32<false>(hist, hist, (int64_t)kRadix * P.ntiles, scan_tmp, s);
      if (st != SPT_OK) return st;
      hipLaunchKernelGGL(radix_scatter_kernel<VT>, dim3(P.ntiles), dim3(kBlock), 0, s, nnz, shift,
                         (int)is_row, P.ntiles, hist, rin, cin, vin, rout, cout, vout);
      SPT_CHECK_LAUNCH("radix_scatter");
      rin = rout;
      cin = cout;
      vin = vout;
    }
    sorted_rows = rin;
  }
  spt_status ps = launch_pos_from_sorted_rows(sorted_rows, nnz, (int)N, pos_out, s);
  if (ps != SPT_OK) return ps;
  return SPT_OK;
}

spt_status coo_to_csr_dispatch(const spt_tensor* A, int32_t order, int32_t* pos_out,
                               int32_t* crd_out, void* vals_out, void* ws, size_t ws_bytes,
                               hipStream_t s) {
  if (A->dtype == SPT_F64)
    return convert_typed<uint64_t>(A, order, pos_out, crd_out, static_cast<uint64_t*>(vals_out), ws,
                                   ws_bytes, s);
  return convert_typed<uint32_t>(A, order, pos_out, crd_out, static_cast<uint32_t*>(vals_out), ws,
                                 ws_bytes, s);
}

}  // namespace spt
