// SpMV on UNORDERED COO without one global atomic per entry.
//
// The paper's COO kernel is a single fused loop that scatters v*x[j] into y
// (Section 4.5, fusing iterators; Section 5.2.1). A literal GPU version issues
// one floating-point atomic per stored entry at a random address, which the
// memory system serves at only ~15 G atomics/s. Here the scatter is split in
// two coalesced steps:
//   1. bin: one pass of the radix machinery moves (row, v*x[col]) into 256 bins of
//      equally many rows (histogram, scan, stable scatter);
//      the gather of x happens here, once per entry.
//   2. accumulate: a workgroup owns a slice of one bin's entries and a sub-range
//      of the bin's rows that fits LDS (128 KB: usually the whole bin), adds the products
//      with LDS atomics and stores its rows: to y when it holds the whole bin, otherwise
//      to scratch, from where a last kernel adds up the slices of each bin.
// Like the atomic kernel the result is order-dependent in the last bits
// (tolerance-checked, not bit-reproducible); the ordered COO path is exact-order.
#include <algorithm>

#include "common.hpp"
#include "radix.hpp"
#include "scan.hpp"
#include "wavescan.hpp"

namespace spt {

template <typename T>
__device__ __forceinline__ T ld_nt(const T* p) {
  return __builtin_nontemporal_load(p);
}

// Stable scatter by bin of (row, vals * x[col]); the same
// ranking and in-LDS tile sort as the sort's scatter kernel.
template <typename T>
__global__ __launch_bounds__(kBlock) void bin_scatter_kernel(
    int n, const StretchDigit digit, int ntiles, const int32_t* __restrict__ off, const int32_t* __restrict__ row,
    const int32_t* __restrict__ col, const T* __restrict__ vals, const T* __restrict__ x,
    int32_t* __restrict__ brow, T* __restrict__ bprod) {
  __shared__ int s_cnt[kWaves][kRadix];
  __shared__ int s_gdelta[kRadix];
  __shared__ T s_buf[kSortTile];
  int32_t* s_buf32 = reinterpret_cast<int32_t*>(s_buf);
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const int tile = xcd_contiguous_block_id();
  for (int q = tid; q < kWaves * kRadix; q += kBlock) (&s_cnt[0][0])[q] = 0;
  __syncthreads();
  const int tile_base = tile * kSortTile;
  const int tile_n = min(kSortTile, n - tile_base);
  const int wave_base = tile_base + w * (kWave * kSortIPT);
  const uint64_t lanes_below = ((uint64_t)1 << lane) - 1;
  volatile int* cnt = s_cnt[w];

  int32_t key[kSortIPT];
  T prod[kSortIPT];
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const int i = wave_base + k * kWave + lane;
    const bool valid = i < n;
    key[k] = valid ? ld_nt(row + i) : 0;
    prod[k] = valid ? ld_nt(vals + i) * x[ld_nt(col + i)] : T(0);
  }
  int lpos[kSortIPT];
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const bool valid = wave_base + k * kWave + lane < n;
    const int d = digit.of(key[k]);
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
  {
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
      lpos[k] += s_cnt[w][digit.of(key[k])];
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
      dst[k] = j + s_gdelta[digit.of(kk)];
      brow[dst[k]] = kk;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k)
    if (wave_base + k * kWave + lane < n) s_buf[lpos[k]] = prod[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortIPT; ++k) {
    const int j = k * kBlock + tid;
    if (j < tile_n) bprod[dst[k]] = s_buf[j];
  }
}

// Work item = (bin b, slice k of the bin's entries, row sub-range sub).
// Bound by the LDS atomics (2.4 to 3.2 clocks per lane, fp64 and fp32): what counts is that all
// compute units have equally many. Bins of about the same size are one slice each. If one holds more
// than one and a half times the mean (it has long rows), all bins are cut in slices of an eighth of
// the mean, but of no fewer entries than six times the rows of a bin, so that storing and adding up
// the slices' rows costs little next to the entries. Whole call, power-law rows, 10M entries, fp32:
// 230 us, with only the larger bins cut 271; uniform rows, 12.8M entries, fp32: 259 us, with every
// bin cut 281 to 291.
struct Cut {
  int even, slice;  // the largest bin of an even matrix; the longest slice of any other
  Cut() = default;
  Cut(int64_t nnz, int64_t rows_in_bin) {
    even = (int)std::max<int64_t>(nnz / kRadix * 3 / 2, 8192);
    slice = (int)std::max<int64_t>({nnz / (8 * kRadix), 6 * rows_in_bin, 8192});
  }
};

// Where the slices of the 256 bins lie: first[b] = slices before bin b, wide[b] = slices of bins
// with more than one slice before bin b (their place in scratch). Every thread of the workgroup
// calls; the result is ready after it.
struct SliceTable {
  int start[kRadix + 1], first[kRadix + 1], wide[kRadix + 1], wave[2][kRadix / kWave];
};
__device__ __forceinline__ void fill_slices(SliceTable& t, int n, const Cut& cut, int ntiles,
                                            const int32_t* __restrict__ off) {
  const int tid = threadIdx.x;
  if (tid < kRadix) t.start[tid] = off[(int64_t)tid * ntiles];  // first position of bin tid
  if (tid == 0) t.start[kRadix] = n;
  __syncthreads();
  const int entries = tid < kRadix ? t.start[tid + 1] - t.start[tid] : 0;
  const bool uneven = __syncthreads_or(entries > cut.even);
  const int cnt = uneven ? (entries + cut.slice - 1) / cut.slice : entries > 0;
  const int many = cnt > 1 ? cnt : 0;
  int a = wave_inclusive_sum(cnt), b = wave_inclusive_sum(many);
  if (lane_id() == kWave - 1 && tid < kRadix) {
    t.wave[0][wave_id()] = a;
    t.wave[1][wave_id()] = b;
  }
  __syncthreads();
  if (tid < kRadix) {
    for (int u = 0; u < wave_id(); ++u) {
      a += t.wave[0][u];
      b += t.wave[1][u];
    }
    t.first[tid] = a - cnt;
    t.wide[tid] = b - many;
    if (tid == kRadix - 1) {
      t.first[kRadix] = a;
      t.wide[kRadix] = b;
    }
  }
  __syncthreads();
}

template <typename T>
struct BinRows {
  // at most 128 KB of the CU's 160 KB LDS: with 256 bins every matrix of up to 4M (fp64) or 8M
  // (fp32) rows has a single sub-range, so each binned entry is read exactly once
  static constexpr int value = 131072 / sizeof(T);
};

constexpr int kAccBlock = 1024;  // one workgroup streams a whole slice: it needs many loads in flight

template <typename T>
__global__ __launch_bounds__(kAccBlock) void bin_accumulate_kernel(
    int n, const Cut cut, const StretchDigit digit, int ntiles, int nsub, const int32_t* __restrict__ off,
    const int32_t* __restrict__ brow, const T* __restrict__ bprod, int nrows, int scratch_rows, T* __restrict__ y,
    T* __restrict__ scratch) {
  constexpr int RB = BinRows<T>::value;
  extern __shared__ __attribute__((aligned(16))) char s_dyn[];  // fp64 LDS atomics need 8-byte addresses
  T* s_acc = reinterpret_cast<T*>(s_dyn);
  __shared__ SliceTable t;
  const int tid = threadIdx.x;
  const int item = blockIdx.x / nsub, sub = blockIdx.x % nsub;

  fill_slices(t, n, cut, ntiles, off);
  if (item >= t.first[kRadix]) return;  // uniform: the grid is an upper bound on the item count
  int b = 0;  // the bin whose slice range contains item (every thread searches, 8 steps)
  for (int step = kRadix / 2; step > 0; step >>= 1)
    if (t.first[b + step] <= item) b += step;
  const int k = item - t.first[b];
  const bool whole_bin = t.first[b + 1] - t.first[b] == 1;
  const int begin = t.start[b] + k * cut.slice;
  const int len = whole_bin ? t.start[b + 1] - begin : min(cut.slice, t.start[b + 1] - begin);
  // from here on entries are counted from the slice's first: the pipeline looks up to 23 551 entries past its
  // end, and the last slice may end that close to 2^31
  brow += begin;
  bprod += begin;
  const int64_t r0 = digit.first(b) + (int64_t)sub * RB;  // first row of this sub-range
  const int nr = (int)max<int64_t>(0, min<int64_t>(RB, digit.first(b + 1) - r0));

  for (int q = tid; q < nr; q += kAccBlock) s_acc[q] = T(0);
  __syncthreads();
  // software pipeline: the loads of batch i+1 are in flight while batch i is accumulated (no load
  // behind a branch: those beyond the end re-read the last entry and are not added)
  constexpr int U = 8;
  int32_t r[2][U];
  T v[2][U];
  const auto load = [&](int p0, int32_t (&rr)[U], T (&vv)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = min(p0 + u * kAccBlock, len - 1);
      rr[u] = ld_nt(brow + p);
      vv[u] = ld_nt(bprod + p);
    }
  };
  const auto add = [&](int p0, const int32_t (&rr)[U], const T (&vv)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t q = static_cast<uint32_t>(rr[u] - static_cast<int>(r0));
      if (p0 + u * kAccBlock < len && q < static_cast<uint32_t>(nr)) atomicAdd(&s_acc[q], vv[u]);
    }
  };
  constexpr int kStep = U * kAccBlock;
  if (len > 0) load(tid, r[0], v[0]);
  for (int p0 = tid; p0 - tid < len; p0 += 2 * kStep) {
    load(p0 + kStep, r[1], v[1]);
    add(p0, r[0], v[0]);
    load(p0 + 2 * kStep, r[0], v[0]);
    add(p0 + kStep, r[1], v[1]);
  }
  __syncthreads();
  T* out = whole_bin ? y + r0 : scratch + (int64_t)(t.wide[b] + k) * scratch_rows + (int64_t)sub * RB;
  for (int q = tid; q < nr && r0 + q < nrows; q += kAccBlock) out[q] = s_acc[q];
}

// The rows of bins without entries and of bins with several slices.
constexpr int kReduceParts = 8;  // workgroups per bin
template <typename T>
__global__ __launch_bounds__(kBlock) void bin_reduce_kernel(int n, const Cut cut, const StretchDigit digit, int ntiles,
                                                            const int32_t* __restrict__ off, int nrows,
                                                            int scratch_rows, const T* __restrict__ scratch,
                                                            T* __restrict__ y) {
  __shared__ SliceTable t;
  fill_slices(t, n, cut, ntiles, off);
  const int b = blockIdx.x / kReduceParts, part = blockIdx.x % kReduceParts;
  const int slices = t.first[b + 1] - t.first[b];
  if (slices == 1) return;
  const int64_t r0 = digit.first(b);
  const int64_t r1 = min<int64_t>(digit.first(b + 1), nrows);
  const T* in = scratch + (int64_t)t.wide[b] * scratch_rows;
  for (int64_t r = r0 + part * kBlock + threadIdx.x; r < r1; r += kReduceParts * kBlock) {
    T sum = 0;
#pragma unroll 4
    for (int k = 0; k < slices; ++k) sum += in[(int64_t)k * scratch_rows + (r - r0)];
    y[r] = sum;
  }
}

struct BinPlan {
  int ntiles, nsub, scratch_rows;
  Cut cut;
  size_t scratch, total;  // scratch: values
};

template <typename T>
static BinPlan bin_plan(int64_t nnz, int64_t nrows) {
  BinPlan P;
  P.ntiles = (int)((nnz + kSortTile - 1) / kSortTile);
  const int64_t rows_in_bin = StretchDigit(nrows).most();
  P.nsub = (int)((rows_in_bin + BinRows<T>::value - 1) / BinRows<T>::value);
  P.cut = Cut(nnz, rows_in_bin);
  P.scratch_rows = (int)rows_in_bin;
  // a bin of S > 1 slices holds more than (S - 1) slices of entries: at most 2 nnz / slice such slices
  P.scratch = (size_t)(2 * (nnz / P.cut.slice) + 2) * rows_in_bin;
  P.total = align_up((size_t)nnz * 4, 256) + align_up((size_t)nnz * sizeof(T), 256) +
            align_up(P.scratch * sizeof(T), 256) +
            align_up((size_t)kRadix * P.ntiles * 4, 256) + scan_workspace((int64_t)kRadix * P.ntiles) +
            256;
  return P;
}

size_t coo_binned_workspace(int dtype, int64_t nnz, int64_t nrows) {
  return dtype == SPT_F64 ? bin_plan<double>(nnz, nrows).total : bin_plan<float>(nnz, nrows).total;
}

template <typename T>
spt_status coo_binned_spmv(int64_t nnz64, int64_t nrows, const int32_t* row, const int32_t* col,
                           const T* vals, const T* x, T* y, void* ws, size_t ws_bytes,
                           hipStream_t s) {
  if (nnz64 + kSortTile >= INT32_MAX || nrows + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries or rows");
  const int nnz = (int)nnz64;
  const BinPlan P = bin_plan<T>(nnz, nrows);
  if (!ws || ws_bytes < P.total)
    return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", P.total,
                ws_bytes);
  Workspace W(ws, ws_bytes);
  int32_t* brow = W.take<int32_t>(nnz);
  T* bprod = W.take<T>(nnz);
  T* scratch = W.take<T>(P.scratch);
  int32_t* hist = W.take<int32_t>((size_t)kRadix * P.ntiles);
  int32_t* scan_tmp = reinterpret_cast<int32_t*>(W.take<char>(scan_workspace((int64_t)kRadix * P.ntiles)));

  const StretchDigit digit(nrows);
  spt_status st = launch_radix_hist(row, nnz, digit, P.ntiles, hist, s);
  if (st != SPT_OK) return st;
  st = device_scan_i32<false>(hist, hist, (int64_t)kRadix * P.ntiles, scan_tmp, s);
  if (st != SPT_OK) return st;
  hipLaunchKernelGGL(bin_scatter_kernel<T>, dim3(P.ntiles), dim3(kBlock), 0, s, nnz, digit,
                     P.ntiles, hist, row, col, vals, x, brow, bprod);
  SPT_CHECK_LAUNCH("bin_scatter");
  const int64_t items = (nnz64 + P.cut.slice - 1) / P.cut.slice + kRadix;  // upper bound
  const size_t lds = (size_t)std::min<int64_t>(P.scratch_rows, BinRows<T>::value) * sizeof(T);
  hipLaunchKernelGGL(bin_accumulate_kernel<T>, dim3((unsigned)(items * P.nsub)), dim3(kAccBlock), lds, s,
                     nnz, P.cut, digit, P.ntiles, P.nsub, hist, brow, bprod, (int)nrows, P.scratch_rows, y, scratch);
  SPT_CHECK_LAUNCH("bin_accumulate");
  hipLaunchKernelGGL(bin_reduce_kernel<T>, dim3(kRadix * kReduceParts), dim3(kBlock), 0, s, nnz, P.cut, digit,
                     P.ntiles, hist, (int)nrows, P.scratch_rows, scratch, y);
  SPT_CHECK_LAUNCH("bin_reduce");
  return SPT_OK;
}

template spt_status coo_binned_spmv<double>(int64_t, int64_t, const int32_t*, const int32_t*,
                                            const double*, const double*, double*, void*, size_t,
                                            hipStream_t);
template spt_status coo_binned_spmv<float>(int64_t, int64_t, const int32_t*, const int32_t*,
                                           const float*, const float*, float*, void*, size_t,
                                           hipStream_t);

}  // namespace spt
