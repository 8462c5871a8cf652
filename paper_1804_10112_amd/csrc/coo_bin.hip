// SpMV on UNORDERED COO without one global atomic per entry.
//
// The paper's COO kernel is a single fused loop that scatters v*x[j] into y
// (Section 4.5, fusing iterators; Section 5.2.1). A literal GPU version issues
// one floating-point atomic per stored entry at a random address, which the
// memory system serves at only ~15 G atomics/s. Here the scatter is split in
// two coalesced steps:
//   1. tiles: a workgroup takes a tile of up to 16 384 entries, gathers x, and leaves (row, v*x[col]) in place, sorted
//      by bin inside the tile: 256 bins of equally many rows. Where a bin begins in each tile goes to a table.
//   2. accumulate: a workgroup owns a slice of one bin's entries, a stretch of each tile, and a sub-range
//      of the bin's rows that fits LDS (128 KB: usually the whole bin), adds the products
//      with LDS atomics and stores its rows: to y when it holds the whole bin, otherwise
//      to scratch, from where a last kernel adds up the slices of each bin.
// Sorting inside the tile instead of over all entries needs no histogram, no scan of one and no rows read twice; a
// stretch of a bin is 64 entries long on average. 10M entries, power-law rows, fp32: 231 -> 126 us (sorted over all
// entries: histogram and scan 24, scatter 120, accumulate 82, reduce 10; here tiles 72, prefix 5, accumulate 39, reduce 9).
// Like the atomic kernel the result is order-dependent in the last bits
// (tolerance-checked, not bit-reproducible); the ordered COO path is exact-order.
#include <algorithm>

#include "common.hpp"
#include "radix.hpp"
#include "search.hpp"
#include "slices.hpp"
#include "wavescan.hpp"

namespace spt {

constexpr int kTileBlock = 512, kTileVecs = 8, kTileStep = 4 * kTileBlock;  // a thread has up to 8 vectors of 4 entries
constexpr int kTileMost = kTileVecs * kTileStep, kTileLeast = 2 * kTileStep, kTileGrain = 64;
constexpr int kTileLds = 65536;          // bytes: two workgroups share a compute unit
constexpr int kTileRow = kRadix + 1;     // of the table: where each bin begins in the tile, and its end

// Entries buf[0 .. len) to out + from; both are 16-byte aligned.
template <typename E>
__device__ __forceinline__ void store_tile(const E* __restrict__ buf, E* __restrict__ out, int from, int len) {
  constexpr int K = 16 / sizeof(E);
  typedef E V __attribute__((ext_vector_type(K)));
  for (int q = threadIdx.x * K; q < len; q += kTileBlock * K) {
    if (q + K <= len) *reinterpret_cast<V*>(out + from + q) = *reinterpret_cast<const V*>(buf + q);
    else
      for (int e = q; e < len; ++e) out[from + e] = buf[e];
  }
}

// R: a row within its bin, 16 bits where they do. V: vectors of a thread. Places inside the tile come from LDS
// counters (0.2 clocks a lane, against the eight ballots per entry that a stable order takes). Entries that meet in one
// counter wait for each other there, and in the sums of step 2, still less than sorting over all entries took (10M
// entries, fp32, sorted so / this way: random order 203 / 105 us, in order of rows 203 / 120, half of them in one row 300 /
// 200, all 323 / 267; fp64 194 / 151, 203 / 166, 283 / 244, 341 / 318; 1.6M fp32 62 / 36, 64 / 34, 81 / 55, 83 / 56).
// Bound by the gathers of x, 200 G/s where an L2 holds x (10M entries, fp32: 50 of 72 us), and by the phases of a tile
// that wait for each other: rows, columns and values on their way early are what the registers allow.
// SLICED: x beyond an L2 is gathered slice by slice (slices.hpp).
template <typename T, typename R, int V, bool SLICED>
__global__ __launch_bounds__(kTileBlock, 4) void bin_tile_kernel(
    int n, const StretchDigit digit, int tile, const int32_t* __restrict__ row, const int32_t* __restrict__ col,
    const T* __restrict__ vals, const T* __restrict__ x, int nslices, int slice, R* __restrict__ brow,
    T* __restrict__ bprod, uint16_t* __restrict__ table) {
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  constexpr int E = 4 * V;
  __shared__ __attribute__((aligned(16))) char s_buf[kTileLds];
  __shared__ int s_cnt[kRadix], s_first[kRadix], s_wave[kRadix / kWave];
  const int tid = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * tile;
  const int len = static_cast<int>(min<int64_t>(tile, n - base));
  row += base;
  col += base;
  vals += base;
  brow += base;
  bprod += base;
  for (int q = tid; q < kRadix; q += kTileBlock) {
    s_cnt[q] = 0;
    s_first[q] = static_cast<int>(digit.first(q));
  }
  // rows and columns are on their way together, and the gathers while the rows are placed (barriers that order LDS only)
  int32_t r[E];
  uint32_t at[E];
  T got[E];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const int p = j * kTileStep + tid * 4;
    if (p + 4 <= len) {
      const I4 v = __builtin_nontemporal_load(reinterpret_cast<const I4*>(row + p));
#pragma unroll
      for (int q = 0; q < 4; ++q) r[4 * j + q] = v[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) r[4 * j + q] = p + q < len ? row[p + q] : -1;
    }
  }
  const auto load_columns = [&] {
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int p = j * kTileStep + tid * 4;
      if (p + 4 <= len) {
        const I4 c = __builtin_nontemporal_load(reinterpret_cast<const I4*>(col + p));
#pragma unroll
        for (int q = 0; q < 4; ++q) at[4 * j + q] = static_cast<uint32_t>(c[q]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) at[4 * j + q] = p + q < len ? static_cast<uint32_t>(col[p + q]) : 0xFFFFFFFFu;
      }
    }
  };
  constexpr bool kAhead = !SLICED && V * sizeof(T) <= 8 * 4;  // (beyond, there are no registers for it)
  if (kAhead) load_columns();
  lds_barrier();
  uint32_t slot[E / 2];  // two places in the tile
#pragma unroll
  for (int k = 0; k < E; k += 2) {
    const int a = r[k] >= 0 ? atomicAdd(&s_cnt[digit.of(r[k])], 1) : 0;
    const int b = r[k + 1] >= 0 ? atomicAdd(&s_cnt[digit.of(r[k + 1])], 1) : 0;
    slot[k / 2] = static_cast<uint32_t>(a) | static_cast<uint32_t>(b) << 16;
  }
  if (kAhead)
#pragma unroll
    for (int k = 0; k < E; ++k) got[k] = at[k] != 0xFFFFFFFFu ? x[at[k]] : T(0);
  lds_barrier();
  int mine = 0, sum = 0;
  if (tid < kRadix) {
    mine = s_cnt[tid];
    sum = wave_inclusive_sum(mine);
    if (lane_id() == kWave - 1) s_wave[wave_id()] = sum;
  }
  lds_barrier();
  uint16_t* out = table + static_cast<int64_t>(blockIdx.x) * kTileRow;
  if (tid < kRadix) {
    for (int u = 0; u < wave_id(); ++u) sum += s_wave[u];
    s_cnt[tid] = sum - mine;
    out[tid] = static_cast<uint16_t>(sum - mine);
  } else if (tid == kRadix) {
    out[kRadix] = static_cast<uint16_t>(len);
  }
  lds_barrier();
  {
    R* buf = reinterpret_cast<R*>(s_buf);
#pragma unroll
    for (int k = 0; k < E; k += 2) {
      const int da = digit.of(r[k]), db = digit.of(r[k + 1]);
      const int a = (slot[k / 2] & 0xFFFF) + (r[k] >= 0 ? s_cnt[da] : 0), b = (slot[k / 2] >> 16) + (r[k + 1] >= 0 ? s_cnt[db] : 0);
      if (r[k] >= 0) buf[a] = static_cast<R>(r[k] - s_first[da]);
      if (r[k + 1] >= 0) buf[b] = static_cast<R>(r[k + 1] - s_first[db]);
      slot[k / 2] = static_cast<uint32_t>(a) | static_cast<uint32_t>(b) << 16;
    }
    lds_barrier();
    store_tile<R>(buf, brow, 0, len);
  }
  if (!kAhead) load_columns();
  if constexpr (SLICED) {
#pragma unroll
    for (int k = 0; k < E; ++k) {
      at[k] = at[k] == 0xFFFFFFFFu ? at[k] : at[k] * sizeof(T);
      got[k] = 0;
    }
    SliceGather<T, E>::run(x, nslices, slice, at, got);
  } else if (!kAhead) {
#pragma unroll
    for (int k = 0; k < E; ++k) got[k] = at[k] != 0xFFFFFFFFu ? x[at[k]] : T(0);
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const int p = j * kTileStep + tid * 4;
    if (p + 4 <= len) {
      const V4 v = __builtin_nontemporal_load(reinterpret_cast<const V4*>(vals + p));
#pragma unroll
      for (int q = 0; q < 4; ++q) got[4 * j + q] *= v[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (p + q < len) got[4 * j + q] *= vals[p + q];
    }
  }
  T* buf = reinterpret_cast<T*>(s_buf);
  constexpr int kPart = kTileLds / sizeof(T);
  for (int part = 0; part < len; part += kPart) {
    lds_barrier();
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int p = (k / 4) * kTileStep + tid * 4 + k % 4;
      const uint32_t q = (slot[k / 2] >> (k % 2 * 16) & 0xFFFF) - part;
      if (p < len && q < static_cast<uint32_t>(kPart)) buf[q] = got[k];
    }
    lds_barrier();
    store_tile<T>(buf, bprod, part, min(len - part, kPart));
  }
}

// prefix[b * ntiles + t] = entries of bin b in the tiles before t; total[b] = in all. A workgroup per bin.
constexpr int kPrefixBlock = 1024;
__global__ __launch_bounds__(kPrefixBlock) void bin_prefix_kernel(int ntiles, const uint16_t* __restrict__ table,
                                                                  int32_t* __restrict__ prefix, int32_t* __restrict__ total) {
  __shared__ int s_wave[2][kPrefixBlock / kWave];
  const int b = blockIdx.x, tid = threadIdx.x;
  int run = 0;
  for (int t0 = 0, turn = 0; t0 < ntiles; t0 += kPrefixBlock, turn ^= 1) {
    const int t = t0 + tid;
    const uint16_t* in = table + static_cast<int64_t>(t) * kTileRow + b;
    const int c = t < ntiles ? in[1] - in[0] : 0;
    int sum = wave_inclusive_sum(c);
    if (lane_id() == kWave - 1) s_wave[turn][wave_id()] = sum;
    __syncthreads();
    int all = 0;
    for (int u = 0; u < kPrefixBlock / kWave; ++u) {
      const int q = s_wave[turn][u];
      if (u < wave_id()) sum += q;
      all += q;
    }
    if (t < ntiles) prefix[static_cast<int64_t>(b) * ntiles + t] = run + sum - c;
    run += all;
  }
  if (tid == 0) total[b] = run;
}

// Work item = (bin b, slice k of the bin's entries, row sub-range sub).
// What counts is that all compute units have equally many entries. Bins of about the same size are one slice each.
// If one holds more than one and a half times the mean (it has long rows), all bins are cut in slices of an eighth of
// the mean, but of no fewer entries than six times the rows of a bin, so that storing and adding up
// the slices' rows costs little next to the entries. Slices of half and of twice that: no faster.
struct Cut {
  int even, slice;  // the largest bin of an even matrix; the longest slice of any other
  Cut() = default;
  Cut(int64_t nnz, int64_t rows_in_bin) {
    even = (int)std::max<int64_t>(nnz / kRadix * 3 / 2, 8192);
    slice = (int)std::max<int64_t>({nnz / (8 * kRadix), 6 * rows_in_bin, 8192});
  }
};

// How the 256 bins are cut: first[b] = slices before bin b, wide[b] = slices of bins
// with more than one slice before bin b (their place in scratch). Every thread of the workgroup
// calls; the result is ready after it.
struct SliceTable {
  int entries[kRadix], first[kRadix + 1], wide[kRadix + 1], wave[2][kRadix / kWave];
};
__device__ __forceinline__ void fill_slices(SliceTable& t, const Cut& cut, const int32_t* __restrict__ total) {
  const int tid = threadIdx.x;
  const int entries = tid < kRadix ? total[tid] : 0;
  if (tid < kRadix) t.entries[tid] = entries;
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

// At most 128 KB of the CU's 160 KB LDS: with 256 bins every matrix of up to 4M rows has a single sub-range, so each
// binned entry is read exactly once. fp32 products are added up in double too: an fp32 add in LDS takes 3.0 clocks a
// lane, one in double 0.36 (0.8 where most lanes meet in a few rows): 10M entries, power law, 82 -> 41 us. Of 4M rows or
// more, fp32 entries are so read twice, once with sums in fp32 (16M entries, x of 2 MB, sorted over all entries with sums in
// fp32 / this way: 3M rows 300 / 164 us, 4.4M 297 / 210, 8M 299 / 209; 40M entries, 8M rows 706 / 454).
constexpr int kBinRows = 131072 / sizeof(double);

constexpr int kAccBlock = 1024;  // one workgroup streams a whole slice: it needs many loads in flight

template <typename T, typename R>
__global__ __launch_bounds__(kAccBlock) void bin_accumulate_kernel(
    const Cut cut, const StretchDigit digit, int tile, int ntiles, int nsub, const uint16_t* __restrict__ table,
    const int32_t* __restrict__ prefix, const int32_t* __restrict__ total, const R* __restrict__ brow,
    const T* __restrict__ bprod, int nrows, int scratch_rows, T* __restrict__ y, T* __restrict__ scratch) {
  extern __shared__ __attribute__((aligned(16))) char s_dyn[];  // fp64 LDS atomics need 8-byte addresses
  double* s_acc = reinterpret_cast<double*>(s_dyn);
  __shared__ SliceTable t;
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  const int item = blockIdx.x / nsub, sub = blockIdx.x % nsub;

  fill_slices(t, cut, total);
  if (item >= t.first[kRadix]) return;  // uniform: the grid is an upper bound on the item count
  int b = 0;  // the bin whose slice range contains item (every thread searches, 8 steps)
  for (int step = kRadix / 2; step > 0; step >>= 1)
    if (t.first[b + step] <= item) b += step;
  b = __builtin_amdgcn_readfirstlane(b);
  const int k = item - t.first[b];
  const bool whole_bin = t.first[b + 1] - t.first[b] == 1;
  const int entries = t.entries[b];
  const int begin = whole_bin ? 0 : k * cut.slice, len = whole_bin ? entries : min(cut.slice, entries - begin);
  const int64_t bin0 = digit.first(b);
  const int sub0 = sub * kBinRows;  // first row of this sub-range in the bin
  const int nr = (int)max<int64_t>(0, min<int64_t>(kBinRows, digit.first(b + 1) - bin0 - sub0));
  for (int q = tid; q < nr; q += kAccBlock) s_acc[q] = 0.0;
  __syncthreads();

  // a wave has a sixteenth of the slice: entries [e0, e1) of the bin, in order of tiles
  constexpr int kWavesOf = kAccBlock / kWave;
  const int e0 = begin + static_cast<int>(static_cast<int64_t>(len) * w / kWavesOf);
  const int e1 = begin + static_cast<int>(static_cast<int64_t>(len) * (w + 1) / kWavesOf);
  const int32_t* pre = prefix + static_cast<int64_t>(b) * ntiles;
  const auto add = [&](bool in, int r, T v) {
    const uint32_t q = static_cast<uint32_t>(r - sub0);
    if (in && q < static_cast<uint32_t>(nr)) atomicAdd(&s_acc[q], static_cast<double>(v));
  };
  if (e0 < e1) {
    int t0 = group_last_true<kWave>(0, ntiles, [&](int q) { return q == 0 || pre[q] <= e0; });
    for (bool more = true; more; t0 += kWave) {
      // a lane looks up where the stretch of one tile lies
      const int tt = t0 + lane;
      int count = 0, at = 0;
      bool ends = true;
      if (tt < ntiles) {
        const int p = pre[tt];
        const uint16_t* in = table + static_cast<int64_t>(tt) * kTileRow + b;
        const int s0 = in[0], size = in[1] - s0;
        const int from = max(e0 - p, 0), to = min(e1 - p, size);
        count = max(to - from, 0);
        at = count > 0 ? tt * tile + s0 + from : 0;
        ends = p + size >= e1;
      }
      more = __ballot(ends) == 0;
      // The stretches in pieces of up to 64 entries, numbered through: lane l's are first .. upto - 1. (What is
      // longer than 64 U loads at a time, whatever its length: 47 instead of 40 us for 10M entries of power-law rows, fp32,
      // and 707 instead of 603 for the whole product of 40M, fp64. Four or eight pieces in flight: 1 % longer.)
      const auto take = [&](int n, const auto& piece_of) {  // piece z: lane src's entries from `from` on
        constexpr int U = 6;
        for (int z = 0; z < n; z += U) {
          int r[U], c[U];
          T v[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            int src, from;
            piece_of(min(z + u, n - 1), src, from);
            c[u] = z + u < n ? __builtin_amdgcn_readlane(count, src) - from : 0;
            const int p = __builtin_amdgcn_readlane(at, src) + from + min(lane, max(c[u] - 1, 0));
            r[u] = brow[p];
            v[u] = bprod[p];
          }
#pragma unroll
          for (int u = 0; u < U; ++u) add(lane < c[u], r[u], v[u]);
        }
      };
      if (__ballot(count > kWave) == 0) {  // lane by lane (1.2M entries, power-law rows, fp32, whole product: numbered through 41.4, 39.8)
        const uint64_t any = __ballot(count > 0);
        take(any ? 64 - __clzll(static_cast<long long>(any)) : 0, [](int z, int& src, int& from) {
          src = z;
          from = 0;
        });
      } else {
        const int upto = wave_inclusive_sum((count + kWave - 1) / kWave), first = upto - (count + kWave - 1) / kWave;
        take(__builtin_amdgcn_readlane(upto, kWave - 1), [&](int z, int& src, int& from) {
          src = __popcll(__ballot(upto <= z));  // uniform
          from = (z - __builtin_amdgcn_readlane(first, src)) * kWave;
        });
      }
    }
  }
  __syncthreads();
  T* out = whole_bin ? y + bin0 + sub0 : scratch + (int64_t)(t.wide[b] + k) * scratch_rows + sub0;
  for (int q = tid; q < nr && bin0 + sub0 + q < nrows; q += kAccBlock) out[q] = static_cast<T>(s_acc[q]);
}

// The rows of bins without entries and of bins with several slices.
constexpr int kReduceParts = 8;  // workgroups per bin
template <typename T>
__global__ __launch_bounds__(kBlock) void bin_reduce_kernel(const Cut cut, const StretchDigit digit,
                                                            const int32_t* __restrict__ total, int nrows,
                                                            int scratch_rows, const T* __restrict__ scratch,
                                                            T* __restrict__ y) {
  __shared__ SliceTable t;
  fill_slices(t, cut, total);
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

// x slice by slice from here on. Unsliced / sliced, uniform columns, us: fp64, 6.4 MB, 1.6M entries 44 / 53, 3.2M 66 / 70,
// 6.4M 111 / 105; 16 MB, 8M 183 / 134; 32 MB, 16M 389 / 273; fp32, 6.4 MB, 3.2M 60 / 59, 6.4M 96 / 86; shuffled
// entries of a banded matrix, fp64, 32 MB, 28M 575 / 407. (30M, fp64, 64 MB, in slices of 3.2 MB 714, of 5.6 627.)
constexpr int64_t kSlicedMinEntries = int64_t(1) << 22;

struct BinPlan {
  int tile, ntiles, nsub, scratch_rows;
  bool wide;  // rows within a bin need more than 16 bits
  Cut cut;
  size_t scratch, total;  // scratch: values
};

// Tiles: as many as fill two workgroups on every compute unit a whole number of times (and not fewer, by whole vectors of
// every thread: 19M entries, fp32, 200 us so, 189).
template <typename T>
static BinPlan bin_plan(int64_t nnz, int64_t nrows) {
  BinPlan P;
  const int64_t slots = 2 * 256, rounds = (nnz + slots * kTileMost - 1) / (slots * kTileMost);
  const int64_t even = (nnz + slots * rounds - 1) / (slots * rounds);
  P.tile = (int)std::max<int64_t>((even + kTileGrain - 1) / kTileGrain * kTileGrain, kTileLeast);
  P.ntiles = (int)((nnz + P.tile - 1) / P.tile);
  const int64_t rows_in_bin = StretchDigit(nrows).most();
  P.wide = rows_in_bin > 65536;
  P.nsub = (int)((rows_in_bin + kBinRows - 1) / kBinRows);
  P.cut = Cut(nnz, rows_in_bin);
  P.scratch_rows = (int)rows_in_bin;
  // a bin of S > 1 slices holds more than (S - 1) slices of entries: fewer than 2 nnz / slice such slices
  P.scratch = (size_t)(2 * (nnz / P.cut.slice) + 1) * rows_in_bin;
  P.total = align_up((size_t)nnz * (P.wide ? 4 : 2), 256) + align_up((size_t)nnz * sizeof(T), 256) + align_up(P.scratch * sizeof(T), 256) +
            align_up((size_t)kTileRow * P.ntiles * 2, 256) + align_up((size_t)kRadix * P.ntiles * 4, 256) + 1024 + 256;
  return P;
}

size_t coo_binned_workspace(int dtype, int64_t nnz, int64_t nrows) {
  return dtype == SPT_F64 ? bin_plan<double>(nnz, nrows).total : bin_plan<float>(nnz, nrows).total;
}

template <typename T, typename R>
static spt_status binned_spmv(int nnz, int64_t nrows, int64_t ncols, const int32_t* row, const int32_t* col, const T* vals,
                              const T* x, T* y, const BinPlan& P, Workspace W, hipStream_t s) {
  R* brow = W.take<R>(nnz);
  T* bprod = W.take<T>(nnz);
  T* scratch = W.take<T>(P.scratch);
  uint16_t* table = W.take<uint16_t>((size_t)kTileRow * P.ntiles);
  int32_t* prefix = W.take<int32_t>((size_t)kRadix * P.ntiles);
  int32_t* total = W.take<int32_t>(kRadix);
  const StretchDigit digit(nrows);
  const int64_t xbytes = ncols * (int64_t)sizeof(T);
  const bool sliced = nnz >= kSlicedMinEntries && xbytes > kSlicesMinX && xbytes <= kSlicesMaxX;
  const int nslices = sliced ? slices_of(ncols, sizeof(T), int64_t(2) * 256 * kTileMost) : 1;
  const int slice = (int)((ncols + nslices - 1) / nslices * sizeof(T));
#define SPT_TILE(V_, SLICED_)                                                                                             \
  hipLaunchKernelGGL((bin_tile_kernel<T, R, V_, SLICED_>), dim3(P.ntiles), dim3(kTileBlock), 0, s, nnz, digit, P.tile, row, col, \
                     vals, x, nslices, slice, brow, bprod, table)
  if (sliced) { SPT_TILE(8, true); }
  else {
    switch ((P.tile + kTileStep - 1) / kTileStep) {
      case 2: SPT_TILE(2, false); break;
      case 3: SPT_TILE(3, false); break;
      case 4: SPT_TILE(4, false); break;
      case 5: SPT_TILE(5, false); break;
      case 6: SPT_TILE(6, false); break;
      default: SPT_TILE(8, false);
    }
  }
#undef SPT_TILE
  SPT_CHECK_LAUNCH("bin_tile");
  hipLaunchKernelGGL(bin_prefix_kernel, dim3(kRadix), dim3(kPrefixBlock), 0, s, P.ntiles, table, prefix, total);
  SPT_CHECK_LAUNCH("bin_prefix");
  const int64_t items = (nnz + (int64_t)P.cut.slice - 1) / P.cut.slice + kRadix;  // upper bound
  const size_t lds = (size_t)std::min<int64_t>(P.scratch_rows, kBinRows) * sizeof(double);
  hipLaunchKernelGGL((bin_accumulate_kernel<T, R>), dim3((unsigned)(items * P.nsub)), dim3(kAccBlock), lds, s, P.cut, digit, P.tile,
                     P.ntiles, P.nsub, table, prefix, total, brow, bprod, (int)nrows, P.scratch_rows, y, scratch);
  SPT_CHECK_LAUNCH("bin_accumulate");
  hipLaunchKernelGGL(bin_reduce_kernel<T>, dim3(kRadix * kReduceParts), dim3(kBlock), 0, s, P.cut, digit, total, (int)nrows,
                     P.scratch_rows, scratch, y);
  SPT_CHECK_LAUNCH("bin_reduce");
  return SPT_OK;
}

template <typename T>
spt_status coo_binned_spmv(int64_t nnz64, int64_t nrows, int64_t ncols, const int32_t* row, const int32_t* col, const T* vals,
                           const T* x, T* y, void* ws, size_t ws_bytes, hipStream_t s) {
  if (nnz64 + kSortTile >= INT32_MAX || nrows + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries or rows");
  const int nnz = (int)nnz64;
  const BinPlan P = bin_plan<T>(nnz, nrows);
  if (!ws || ws_bytes < P.total)
    return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", P.total, ws_bytes);
  const Workspace W(ws, ws_bytes);
  return P.wide ? binned_spmv<T, int32_t>(nnz, nrows, ncols, row, col, vals, x, y, P, W, s)
                : binned_spmv<T, uint16_t>(nnz, nrows, ncols, row, col, vals, x, y, P, W, s);
}

template spt_status coo_binned_spmv<double>(int64_t, int64_t, int64_t, const int32_t*, const int32_t*,
                                            const double*, const double*, double*, void*, size_t,
                                            hipStream_t);
template spt_status coo_binned_spmv<float>(int64_t, int64_t, int64_t, const int32_t*, const int32_t*,
                                           const float*, const float*, float*, void*, size_t,
                                           hipStream_t);

}  // namespace spt
