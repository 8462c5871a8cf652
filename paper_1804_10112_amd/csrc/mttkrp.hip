// MTTKRP A_ij = sum_kl B_ikl C_kj D_lj on ordered COO and on CSF (Section 5.3), gfx950.
//
// A run of consecutive entries with the same i is one row of A (deduplication, Section 4.3). Entries
// are split evenly: a workgroup has a chunk, a group of L lanes `epg` consecutive entries of it, and a
// lane one 16-byte vector of the J columns, so that a load instruction of a wave fetches the factor
// rows of 64 / L entries. A lane holds the coordinates of four entries at a time; they are handed
// around its group, and the eight factor rows of four entries are in flight together (where there are few workgroups, those of eight).
//   - A row that begins and ends inside a group is stored by the group; rows across groups are added
//     up by a segmented scan over the groups; the part of a chunk that continues a row begun before it
//     leaves as a carry (row, J values), which the carry kernels add in a fixed order (no atomics).
//   - CSF: i and k are the last slice and fibre that start at or before an entry. The starts inside a
//     chunk are marked in a bit set in LDS, where a group sees which of its entries begin one; only those look up k or i.
//     C[k, :] is multiplied once per fibre (factored form).
//   - Rows of factors up to 4 GiB are found at 32-bit offsets, and CSF parks a group's first sum in LDS: with the registers
//     that are left, five waves share a SIMD instead of four (i, k and 64-bit addresses in registers): 11M entries in CSF, fp32, J = 32,
//     skewed 158 -> 132 us, even 189 -> 174; fp64 262 -> 215, 386 -> 383; 2.6M, fp32, J = 8 34.2 -> 30.5; factors of 51 MB, whose
//     rows miss L2 whatever is in flight, 748 -> 755. COO, fp64, has four: with five, 16M even entries, J = 8, take 188 instead of 171. So has CSF, fp64,
//     with factors beyond 4 GiB (with five, two to five registers go through scratch memory: 3M entries, J = 64 433 us, 411 with four).
// Bound by the gathers of factor rows, large tensors by those that miss L2: what is fetched from beyond it takes all the
// time there (50M entries, J = 32, fp32: 4.7 GB, 632 us; with all rows in L2, as a probe, 400; chunks in the order of their
// rows of C: 593). A row of C stays in registers while k does (loaded for every entry: 700 us, and 619
// instead of 521 with a D that fits L2; same sums, bit for bit). Chunks go to the
// XCDs in turn, unless they are ordered: with one contiguous part of a skewed tensor to each, the XCD with its last slices fetched twice as
// many lines as the others and took 960 us (738 000 entries in CSF, J = 16, fp64: 41 -> 38; 15M entries, J = 32,
// fp64, 703 -> 555; runs of 4 or 16 chunks the same; even tensors of 0.4 to 0.9M entries lose 3 %, 22.2 -> 22.9). Left out after measuring: C read past the caches (small tensors
// take up to a third longer); half of D to every other XCD, each going through all entries (743 us: the streams are
// read twice), or picking its entries into a list in LDS first (3.0 instead of 4.7 GB, but 684 us: to pick takes 150, to go
// through a list 230 without any row of a factor); chunks of twice the entries (1 % faster, fp64 CSF 2 % slower); six waves a SIMD (spills, 815). Before that: more or
// fewer waves and the next rows loaded ahead change nothing; 32 lanes of one column per
// entry, which issue four times as many loads and hand-arounds, and longer walks per group take 12 % longer, and for
// 738 000 entries twice as long.
#include <algorithm>

#include "common.hpp"
#include "mttkrp_plan.hpp"
#include "radix.hpp"
#include "search.hpp"
#include "wavescan.hpp"

namespace spt {

template <typename T, int V>
struct ColVec {
  typedef T type __attribute__((ext_vector_type(V), aligned(sizeof(T))));
};
template <typename T>
struct ColVec<T, 1> {
  typedef T type;
};
template <typename T, int V>
__device__ __forceinline__ void load_cols(const T* p, T (&x)[V]) {
  const typename ColVec<T, V>::type v = *reinterpret_cast<const typename ColVec<T, V>::type*>(p);
  if constexpr (V == 1) {
    x[0] = v;
  } else {
#pragma unroll
    for (int q = 0; q < V; ++q) x[q] = v[q];
  }
}
template <typename T, int V>
__device__ __forceinline__ void store_cols(T* p, const T (&x)[V]) {
  typename ColVec<T, V>::type v;
  if constexpr (V == 1) {
    v = x[0];
  } else {
#pragma unroll
    for (int q = 0; q < V; ++q) v[q] = x[q];
  }
  *reinterpret_cast<typename ColVec<T, V>::type*>(p) = v;
}

// Row k from column col on. NEAR: at an offset of 32 bits, which takes one register instead of two.
template <bool NEAR, typename T>
__device__ __forceinline__ const T* row_at(const T* p, int k, int J, int col) {
  if constexpr (NEAR)
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + (static_cast<uint32_t>(k) * static_cast<uint32_t>(J * sizeof(T)) + static_cast<uint32_t>(col * sizeof(T))));
  else
    return p + static_cast<int64_t>(k) * J + col;
}

// Four consecutive values from p + e on, those at `end` and beyond as zero.
template <typename E>
__device__ __forceinline__ void load_four(const E* __restrict__ p, int e, int end, E (&x)[4]) {
  typedef E V4 __attribute__((ext_vector_type(4), aligned(sizeof(E))));
  if (e + 4 <= end) {
    const V4 v = __builtin_nontemporal_load(reinterpret_cast<const V4*>(p + e));
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = v[r];
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = e + r < end ? p[e + r] : E(0);
  }
}

// Value of lane addr / 4, through the LDS crossbar.
__device__ __forceinline__ int32_t from_lane(int addr, int32_t v) { return __builtin_amdgcn_ds_bpermute(addr, v); }
__device__ __forceinline__ float from_lane(int addr, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double from_lane(int addr, double v) {
  const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
  const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
  return __hiloint2double(hi, lo);
}

// The upper levels of a CSF tensor; bounds as made by mttkrp_prepare_kernel.
struct CsfLevels {
  const int32_t *crd0, *pos1, *crd1, *pos2, *bounds;
  int nslices, nfibres;
};

// ---- the order of the chunks -----------------------------------------------------------------
// Chunks are sorted by the row of C that one of their entries needs, by kRadix equal stretches of the rows, and each XCD
// has an eighth of them in this order: chunks of different slices that need the same rows of C meet on one XCD, whose L2
// then has them (C and D 10.2 and 6.4 MB, 50M entries of skewed slices: the rows 632 -> 593 us; 20M of even ones 527 -> 345).
// The order changes no result: a chunk's sums and carries have their places. bin_chunks notes for each chunk its bin and
// its place among the chunks of the same bin in its workgroup's share, and the share's counts; mttkrp_order_kernel makes
// the order of that (4.5 us; by one workgroup 90). Both stable.
constexpr int kOrderShare = 4 * kBlock;  // chunks of a workgroup
template <class KEY>
__device__ __forceinline__ void bin_chunks(int share, int nchunks, const StretchDigit& digit, const KEY& row_of,
                                           int32_t* __restrict__ noted, int32_t* __restrict__ hist) {
  __shared__ int s_cnt[kBlock / kWave][kRadix], s_before[kBlock / kWave][kRadix];
  const int tid = threadIdx.x, w = wave_id(), lane = lane_id();
  constexpr int kOwn = kOrderShare / kBlock;
  for (int q = tid; q < kBlock / kWave * kRadix; q += kBlock) (&s_cnt[0][0])[q] = 0;
  int d[kOwn], rank[kOwn];
  const int first = share * kOrderShare + w * kOwn * kWave + lane;
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    d[k] = static_cast<int>(min(static_cast<uint32_t>(digit.of(row_of(min(first + k * kWave, nchunks - 1)))), kRadix - 1u));
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    const bool valid = first + k * kWave < nchunks;
    const uint64_t same = lanes_with(d[k], __ballot(valid));
    const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(same >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(same), 0));
    rank[k] = s_cnt[w][d[k]] + before;
    wave_lds_order();
    if (valid && before == 0) s_cnt[w][d[k]] = rank[k] + __popcll(same);
    wave_lds_order();
  }
  __syncthreads();
  int run = 0;
#pragma unroll
  for (int u = 0; u < kBlock / kWave; ++u) {
    s_before[u][tid] = run;
    run += s_cnt[u][tid];
  }
  hist[share * kRadix + tid] = run;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    if (first + k * kWave < nchunks) noted[first + k * kWave] = d[k] << 16 | (s_before[w][d[k]] + rank[k]);
}
// COO: the row of a chunk's middle entry; CSF: of the first fibre that starts in or after the chunk.
template <bool CSF>
__global__ __launch_bounds__(kBlock) void mttkrp_bin_kernel(int n, int chunk, int nchunks, const StretchDigit digit,
                                                            const int32_t* __restrict__ ck, const CsfLevels csf,
                                                            int32_t* __restrict__ noted, int32_t* __restrict__ hist) {
  bin_chunks(blockIdx.x, nchunks, digit, [&](int c) {
    if (CSF) return csf.crd1[min(csf.bounds[3 * c], csf.nfibres - 1)];
    return ck[min(static_cast<int64_t>(c) * chunk + chunk / 2, static_cast<int64_t>(n) - 1)];
  }, noted, hist);
}
__global__ __launch_bounds__(kBlock) void mttkrp_order_kernel(int nchunks, const int32_t* __restrict__ noted,
                                                              const int32_t* __restrict__ hist, int32_t* __restrict__ bounds) {
  static_assert(kRadix == kBlock, "");
  __shared__ int s_start[kRadix];
  __shared__ int s_sum[kBlock / kWave];
  const int tid = threadIdx.x, share = blockIdx.x, shares = gridDim.x;
  constexpr int kOwn = kOrderShare / kBlock, kAtOnce = 32;
  int x[kOwn];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) x[k] = noted[min(share * kOrderShare + k * kBlock + tid, nchunks - 1)];
  int before = 0, total = 0;
  for (int q0 = 0; q0 < shares; q0 += kAtOnce) {
    int cnt[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) cnt[q] = hist[min(q0 + q, shares - 1) * kRadix + tid];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      before += q0 + q < share ? cnt[q] : 0;
      total += q0 + q < shares ? cnt[q] : 0;
    }
  }
  int start = wave_inclusive_sum(total);
  if (lane_id() == kWave - 1) s_sum[wave_id()] = start;
  __syncthreads();
  for (int u = 0; u < wave_id(); ++u) start += s_sum[u];
  s_start[tid] = start - total + before;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    const int c = share * kOrderShare + k * kBlock + tid;
    if (c < nchunks) bounds[3 * (s_start[x[k] >> 16] + (x[k] & 0xFFFF)) + 2] = c;
  }
}

// Zeroes A (rows without entries stay zero). CSF: for chunk boundary c (entries from c * chunk on),
// bounds[3c] = first fibre that starts at or after it, bounds[3c+1] = first slice that starts at or
// after that fibre (as the end of a chunk: all slices once the fibres are used up). Boundary nchunks is the end. LANES
// lanes search a boundary: a wave while there are few (a chain of six loads instead of ten), else eight lanes.
// (bounds[3c+2]: the order of the chunks.)
constexpr int kWideSearch = 4096;
template <typename T, int LANES>
__global__ __launch_bounds__(kBlock) void mttkrp_prepare_kernel(T* __restrict__ A, int64_t size, int fill_blocks,
                                                                int nchunks, int chunk, int nslices, int nfibres,
                                                                const int32_t* __restrict__ pos1,
                                                                const int32_t* __restrict__ pos2,
                                                                int32_t* __restrict__ bounds) {
  if (static_cast<int>(blockIdx.x) < fill_blocks) {
    typedef T V __attribute__((ext_vector_type(kVec<T>), aligned(sizeof(T))));
    const int64_t e = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) * kVec<T>;
    if (e + kVec<T> <= size) *reinterpret_cast<V*>(A + e) = V(T(0));
    else
      for (int64_t q = e; q < size; ++q) A[q] = T(0);
    return;
  }
  const int c = ((blockIdx.x - fill_blocks) * kBlock + threadIdx.x) / LANES;
  if (c > nchunks) return;
  int f = nfibres;
  if (c < nchunks) {
    const int target = c * chunk;
    f = group_last_true<LANES>(0, static_cast<int64_t>(nfibres) + 2, [&](int q) { return q == 0 || pos2[q - 1] < target; });
  }
  const int sl = group_last_true<LANES>(0, static_cast<int64_t>(nslices) + 2, [&](int q) { return q == 0 || pos1[q - 1] < f; });
  if (threadIdx.x % LANES == 0) {
    bounds[3 * c] = f;
    bounds[3 * c + 1] = sl;
  }
}

// Position of the last marked entry at or before entry e; before[w] = last marked entry before word w.
__device__ __forceinline__ int last_mark(const uint32_t* marks, const int16_t* before, int e) {
  const int w = e >> 5;
  const uint32_t m = marks[w] & ((2u << (e & 31)) - 1);
  return m ? w * 32 + 31 - __clz(m) : before[w];
}

// before[] of `words` words, by one wave. Entry 0 is marked.
__device__ __forceinline__ void marks_before(const uint32_t* marks, int16_t* before, int words) {
  int from = 0;
  for (int w0 = 0; w0 < words; w0 += kWave) {
    const int w = w0 + lane_id();
    const uint32_t m = w < words ? marks[w] : 0;
    const uint64_t any = __ballot(m != 0), below = any & ((uint64_t{1} << lane_id()) - 1);
    const int at = m ? w * 32 + 31 - __clz(m) : 0;
    const int prev = __shfl(at, below ? 63 - __clzll(static_cast<long long>(below)) : 0);
    if (w < words) before[w] = static_cast<int16_t>(below ? prev : from);
    if (any) from = __shfl(at, 63 - __clzll(static_cast<long long>(any)));
  }
}

// PLACED: chunks and columns as `placing` says; else chunk blockIdx.x, and all columns. U: the rows of 4 * U entries are in flight
// together. NEAR: no factor has more than 4 GiB.
template <typename T, int L, int V, bool CSF, bool PLACED, int U = 1, bool NEAR = true>
__global__ __launch_bounds__(kBlock, CSF && U == 1 && NEAR ? 5 : 1) void mttkrp_rows_kernel(int n, int J, int epg, const Placing placing, const int32_t* __restrict__ ci,
                                                             const int32_t* __restrict__ ck,
                                                             const int32_t* __restrict__ cl,
                                                             const T* __restrict__ vals, const T* __restrict__ Cm,
                                                             const T* __restrict__ Dm, const CsfLevels csf,
                                                             T* __restrict__ A, int32_t* __restrict__ carry_key,
                                                             T* __restrict__ carry_vec, const int32_t* __restrict__ bounds) {
  constexpr int NG = kBlock / L, kGroupsOfWave = kWave / L;
  extern __shared__ __attribute__((aligned(16))) int32_t s_csf[];
  __shared__ T s_v[kBlock / kWave][L][V];
  __shared__ int s_f[kBlock / kWave];
  __shared__ T s_lead[CSF ? kBlock : 1][V];  // (CSF: the registers that this takes would leave a wave less)
  __shared__ int s_slice_first;  // the chunk starts with a slice
  const int tid = threadIdx.x, lane = lane_id();
  const int g = tid / L, gl = tid % L;
  // (in turn to the XCDs: in one piece, the last has the slices of few entries, whose rows of C nobody shares)
  int chunk = blockIdx.x, part = 0, cols = J;
  if (PLACED) {
    const int xcd = blockIdx.x % kXcds, turn = blockIdx.x / kXcds, of = kXcds / placing.parts, at = xcd / placing.parts;
    const int q = placing.nchunks / of, rem = placing.nchunks % of;
    if (turn >= q + (at < rem)) return;
    chunk = placing.ordered ? bounds[3 * (at * q + min(at, rem) + turn) + 2] : turn * of + at;
    part = xcd % placing.parts;
    cols = placing.cols;
  }
  const int size = NG * epg;
  const int base = chunk * size, end = min(base + size, n);
  bool jok;
  const int col = column_of(cols, V, part, blockIdx.y * L + gl, &jok);
  const bool keeps_keys = gl == 0 && blockIdx.y == 0 && part == 0;

  const int g0 = base + g * epg, g1 = min(g0 + epg, end);
  // rows of D and values of the first batch: on their way while the bounds are found (738 000 entries in CSF, J = 16, fp64:
  // 33.8 us without, 32.0 also by the wider search; large ordered tensors lose 2 %)
  int32_t rl[4];
  T rv[4];
  constexpr bool kEarly = CSF && !PLACED;
  if (kEarly && g0 < g1) {
    load_four(cl, g0 + 4 * gl, g1, rl);
    load_four(vals, g0 + 4 * gl, g1, rv);
  }
  int32_t *s_k = s_csf, *s_i = s_csf + size;
  uint32_t *s_fibre = reinterpret_cast<uint32_t*>(s_i + size), *s_slice = s_fibre + (size + 31) / 32;
  int16_t *s_fibre_before = reinterpret_cast<int16_t*>(s_slice + (size + 31) / 32), *s_slice_before = s_fibre_before + (size + 31) / 32;
  if (CSF) {
    const int f_lo = csf.bounds[3 * chunk], f_hi = csf.bounds[3 * chunk + 3];
    const int s_lo = csf.bounds[3 * chunk + 1], s_hi = f_hi >= csf.nfibres ? csf.nslices : csf.bounds[3 * chunk + 4];
    int32_t cut_k = -1, cut_i = -1;  // of the fibre and the slice that the chunk's start cuts
    if (tid == 0) {
      if (f_lo > 0) cut_k = csf.crd1[f_lo - 1];
      if (s_lo > 0) cut_i = csf.crd0[s_lo - 1];
    }
    for (int w = tid; w < 2 * ((size + 31) / 32); w += kBlock) s_fibre[w] = 0;
    __syncthreads();
    strided(f_lo, f_hi, tid, kBlock, [&](int f) {
      const int a = csf.pos2[f], b = csf.pos2[f + 1], k = csf.crd1[f];
      if (b > a) {
        s_k[a - base] = k;
        atomicOr(&s_fibre[(a - base) >> 5], 1u << ((a - base) & 31));
      }
    });
    // a slice is marked at its first stored entry, whichever of its fibres holds it (a
    // compressed level may hold empty segments: leading fibres of a slice can be empty)
    strided(s_lo, s_hi, tid, kBlock, [&](int sl) {
      const int a = csf.pos2[csf.pos1[sl]], b = csf.pos2[csf.pos1[sl + 1]];
      if (b > a && a < end) {
        s_i[a - base] = csf.crd0[sl];
        atomicOr(&s_slice[(a - base) >> 5], 1u << ((a - base) & 31));
      }
    });
    __syncthreads();
    if (tid == 0) {
      s_slice_first = s_slice[0] & 1;
      if (!(s_fibre[0] & 1)) {
        s_k[0] = cut_k;
        s_fibre[0] |= 1;
      }
      if (!(s_slice[0] & 1)) {
        s_i[0] = cut_i;
        s_slice[0] |= 1;
      }
    }
    __syncthreads();
    if (wave_id() == 0) marks_before(s_fibre, s_fibre_before, (size + 31) / 32);
    if (wave_id() == 1) marks_before(s_slice, s_slice_before, (size + 31) / 32);
    __syncthreads();
  }

  T acc[V], lead[V], t[V], c_cur[V];
#pragma unroll
  for (int q = 0; q < V; ++q) acc[q] = lead[q] = t[q] = c_cur[q] = T(0);
  bool has_head = false;
  int first_close = -1, cur_k = -1;
  // the row of the entry before this group's first (-1: there is none; -2: a different one)
  int cur;
  if (!CSF) cur = g0 >= end ? ci[end - 1] : g0 > 0 ? ci[g0 - 1] : -1;
  else if (g0 >= end) cur = s_i[last_mark(s_slice, s_slice_before, end - 1 - base)];
  else if (g0 > base) cur = s_i[last_mark(s_slice, s_slice_before, g0 - 1 - base)];
  else cur = base == 0 ? -1 : s_slice_first ? -2 : s_i[0];

  // CSF: fibre and row of the group's first entry; of the others, the marks tell where a new one starts
  int first_k = 0, first_i = 0;
  if (CSF && g0 < g1) {
    first_k = s_k[last_mark(s_fibre, s_fibre_before, g0 - base)];
    first_i = s_i[last_mark(s_slice, s_slice_before, g0 - base)];
  }
  for (int b0 = g0; b0 < g1; b0 += 4 * L) {
    int32_t ri[4], rk[4];
    const int p = b0 + 4 * gl;
    if (!kEarly || b0 > g0) {
      load_four(cl, p, g1, rl);
      load_four(vals, p, g1, rv);
    }
    if (!CSF) {
      load_four(ci, p, g1, ri);
      load_four(ck, p, g1, rk);
    }
    const int batch = min(4 * L, g1 - b0);
    static_assert(L % U == 0, "");
    for (int q = 0; 4 * q < batch; q += U) {
      const int e = b0 + 4 * q - base;  // (a multiple of 4 * U: one word has the marks)
      const bool at_first = CSF && e == g0 - base;
      uint32_t new_fibre = 0, new_row = 0;
      int i[4 * U], k[4 * U];
      T v[4 * U], c[4 * U][V], d[4 * U][V];
      bool fresh[4 * U];
      if (CSF) {
        new_fibre = s_fibre[e >> 5] >> (e & 31) | at_first;
        new_row = s_slice[e >> 5] >> (e & 31) | at_first;
#pragma unroll
        for (int r = 0; r < 4 * U; ++r) k[r] = s_k[e + r];
        if (at_first) k[0] = first_k;
      }
#pragma unroll
      for (int r = 0; r < 4 * U; ++r) {
        const int addr = 4 * ((lane & ~(L - 1)) + q + r / 4);
        const int l = from_lane(addr, rl[r % 4]);
        v[r] = from_lane(addr, rv[r % 4]);
        // a row of C is loaded for the first entry that it belongs to
        if (CSF) {
          fresh[r] = new_fibre >> r & 1;
        } else {
          i[r] = from_lane(addr, ri[r % 4]);
          k[r] = from_lane(addr, rk[r % 4]);
          fresh[r] = k[r] != (r ? k[r - 1] : cur_k);
        }
        if (fresh[r]) load_cols<T, V>(row_at<NEAR>(Cm, k[r], J, col), c[r]);
        load_cols<T, V>(row_at<NEAR>(Dm, l, J, col), d[r]);
      }
#pragma unroll
      for (int r = 0; r < 4 * U; ++r) {
        if (4 * q + r < batch) {
          if (!CSF) {
#pragma unroll
            for (int x = 0; x < V; ++x) c_cur[x] = fresh[r] ? c[r][x] : c_cur[x];
            cur_k = k[r];
          }
          if (CSF && fresh[r]) {  // close the fibre
#pragma unroll
            for (int x = 0; x < V; ++x) {
              acc[x] += c_cur[x] * t[x];
              t[x] = T(0);
              c_cur[x] = c[r][x];
            }
          }
          if (CSF) i[r] = new_row >> r & 1 ? (r == 0 && at_first ? first_i : s_i[e + r]) : cur;
          if (i[r] != cur) {  // close the row
            if (!has_head) {
              has_head = true;
              first_close = cur;
#pragma unroll
              for (int x = 0; x < V; ++x) (CSF ? s_lead[tid] : lead)[x] = acc[x];
            } else if (jok) {
              store_cols<T, V>(A + static_cast<int64_t>(cur) * J + col, acc);
            }
            cur = i[r];
#pragma unroll
            for (int x = 0; x < V; ++x) acc[x] = T(0);
          }
#pragma unroll
          for (int x = 0; x < V; ++x) {
            if (CSF) t[x] += v[r] * d[r][x];
            else acc[x] += v[r] * c_cur[x] * d[r][x];
          }
        }
      }
    }
  }
  if (CSF)
#pragma unroll
    for (int x = 0; x < V; ++x) acc[x] += c_cur[x] * t[x];

  // sums of open rows over the groups: (a row ends here, what is open after it)
  bool f = has_head;
#pragma unroll
  for (int s = 1; s < kGroupsOfWave; s <<= 1) {
    const bool uf = __shfl_up(static_cast<int>(f), s * L);
    const bool in = lane >= s * L;
#pragma unroll
    for (int x = 0; x < V; ++x) {
      const T up = __shfl_up(acc[x], s * L);
      if (in && !f) acc[x] = up + acc[x];
    }
    f = f || (in && uf);
  }
  if (lane / L == kGroupsOfWave - 1) {
#pragma unroll
    for (int x = 0; x < V; ++x) s_v[wave_id()][gl][x] = acc[x];
    if (gl == 0) s_f[wave_id()] = f;
  }
  __syncthreads();
  T pre[V];
  bool pre_f = false;
#pragma unroll
  for (int x = 0; x < V; ++x) pre[x] = T(0);
  for (int w = 0; w < wave_id(); ++w) {
    const bool wf = s_f[w];
#pragma unroll
    for (int x = 0; x < V; ++x) pre[x] = wf ? s_v[w][gl][x] : pre[x] + s_v[w][gl][x];
    pre_f = pre_f || wf;
  }
  T before[V];  // open before this group
  bool before_f = __shfl_up(static_cast<int>(f), L);
  if (lane < L) before_f = false;
#pragma unroll
  for (int x = 0; x < V; ++x) {
    const T up = __shfl_up(acc[x], L);
    before[x] = before_f ? up : (lane < L ? pre[x] : pre[x] + up);
  }
  before_f = before_f || pre_f;
  if (has_head) {
#pragma unroll
    for (int x = 0; x < V; ++x) before[x] += CSF ? s_lead[tid][x] : lead[x];
    if (before_f) {
      if (jok && first_close >= 0) store_cols<T, V>(A + static_cast<int64_t>(first_close) * J + col, before);
    } else {  // precedes the first row that starts in the chunk
      if (jok) store_cols<T, V>(carry_vec + static_cast<int64_t>(chunk) * J + col, before);
      if (keeps_keys) carry_key[chunk] = max(first_close, -1);
    }
  }
  if (g == NG - 1) {
    if (!f)
#pragma unroll
      for (int x = 0; x < V; ++x) acc[x] = pre[x] + acc[x];
    if (f || pre_f) {
      if (jok) store_cols<T, V>(A + static_cast<int64_t>(cur) * J + col, acc);
    } else {  // no row starts in the chunk
      if (jok) store_cols<T, V>(carry_vec + static_cast<int64_t>(chunk) * J + col, acc);
      if (keeps_keys) carry_key[chunk] = cur;
    }
  }
}

// One level of carries: the same sums over 64 carries per workgroup and 32 columns, a thread adding
// eight of them, into A; what continues a row begun in an earlier workgroup leaves as a carry again.
// (Bound by latency: a longer walk per thread only takes longer. 48 800 carries with 32 per thread: 20 us.)
template <typename T>
__global__ __launch_bounds__(kBlock) void mttkrp_carry_kernel(int n, int J, const int32_t* __restrict__ key,
                                                              const T* __restrict__ vec, T* __restrict__ A,
                                                              int32_t* __restrict__ out_key, T* __restrict__ out_vec) {
  constexpr int NG = kBlock / kCarryCols;
  __shared__ T s_lead[NG][kCarryCols], s_tail[NG][kCarryCols];
  __shared__ int s_first[NG], s_last[NG];
  __shared__ bool s_head[NG];
  const int g = threadIdx.x / kCarryCols, c = threadIdx.x % kCarryCols;
  const int j = blockIdx.y * kCarryCols + c, jc = min(j, J - 1);
  const int g0 = blockIdx.x * kCarrySpan + g * kCarryRows;
  int32_t k[kCarryRows];
  T v[kCarryRows];
#pragma unroll
  for (int r = 0; r < kCarryRows; ++r) {
    const int w = min(g0 + r, n - 1);
    k[r] = key[w];
    v[r] = vec[static_cast<int64_t>(w) * J + jc];
  }
  int cur = g0 > 0 ? key[min(g0, n) - 1] : -1, first = -1;
  bool head = false;
  T acc = 0, lead = 0;
#pragma unroll
  for (int r = 0; r < kCarryRows; ++r) {
    if (g0 + r >= n) break;
    if (k[r] != cur) {
      if (!head) {
        head = true;
        first = cur;
        lead = acc;
      } else if (cur >= 0 && j < J) {
        A[static_cast<int64_t>(cur) * J + j] += acc;
      }
      cur = k[r];
      acc = 0;
    }
    acc += v[r];
  }
  s_lead[g][c] = lead;
  s_tail[g][c] = acc;
  if (c == 0) {
    s_head[g] = head;
    s_first[g] = first;
    s_last[g] = cur;
  }
  __syncthreads();
  if (g > 0) return;
  T run = 0;
  bool seen = false;
  for (int q = 0; q < NG; ++q) {
    if (!s_head[q]) {
      run += s_tail[q][c];
      continue;
    }
    const T total = run + s_lead[q][c];
    if (seen) {
      if (s_first[q] >= 0 && j < J) A[static_cast<int64_t>(s_first[q]) * J + j] += total;
    } else {
      if (j < J) out_vec[static_cast<int64_t>(blockIdx.x) * J + j] = total;
      if (j == 0) out_key[blockIdx.x] = s_first[q];
    }
    seen = true;
    run = s_tail[q][c];
  }
  const int last = s_last[NG - 1];
  if (seen) {
    if (last >= 0 && j < J) A[static_cast<int64_t>(last) * J + j] += run;
  } else {
    if (j < J) out_vec[static_cast<int64_t>(blockIdx.x) * J + j] = run;
    if (j == 0) out_key[blockIdx.x] = last;
  }
}

// Adds the remaining carries to A: eight lanes for the first carry of a row and one column add up
// all carries of the row, in double also for float data.
constexpr int kFixLanes = 8;
template <typename T>
__global__ __launch_bounds__(kBlock) void mttkrp_fixup_kernel(int n, int J, const int32_t* __restrict__ key,
                                                              const T* __restrict__ vec, T* __restrict__ A) {
  const int64_t idx = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) / kFixLanes;
  if (idx >= static_cast<int64_t>(n) * J) return;
  const int w = static_cast<int>(idx / J), j = static_cast<int>(idx % J);
  const int32_t k = key[w];
  if (k < 0 || (w > 0 && key[w - 1] == k)) return;  // the same for all eight lanes
  double s = 0;
  for (int u = w + threadIdx.x % kFixLanes; u < n && key[u] == k; u += kFixLanes)
    s += static_cast<double>(vec[static_cast<int64_t>(u) * J + j]);
#pragma unroll
  for (int d = 1; d < kFixLanes; d <<= 1) s += __shfl_xor(s, d);
  if (threadIdx.x % kFixLanes == 0) {
    T* a = A + static_cast<int64_t>(k) * J + j;
    *a = static_cast<T>(static_cast<double>(*a) + s);
  }
}

// Few carries, in one launch: the workgroup of the first carry of a row adds up all of the row, whose end
// it looks up first (rows read ahead without knowing cost 5 us where most rows have one carry). 738 000
// entries in CSF, J = 16, fp64: 4.8 us, 13 in two launches. A row of all 2048 carries of 32 columns takes 16 rounds, which
// two launches take as long for from some 2600 on (6.5M entries in two slices, fp32, J = 32: 73.9 / 76.7 in one); rows of up to 16
// columns only from 4096 on, where launching them all costs as much (one launch / two: 4.5M entries, J = 8, fp32 53.8 / 59.4; 6.5M, J = 16,
// 82.2 / 86.9; J = 32, 4.5M 76.8 / 81.8; 9M in 4400 carries, J = 32, the same). Beyond 32 columns, 2048 carries are 4096 workgroups.
constexpr int kRunBlock = 512;
static int carry_runs_most(int J) { return J <= 16 ? 4096 : J <= 32 ? 2560 : 2048; }
template <typename T>
__global__ __launch_bounds__(kRunBlock) void mttkrp_carry_runs_kernel(int n, int J, int log_cols,
                                                                   const int32_t* __restrict__ key,
                                                                   const T* __restrict__ vec, T* __restrict__ A) {
  __shared__ double s_sum[kRunBlock];
  const int w = blockIdx.x, k = key[w];
  if (k < 0 || (w > 0 && key[w - 1] == k)) return;
  const int tid = threadIdx.x, cols = 1 << log_cols, rows = kRunBlock >> log_cols;
  const int c = tid & (cols - 1), j = blockIdx.y * cols + c, jc = min(j, J - 1);
  int end = w;  // of the row's carries
  for (;;) {
    const int more = __syncthreads_count(end + tid < n && key[min(end + tid, n - 1)] == k);
    end += more;
    if (more < kRunBlock) break;
  }
  constexpr int U = 8;
  double sum = 0;
  for (int u = w + (tid >> log_cols); u < end; u += U * rows) {
    T v[U];
#pragma unroll
    for (int q = 0; q < U; ++q) v[q] = vec[static_cast<int64_t>(min(u + q * rows, end - 1)) * J + jc];
#pragma unroll
    for (int q = 0; q < U; ++q) sum += u + q * rows < end ? static_cast<double>(v[q]) : 0.0;
  }
  s_sum[tid] = sum;
  __syncthreads();
  for (int d = kRunBlock / 2; d >= cols; d >>= 1) {
    if (tid < d) s_sum[tid] += s_sum[tid + d];
    __syncthreads();
  }
  if (tid < cols && j < J) {
    T* a = A + static_cast<int64_t>(k) * J + j;
    *a = static_cast<T>(static_cast<double>(*a) + s_sum[tid]);
  }
}

// ---- host ------------------------------------------------------------------

// The rows of eight entries in flight together instead of four, whose registers leave three workgroups to a compute unit: while there are
// no more (four / eight, us: CSF, 738 000 entries, fp64, J = 16 31.2 / 30.1; COO 25.5 / 24.5; 220 000 16.0 / 15.2, but 400 000
// in 781 workgroups 20.8 / 22.3; of 16 lanes even slices lose 3 %), and where a group has eight, COO, fp32, J up to 8 (30M 225 / 219, even 316 / 284;
// fp64, J = 4 232 / 240, 323 / 313).
static bool mttkrp_eight(const MttkrpPlan& P, int dtype, bool csf) {
  if (P.lanes == 2) return !csf && dtype == SPT_F32 && P.epg == 8;
  return P.vec > 1 && (P.lanes == 4 || P.lanes == 8) && P.epg >= 8 && P.blocks <= 3 * 256;
}

// Is it worth 10 us to order the chunks by their rows of C? An L2 has to be too small for the factors, C to be
// the larger part of an eighth's traffic saved, and the gathers long enough. Given order / ordered, us:
//   COO, slices of 10 000 entries, C and D 10.2 and 6.4 MB, 20M entries 536 / 361; C and D 7.7 MB, 5M 149 / 131
//   COO, skewed slices, 10.2 and 6.4 MB, 50M 648 / 617; 12.8 and 12.8, 20M (fp64) 389 / 370; 6.4 and 6.4, 10M 185 / 176;
//     3.8 and 6.4, 10M 172 / 170; 1.9 and 6.4, 10M 157 / 164; 6.4 and 1.3, 10M 125 / 128; 7.9 and 7.9, 6M 196 / 195
//   CSF, skewed, 10.2 and 6.4, 40M 578 / 523; 20.5 and 12.8, 20M (fp64) 720 / 690; 1.9 and 3.8, 10M 119 / 128
//   COO and CSF, even slices shorter than a chunk (which then needs rows from all of C), 10.2 and 6.4: 8.5M entries in slices of 85 or
//     212 254 / 262 and 268 / 276, 20M in slices of 200 556 / 567, 40M in slices of 400 1091 / 1101. Skewed slices of the same mean
//     length gain, 157 / 150, 302 / 283, 536 / 506, and a descriptor does not tell the two apart.
static bool mttkrp_orders(const MttkrpPlan& P, int64_t nnz, int64_t J, int64_t value, int64_t rows_c, int64_t rows_d) {
  const int64_t c = rows_c * J * value, d = rows_d * J * value;
  return nnz >= 8000000 && c >= 6000000 && c + d >= 12000000 &&
         P.n1 * J * value >= (P.n1 / kOrderShare + 1) * kRadix * 4;  // (the counts take the room of the carries)
}

static size_t mttkrp_bytes(const MttkrpPlan& P, size_t row) {
  return align_up(static_cast<size_t>(P.n1) * 4, 256) + align_up(P.n1 * row, 256) +
         align_up(static_cast<size_t>(P.n2) * 4, 256) + align_up(P.n2 * row, 256) +
         align_up(static_cast<size_t>(P.n1 + 1) * 12, 256) + 256;
}
static MttkrpPlan mttkrp_least(const spt_tensor* B, int32_t J) {
  return mttkrp_plan(B->nvals, J, B->dtype, B->level[1].kind == SPT_COMPRESSED, 1, true);
}
// What a call makes best use of: of one plan, or of another where both factors lie on lines, or a workgroup's carries are short.
size_t mttkrp3_workspace(const spt_tensor* B, int32_t J) {
  J = std::max(J, 1);
  const size_t row = static_cast<size_t>(J) * (B->dtype == SPT_F64 ? 8 : 4);
  const bool csf = B->level[1].kind == SPT_COMPRESSED;
  const int parts = mttkrp_parts(B->nvals, row, B->level[1].N, B->level[2].N, csf);
  return std::max({mttkrp_bytes(mttkrp_least(B, J), row), mttkrp_bytes(mttkrp_plan(B->nvals, J, B->dtype, csf, 1), row),
                   mttkrp_bytes(mttkrp_plan(B->nvals, J, B->dtype, csf, parts), row)});
}

template <typename T>
static spt_status mttkrp3_typed(Format f, const spt_tensor* B, const T* Cm, const T* Dm, int J, T* A, void* ws,
                                size_t ws_bytes, hipStream_t s) {
  const int64_t I = B->level[0].N, nnz64 = B->nvals, size = I * J;
  const bool csf = f == Format::CSF3;
  const int64_t nsl = csf ? B->level[1].M : 0, nfib = csf ? B->level[2].M : 0;
  const bool on_lines = (reinterpret_cast<uintptr_t>(Cm) | reinterpret_cast<uintptr_t>(Dm)) % kLine == 0;
  MttkrpPlan P = mttkrp_plan(nnz64, J, B->dtype, csf, on_lines ? mttkrp_parts(nnz64, J * (int64_t)sizeof(T), B->level[1].N, B->level[2].N, csf) : 1);
  const size_t row = std::max(J, 1) * sizeof(T);
  if (ws_bytes < mttkrp_bytes(P, row)) P = mttkrp_least(B, std::max(J, 1));
  if (nnz64 + P.chunk >= INT32_MAX || size >= ((int64_t)1 << 38) || nsl + 1 >= INT32_MAX || nfib + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "mttkrp: tensor too large");
  if (nnz64 > 0 && (!ws || ws_bytes < mttkrp_bytes(P, row)))
    return fail(SPT_ERR_WORKSPACE, "mttkrp: workspace of %zu bytes needed, %zu given", mttkrp_bytes(P, row), ws_bytes);
  const int nnz = (int)nnz64, n1 = (int)P.n1, n2 = (int)P.n2;
  Workspace W(ws, ws_bytes);
  int32_t *key1 = nullptr, *key2 = nullptr, *bounds = nullptr;
  T *vec1 = nullptr, *vec2 = nullptr;
  if (nnz > 0) {
    key1 = W.take<int32_t>(n1);
    vec1 = W.take<T>((size_t)n1 * J);
    key2 = W.take<int32_t>(n2);
    vec2 = W.take<T>((size_t)n2 * J);
    bounds = W.take<int32_t>(3 * ((size_t)n1 + 1));
  }
  const int fill = (int)((size + kBlock * kVec<T> - 1) / (kBlock * kVec<T>));
  const bool wide = n1 <= kWideSearch;
  const int search = csf && nnz > 0 ? ((n1 + 1) * (wide ? kWave : 8) + kBlock - 1) / kBlock : 0;
  if (fill + search > 0) {
    if (wide)
      hipLaunchKernelGGL((mttkrp_prepare_kernel<T, kWave>), dim3(fill + search), dim3(kBlock), 0, s, A, size, fill, n1, P.chunk,
                         (int)nsl, (int)nfib, B->level[1].pos, B->level[2].pos, bounds);
    else
      hipLaunchKernelGGL((mttkrp_prepare_kernel<T, 8>), dim3(fill + search), dim3(kBlock), 0, s, A, size, fill, n1, P.chunk,
                         (int)nsl, (int)nfib, B->level[1].pos, B->level[2].pos, bounds);
    SPT_CHECK_LAUNCH("mttkrp prepare");
  }
  if (nnz == 0 || J == 0) return SPT_OK;
  const CsfLevels up{B->level[0].crd, B->level[1].pos, B->level[1].crd, B->level[2].pos, bounds, (int)nsl, (int)nfib};
  const bool in_order = mttkrp_orders(P, nnz64, J, sizeof(T), B->level[1].N, B->level[2].N);
  if (in_order) {
    const StretchDigit digit(B->level[1].N);
    const int shares = (n1 + kOrderShare - 1) / kOrderShare;
    int32_t *noted = key1, *hist = reinterpret_cast<int32_t*>(vec1);  // free until the rows are made
    if (csf)
      hipLaunchKernelGGL(mttkrp_bin_kernel<true>, dim3(shares), dim3(kBlock), 0, s, nnz, P.chunk, n1, digit, nullptr, up, noted, hist);
    else
      hipLaunchKernelGGL(mttkrp_bin_kernel<false>, dim3(shares), dim3(kBlock), 0, s, nnz, P.chunk, n1, digit, B->level[1].crd, up, noted, hist);
    SPT_CHECK_LAUNCH("mttkrp bins");
    hipLaunchKernelGGL(mttkrp_order_kernel, dim3(shares), dim3(kBlock), 0, s, n1, noted, hist, bounds);
    SPT_CHECK_LAUNCH("mttkrp order");
  }
  const Placing placing{n1, P.parts, J / P.parts, in_order};
  const bool near = static_cast<uint64_t>(std::max(B->level[1].N, B->level[2].N)) * J * sizeof(T) <= uint64_t{1} << 32;
  const bool placed = in_order || P.parts > 1 || !near;
  const int of = kXcds / P.parts;
  const int64_t blocks = placed ? kXcds * ((P.n1 + of - 1) / of) : n1;
  const size_t lds = csf ? (size_t)P.chunk * 8 + 2 * (size_t)((P.chunk + 31) / 32) * 6 : 0;
  const bool eight = !placed && mttkrp_eight(P, B->dtype, csf);
#define SPT_MTTKRP_AS(L_, V_, CSF_, PLACED_, ...)                                                                      \
  hipLaunchKernelGGL((mttkrp_rows_kernel<T, L_, V_, CSF_, PLACED_, __VA_ARGS__>), dim3((unsigned)blocks, P.tiles), dim3(kBlock), lds, s, nnz, J, P.epg, placing, \
                     csf ? nullptr : B->level[0].crd, csf ? nullptr : B->level[1].crd, B->level[2].crd,                  \
                     static_cast<const T*>(B->vals), Cm, Dm, up, A, key1, vec1, bounds)
#define SPT_MTTKRP(L_, V_)                                \
  if (csf && !near) SPT_MTTKRP_AS(L_, V_, true, true, 1, false);   \
  else if (!near) SPT_MTTKRP_AS(L_, V_, false, true, 1, false);   \
  else if (csf && placed) SPT_MTTKRP_AS(L_, V_, true, true, 1);   \
  else if (csf) SPT_MTTKRP_AS(L_, V_, true, false, 1);         \
  else if (placed) SPT_MTTKRP_AS(L_, V_, false, true, 1);    \
  else SPT_MTTKRP_AS(L_, V_, false, false, 1)
#define SPT_MTTKRP_EIGHT(L_)                                        \
  if (csf) SPT_MTTKRP_AS(L_, kVec<T>, true, false, 2);                \
  else SPT_MTTKRP_AS(L_, kVec<T>, false, false, 2)
  if (P.vec == 1) { SPT_MTTKRP(4, 1); }
  else if (P.lanes == 2 && eight) { if constexpr (sizeof(T) == 4) SPT_MTTKRP_AS(2, kVec<T>, false, false, 2); }
  else if (P.lanes == 2) { SPT_MTTKRP(2, kVec<T>); }
  else if (P.lanes == 4 && eight) { SPT_MTTKRP_EIGHT(4); }
  else if (P.lanes == 4) { SPT_MTTKRP(4, kVec<T>); }
  else if (P.lanes == 8 && eight) { SPT_MTTKRP_EIGHT(8); }
  else if (P.lanes == 8) { SPT_MTTKRP(8, kVec<T>); }
  else if (P.lanes == 16) { SPT_MTTKRP(16, kVec<T>); }
  else { SPT_MTTKRP(32, kVec<T>); }
#undef SPT_MTTKRP_EIGHT
#undef SPT_MTTKRP
#undef SPT_MTTKRP_AS
  SPT_CHECK_LAUNCH("mttkrp rows");
  if (n1 <= carry_runs_most(J)) {
    int log_cols = 2;
    while (log_cols < 5 && (1 << log_cols) < J) ++log_cols;
    hipLaunchKernelGGL(mttkrp_carry_runs_kernel<T>, dim3(n1, (J + (1 << log_cols) - 1) >> log_cols), dim3(kRunBlock), 0, s,
                       n1, J, log_cols, key1, vec1, A);
    SPT_CHECK_LAUNCH("mttkrp carry runs");
    return SPT_OK;
  }
  hipLaunchKernelGGL(mttkrp_carry_kernel<T>, dim3(n2, (J + kCarryCols - 1) / kCarryCols), dim3(kBlock), 0, s, n1, J, key1,
                     vec1, A, key2, vec2);
  SPT_CHECK_LAUNCH("mttkrp carries");
  hipLaunchKernelGGL(mttkrp_fixup_kernel<T>, dim3((unsigned)(((int64_t)n2 * J * kFixLanes + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, n2, J, key2, vec2, A);
  SPT_CHECK_LAUNCH("mttkrp fixup");
  return SPT_OK;
}

spt_status mttkrp_dispatch(Format f, const spt_tensor* B, const void* C, const void* D, int32_t J,
                           void* A_out, void* ws, size_t ws_bytes, hipStream_t s) {
  for (int k = 0; k < 3; ++k)
    if (!(B->level[k].flags & SPT_ORDERED))
      return fail(SPT_ERR_UNSUPPORTED, "mttkrp: every level of B must be ordered");
  if (B->dtype == SPT_F64)
    return mttkrp3_typed<double>(f, B, static_cast<const double*>(C), static_cast<const double*>(D), J,
                                 static_cast<double*>(A_out), ws, ws_bytes, s);
  return mttkrp3_typed<float>(f, B, static_cast<const float*>(C), static_cast<const float*>(D), J,
                              static_cast<float*>(A_out), ws, ws_bytes, s);
}

}  // namespace spt
