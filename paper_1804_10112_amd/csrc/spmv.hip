// SpMV y = A x on CSR, COO, DIA and ELL (paper Section 5.2), gfx950.
//
// The matrix arrays are read once with coalesced, mostly non-temporal loads, x is gathered through the
// caches. What bounds a kernel: the rate of a large copy where x is read in order (DIA, banded CSR: 5 TB/s);
// the gathers of x where columns are anywhere (ELL, CSR, COO: 0.95 to 1.05 of what a kernel that only gathers
// reaches); launches and latency for some ten thousand entries.
//  * CSR: a group of lanes per row; fp32 rows of 8 to 32 entries, many of them, 256 at a time through LDS.
//    CSR with long or strongly skewed rows and large sorted COO share one kernel: a
//    workgroup owns a fixed chunk of stored entries (balanced in entries, not rows, so power-law rows cost
//    nothing extra), stages the products in LDS and reduces them per row with a
//    segmented scan; a row cut by a chunk boundary is finished by a tiny carry
//    kernel. No atomics, results are bit-reproducible.
//  * Sorted COO of up to 2^24 entries: a wave per 256 entries, in one launch up to 65 536.
//  * Unsorted COO is the paper's scatter loop with atomic adds into y, from 786 432 entries on the binned
//    scatter of coo_bin.hip.
//  * DIA and ELL read the diagonal-major / slot-major arrays with consecutive
//    rows in consecutive lanes.
#include <algorithm>
#include <type_traits>

#include "carry.hpp"
#include "common.hpp"
#include "segreduce.hpp"
#include "slices.hpp"
#include "wavescan.hpp"

namespace spt {

template <typename T>
__device__ __forceinline__ T ld_stream(const T* p) {
  return __builtin_nontemporal_load(p);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fill_kernel(T* __restrict__ out, int64_t n, T value) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) out[i] = value;
}

// ---------------------------------------------------------------- DIA
// Cell (d,i) at d*N+i holds A(i, i+offset[d]) (range level: rows, offset
// level: cols; Table 2). One row per thread, the diagonals in a register loop.
constexpr int kDiaMaxLdsOffsets = 1024;

template <typename T>
__global__ __launch_bounds__(kBlock) void dia_spmv_kernel(int64_t N, int64_t M, int K,
                                                          const int32_t* __restrict__ offset,
                                                          const T* __restrict__ vals,
                                                          const T* __restrict__ x,
                                                          T* __restrict__ y) {
  __shared__ int32_t s_off[kDiaMaxLdsOffsets];
  const bool in_lds = K <= kDiaMaxLdsOffsets;
  if (in_lds) {
    for (int d = threadIdx.x; d < K; d += kBlock) s_off[d] = offset[d];
    __syncthreads();
  }
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= N) return;
  T acc = 0;
#pragma unroll 8
  for (int d = 0; d < K; ++d) {
    const int64_t j = i + (in_lds ? s_off[d] : offset[d]);
    if (j >= 0 && j < M) acc += ld_stream(vals + (int64_t)d * N + i) * x[j];
  }
  y[i] = acc;
}

// ---------------------------------------------------------------- DIA / ELL, R rows per lane
// 16-byte loads: a lane owns R consecutive rows (R = 2 for fp64, 4 for fp32), and every access to
// the diagonal-major / slot-major arrays is one 16-byte vector. HBM delivers ~7 TB/s to 16-byte
// lane loads but under 4 TB/s to 4-byte ones, hence the width. The vectors need element alignment
// only (the hardware takes them at any dword), so any number of rows will do: the last lane starts
// at row N - R, and rows that two lanes compute get the same value twice.
// 16 bytes of values and the columns that go with them, at any entry: vector loads that are only
// element-aligned.
template <typename T> struct Entries;
template <> struct Entries<double> {
  static constexpr int K = 2;
  typedef double V __attribute__((ext_vector_type(2), aligned(8)));
  typedef int32_t I __attribute__((ext_vector_type(2), aligned(4)));
};
template <> struct Entries<float> {
  static constexpr int K = 4;
  typedef float V __attribute__((ext_vector_type(4), aligned(4)));
  typedef int32_t I __attribute__((ext_vector_type(4), aligned(4)));
};

template <typename T> struct VecOf;
template <> struct VecOf<double> { static constexpr int R = 2; typedef double type __attribute__((ext_vector_type(2))); typedef int32_t itype __attribute__((ext_vector_type(2))); };
template <> struct VecOf<float> { static constexpr int R = 4; typedef float type __attribute__((ext_vector_type(4))); typedef int32_t itype __attribute__((ext_vector_type(4))); };

// KT > 0: the number of diagonals is the compile-time constant KT, so all KT
// diagonal loads and their x loads are issued before the first use (one memory
// round trip per lane). KT == 0: any K, in batches of 8 (the tail batch re-reads
// the last diagonal and masks it out).
// A diagonal whose row range [max(0,-off), min(N, M-off)) misses all rows of the
// wave is skipped by the whole wave (a scalar branch: far diagonals are empty
// over half the matrix, and loading their cells would move bytes that are never
// used). Where the range covers the wave's rows, x is one vector per lane as well; only
// the waves at a diagonal's ends read x element by element, at a clamped index.
// 7 diagonals, against x gathered element by element and a lane per row where no vector divides the
// rows: 3.66M rows fp32 38 -> 23 us, 1.83M rows fp64 30 -> 24 us, 1.5M rows (odd) fp64 24 -> 20 us.
template <typename T, int KT>
__global__ __launch_bounds__(kBlock) void dia_spmv_vec_kernel(int64_t N, int64_t M, int K,
                                                              const int32_t* __restrict__ offset,
                                                              const T* __restrict__ vals,
                                                              const T* __restrict__ x,
                                                              T* __restrict__ y) {
  constexpr int R = Entries<T>::K;
  constexpr int B = KT > 0 ? KT : 8;
  using V = typename Entries<T>::V;
  const int64_t blk0 = (int64_t)xcd_contiguous_block_id() * kBlock;
  // rows [w0, w1) belong to this wave (uniform: kept in scalar registers)
  const int64_t w0 = (blk0 + __builtin_amdgcn_readfirstlane(threadIdx.x & ~(kWave - 1))) * R;
  if (w0 >= N) return;
  const int64_t w1 = w0 + kWave * R < N ? w0 + kWave * R : N;
  int64_t i0 = (blk0 + threadIdx.x) * R;
  if (i0 > N - R) i0 = N - R;
  T acc[R] = {};
  const int kend = KT > 0 ? KT : K;
  for (int d0 = 0; d0 < kend; d0 += B) {
    V v[B];
    V xv[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int d = min(d0 + u, kend - 1);
      const int64_t off = offset[d];  // uniform address: a scalar load
      v[u] = 0;
      xv[u] = 0;
      const int64_t lo = off < 0 ? -off : 0, hi = (M - off) < N ? (M - off) : N;
      if (w0 < hi && w1 > lo && d0 + u < kend) {  // uniform
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(vals + (int64_t)d * N + i0));
        if (w0 - R >= lo && w1 <= hi) {  // uniform (the last lane may start before w0)
          xv[u] = *reinterpret_cast<const V*>(x + i0 + off);
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int64_t j = i0 + off + r;
            const bool in = j >= 0 && j < M;
            xv[u][r] = x[in ? j : 0];
            if (!in) v[u][r] = xv[u][r] = 0;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += v[u][r] * xv[u][r];
  }
  V out;
#pragma unroll
  for (int r = 0; r < R; ++r) out[r] = acc[r];
  *reinterpret_cast<V*>(y + i0) = out;
}

// Fewer rows than a vector holds.
template <typename T>
__global__ __launch_bounds__(kBlock) void ell_spmv_kernel(int64_t N, int W, const int32_t* __restrict__ crd,
                                                          const T* __restrict__ vals, const T* __restrict__ x,
                                                          T* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= N) return;
  T acc = 0;
  for (int k = 0; k < W; ++k) {
    const int32_t j = crd[(int64_t)k * N + i];
    if (j >= 0) acc += vals[(int64_t)k * N + i] * x[j];
  }
  y[i] = acc;
}

// ELL: cell (k,i) at k*N+i; a negative column marks padding and is skipped without touching its
// value or x. S waves share the slots of 64 * R rows and add up their parts in LDS: a matrix of few
// rows would otherwise keep a wave for every 128 or 256 rows walking through all slots, one batch
// of memory round trips after the other (42 000 rows of 32 slots: fp64 27 -> 9 us, fp32 25 -> 6.5 us;
// 16 waves with two slots each gain nothing more). From kEllWaves waves on the chip is full without
// that, and the plain loop over the slots reaches the rate of the x gathers (1M rows, fp32: 111 us;
// split, or with batches of 4 or 8 slots, 117 to 135).
constexpr int kEllWaves = 2800;

template <typename T, int S>
__global__ __launch_bounds__(kBlock) void ell_spmv_vec_kernel(
    int64_t N, int W, const int32_t* __restrict__ crd, const T* __restrict__ vals, const T* __restrict__ x,
    T* __restrict__ y) {
  constexpr int R = Entries<T>::K;
  constexpr int NR = kBlock / S;  // a workgroup takes NR * R rows
  constexpr int kBatch = 8;  // slots whose loads are in flight together
  using V = typename Entries<T>::V;
  using I = typename Entries<T>::I;
  __shared__ T s_part[S > 1 ? S : 1][S > 1 ? NR * R : 1];
  const int lr = threadIdx.x % NR, part = S > 1 ? threadIdx.x / NR : 0;
  int64_t i0 = ((int64_t)blockIdx.x * NR + lr) * R;
  const bool live = i0 < N;
  if (i0 > N - R) i0 = N - R;
  const int per = (W + S - 1) / S;
  const int k0 = part * per, k1 = min(k0 + per, W);
  T acc[R] = {};
  if (live && S == 1) {
#pragma unroll 4
    for (int k = 0; k < W; ++k) {
      const int64_t c = (int64_t)k * N + i0;
      const I j = __builtin_nontemporal_load(reinterpret_cast<const I*>(crd + c));
      const V v = __builtin_nontemporal_load(reinterpret_cast<const V*>(vals + c));
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (j[r] >= 0) acc[r] += v[r] * x[j[r]];
    }
  } else if (live) {
    for (int k = k0; k < k1; k += kBatch) {
      I j[kBatch];
      V v[kBatch];
      T g[kBatch][R];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t c = (int64_t)min(k + u, k1 - 1) * N + i0;
        j[u] = __builtin_nontemporal_load(reinterpret_cast<const I*>(crd + c));
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(vals + c));
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          g[u][r] = 0;
          if (k + u < k1 && j[u][r] >= 0) g[u][r] = x[j[u][r]];
          else v[u][r] = 0;
        }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += v[u][r] * g[u][r];
    }
  }
  if (S > 1) {
#pragma unroll
    for (int r = 0; r < R; ++r) s_part[part][r * NR + lr] = acc[r];
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int q = 1; q < S; ++q)
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += s_part[q][r * NR + lr];
  }
  if (!live) return;
  V out;
#pragma unroll
  for (int r = 0; r < R; ++r) out[r] = acc[r];
  *reinterpret_cast<V*>(y + i0) = out;
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// ---------------------------------------------------------------- CSR / sorted COO
// Chunk of IPT*256 consecutive entries per workgroup.
//   phase 1  coalesced load of col/vals (and row for COO), gather x, product
//            and key into LDS (padded so that phase 2 is bank-conflict free)
//   CSR only the rows that start inside the chunk are found with two wave-wide
//            searches of pos; each such row marks its first entry as a head
//            (empty rows store y = 0 directly)
//   phase 2  every thread reduces IPT consecutive entries, segments that start
//            and end inside one thread are stored at once; a workgroup scan of
//            the per-thread summaries closes the rest
// Output protocol: the workgroup that contains a row's first entry stores the
// row's (possibly partial) sum with a plain store; the sum of the entries that
// precede the first head of a chunk leaves as carry (key, value) number
// `chunk`, key -1 if there is none.
template <int IPT>
__device__ __forceinline__ int lds_slot(int e) { return e + e / IPT; }

// How an entry's column is turned into x_j ("locate" into the vector operand,
// Section 3.2): a dense array, an ordered sparse vector (binary search of its
// crd), or a hash-map vector (Table 2's probing: start at j % W, step +1 with
// wrap, stop at j, at an empty bucket (-1) or after a full cycle).
template <typename T>
struct DenseX {
  const T* __restrict__ x;
  __device__ __forceinline__ T at(int32_t j) const { return x[j]; }
};
template <typename T>
struct SparseX {
  const int32_t* __restrict__ crd;
  const T* __restrict__ vals;
  int n;
  __device__ __forceinline__ T at(int32_t j) const {
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (crd[mid] < j) lo = mid + 1;
      else hi = mid;
    }
    return (lo < n && crd[lo] == j) ? vals[lo] : T(0);
  }
};
template <typename T>
struct HashX {
  const int32_t* __restrict__ crd;
  const T* __restrict__ vals;
  int W;
  __device__ __forceinline__ T at(int32_t j) const {
    int p = j % W;
    for (int step = 0; step < W; ++step) {
      const int32_t c = crd[p];
      if (c == j) return vals[p];
      if (c == -1) break;
      p = p + 1 == W ? 0 : p + 1;
    }
    return T(0);
  }
};

template <typename T, bool CSR, int IPT, bool VEC, class XP = DenseX<T>>
__global__ __launch_bounds__(kBlock) void seg_spmv_kernel(
    int nnz, int nrows, const int32_t* __restrict__ pos_or_row, const int32_t* __restrict__ col,
    const T* __restrict__ vals, const XP x, T* __restrict__ y,
    int32_t* __restrict__ carry_key, T* __restrict__ carry_val,
    const uint8_t* __restrict__ select, int want) {
  constexpr int CHUNK = IPT * kBlock;
  if (!selected(select, want)) return;  // the other CSR kernel was chosen on the device
  __shared__ T s_val[CHUNK + kBlock];
  __shared__ int32_t s_key[CHUNK + kBlock];
  __shared__ SegScanStorage<T> s_scan;
  __shared__ int s_rows[2];

  const int tid = threadIdx.x;
  const int chunk = xcd_contiguous_block_id();
  const int base = chunk * CHUNK;  // host guarantees nnz + CHUNK < 2^31
  const int end = min(base + CHUNK, nnz);
  const bool last_chunk = (end == nnz);

  if (CSR) {
    if (wave_id() == 0) {
      int r = wave_lower_bound(pos_or_row, nrows + 1, base);
      if (lane_id() == 0) s_rows[0] = r;
    } else if (wave_id() == 1) {
      int r = last_chunk ? nrows : wave_lower_bound(pos_or_row, nrows + 1, end);
      if (lane_id() == 0) s_rows[1] = r;
    }
  }

  // phase 1: a lane loads R consecutive entries per step with 16-byte (fp32) or
  // 8+16-byte (fp64) vector loads when the arrays allow it
  constexpr int R = VecOf<T>::R;
  using V = typename VecOf<T>::type;
  using IV = typename VecOf<T>::itype;
  int32_t fill_key = -1;
  if (!CSR) fill_key = pos_or_row[end - 1];  // tail padding extends the last segment
#pragma unroll
  for (int q = 0; q < IPT / R; ++q) {
    const int e0 = (q * kBlock + tid) * R;
    const int p0 = base + e0;
    int32_t c[R], key[R];
    T v[R];
    bool ok[R];
    if (VEC && p0 + R <= end) {
      const IV cv = ld_stream(reinterpret_cast<const IV*>(col + p0));
      const V vv = ld_stream(reinterpret_cast<const V*>(vals + p0));
      IV kv = fill_key;
      if (!CSR) kv = ld_stream(reinterpret_cast<const IV*>(pos_or_row + p0));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        c[r] = cv[r];
        v[r] = vv[r];
        key[r] = kv[r];
        ok[r] = true;
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        ok[r] = p0 + r < end;
        c[r] = ok[r] ? ld_stream(col + p0 + r) : 0;
        v[r] = ok[r] ? ld_stream(vals + p0 + r) : T(0);
        key[r] = (!CSR && ok[r]) ? ld_stream(pos_or_row + p0 + r) : fill_key;
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      s_val[lds_slot<IPT>(e0 + r)] = ok[r] ? v[r] * x.at(c[r]) : T(0);
      s_key[lds_slot<IPT>(e0 + r)] = key[r];
    }
  }
  int32_t prev_key = -1;  // key of the entry before the chunk (COO)
  if (!CSR && base > 0) prev_key = pos_or_row[base - 1];
  __syncthreads();

  int carry_row = prev_key;
  if (CSR) {
    const int r_lo = s_rows[0], r_hi = s_rows[1];
    // the row cut by the chunk start, if the chunk does not begin with a head
    carry_row = r_lo - 1;
    strided(r_lo, r_hi, tid, kBlock, [&](int r) {
      const int a = pos_or_row[r], b = pos_or_row[r + 1];
      if (b > a) s_key[lds_slot<IPT>(a - base)] = r;
      else y[r] = T(0);
    });
    __syncthreads();
  }

  // phase 2
  T acc = 0, lead = 0;
  int has_head = 0, last_key = -1, first_close_key = -1;
  bool head_at_chunk_start = false;
  int32_t kprev = prev_key;
  if (!CSR && tid > 0) kprev = s_key[lds_slot<IPT>(tid * IPT - 1)];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int e = tid * IPT + k;
    const int32_t key = s_key[lds_slot<IPT>(e)];
    const T v = s_val[lds_slot<IPT>(e)];
    const bool head = CSR ? (key >= 0) : (key != kprev);
    if (head) {
      if (!has_head) {
        lead = acc;
        has_head = 1;
        first_close_key = kprev;  // COO; CSR takes it from the scan
        head_at_chunk_start = (e == 0);
      } else {
        y[CSR ? last_key : kprev] = acc;
      }
      acc = 0;
      last_key = key;
    }
    acc += v;
    if (!CSR) kprev = key;
  }

  SegSum<T> in = block_seg_exclusive_scan<T>(SegSum<T>{has_head, acc, last_key}, s_scan);

  if (has_head) {
    const T total = in.v + lead;
    if (in.f) {
      y[CSR ? in.k : first_close_key] = total;
    } else {  // first head of the chunk: what precedes it continues an earlier chunk
      carry_key[chunk] = head_at_chunk_start ? -1 : (CSR ? carry_row : first_close_key);
      carry_val[chunk] = total;
    }
  }
  if (tid == kBlock - 1) {  // the segment still open at the end of the chunk
    if (has_head) {
      y[last_key] = acc;  // COO: last_key == kprev
    } else if (in.f) {
      y[CSR ? in.k : kprev] = in.v + acc;
    } else {  // no head in the whole chunk: everything is carry
      carry_key[chunk] = CSR ? carry_row : kprev;
      carry_val[chunk] = in.v + acc;
    }
  }
}

// ---------------------------------------------------------------- CSR
// G lanes per row, each with 16 bytes of values and the columns that go with them: the lanes of a
// wave, row after row, read one stretch of the arrays, and nothing is staged, searched or waited
// for at a barrier: bounds, entries, x, y are the only memory round trips of a row. K entries per
// lane (2 fp64, 4 fp32) halve or quarter the load instructions against one entry per lane, which
// is what large short-rowed matrices are bound by (7 entries per row, 12.8M entries: fp64 46 ->
// 28 us, fp32 43 -> 18 us). Rows beyond 4 K G entries are added up by the whole wave, beyond
// kRowsWide by the whole workgroup, so that a long row costs its length divided by what those
// have in flight. Fixed order of additions: bit-reproducible.
// Against a kernel that streamed 256 rows at a time through LDS and let a lane add up each, in us,
// three matrices in turn:
//   entries                800 000      1.6M      6.4M      12.8M      25.6M
//   7 per row, fp64      8.0 / 5.7  8.6 / 6.8  20 / 18    39 / 35    74 / 67
//   uniform, mean 10, "   10 / 7.8   16 / 12   55 / 53  158 / 155  393 / 388
//   power law, mean 15, " 25 / 11    31 / 18   77 / 71  194 / 165  429 / 416
//   8 to 32, fp32        9.6 / 5.8   14 / 10   39 / 32    68 / 75  170 / 178
constexpr int kRowsWide = 4096;
constexpr int kShortRow = 32;    // a declared bound up to here means rows of much the same length

// Sum over the G lanes of a group, in every lane of it.
template <int G, typename T>
__device__ __forceinline__ T group_sum(T v) {
  if (G >= 16) v += dpp_move<0x128, 0xf>(T(0), v);                  // row_ror:8
  if (G >= 16) v += dpp_move<0x124, 0xf>(T(0), v);                  // row_ror:4
  if (G == 8) v += dpp_move<0x141, 0xf>(T(0), v);                   // row_half_mirror
  if (G >= 4) v += dpp_move<0x4E, 0xf>(T(0), v);                    // quad_perm 2,3,0,1
  if (G >= 2) v += dpp_move<0xB1, 0xf>(T(0), v);                    // quad_perm 1,0,3,2
#pragma unroll
  for (int d = 16; d < G; d <<= 1) v += __shfl_xor(v, d);
  return v;
}

// Rows block * NG * R and the NG * R - 1 that follow.
template <typename T, int G, int R, bool NT, class XP>
__device__ __forceinline__ void csr_rows_block(int block, int nrows, int nnz,
                                               const int32_t* __restrict__ pos, const int32_t* __restrict__ crd,
                                               const T* __restrict__ vals, const XP& x, T* __restrict__ y) {
  constexpr int NG = kBlock / G;
  constexpr int K = Entries<T>::K;
  constexpr int KG = K * G;
  using V = typename Entries<T>::V;
  using I = typename Entries<T>::I;
  __shared__ int s_wide[NG * R];  // rows left to the whole workgroup
  __shared__ int s_nwide;
  __shared__ T s_part[kBlock / kWave];
  const int tid = threadIdx.x, lane = lane_id();
  const int gl = tid % G;
  // rows of one pass over the groups are neighbours: a wave reads one stretch of entries per pass
  const int row0 = block * (NG * R) + tid / G;
  int a[R], b[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = min(row0 + r * NG, nrows - 1);
    a[r] = pos[row];
    b[r] = pos[row + 1];
  }
  if (tid == 0) s_nwide = 0;
  T acc[R];
  bool wide = false;
  // K entries from `off` on in the row that begins at `base`; loads stay inside the arrays, and no index
  // passes nnz, which may be 2^31 - 2
  const int lastv = nnz - K;
  const auto load = [&](int base, int off, I& c, V& v) {
    const int q = base + min(off, lastv - base);
    c = NT ? __builtin_nontemporal_load(reinterpret_cast<const I*>(crd + q)) : *reinterpret_cast<const I*>(crd + q);
    v = NT ? __builtin_nontemporal_load(reinterpret_cast<const V*>(vals + q)) : *reinterpret_cast<const V*>(vals + q);
  };
  // x at those that count (they belong to the row, of `len` entries; an idle lane gathers nothing), 0 at the
  // others: all gathers of a step are on their way before the first is used
  const auto counts = [&](int base, int off, int len, int k) {
    const int q = min(off, lastv - base);
    return q + k >= off && q + k < len;
  };
  const auto gather = [&](int base, int off, int len, const I& c, T (&g)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      g[k] = 0;
      if (counts(base, off, len, k)) g[k] = x.at(c[k]);
    }
  };
  // What does not count is not added: its value may be another row's infinity. The sum is selected, not
  // the value, whose load a selection ahead of the gathers would wait for (7 per row, 14M entries, fp32:
  // 19.3 against 23.3 us).
  const auto dot = [&](int base, int off, int len, const V& v, const T (&g)[K]) {
    T t = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const T sum = t + v[k] * g[k];
      t = counts(base, off, len, k) ? sum : t;
    }
    return t;
  };
  {
    I c[R];
    V v[R];
    T g[R][K];
    int len[R];  // a row for the whole wave or workgroup is left out
#pragma unroll
    for (int r = 0; r < R; ++r) {
      len[r] = b[r] - a[r];
      load(a[r], gl * K < len[r] ? gl * K : 0, c[r], v[r]);  // an idle lane reads what its row's first lane reads
      if (len[r] > 4 * KG) len[r] = 0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) gather(a[r], gl * K, len[r], c[r], g[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = dot(a[r], gl * K, len[r], v[r], g[r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int len = b[r] - a[r];
    if (len > KG && len <= 4 * KG) {
      for (int off = KG + gl * K; off < len; off += KG) {
        I c;
        V v;
        T g[K];
        load(a[r], off, c, v);
        gather(a[r], off, len, c, g);
        acc[r] += dot(a[r], off, len, v, g);
      }
    }
    acc[r] = group_sum<G>(acc[r]);
    uint64_t todo = __ballot(gl == 0 && len > 4 * KG && len <= kRowsWide);
    while (todo) {
      const int src = __ffsll(static_cast<long long>(todo)) - 1;
      todo &= todo - 1;
      const int base = __builtin_amdgcn_readlane(a[r], src), wlen = __builtin_amdgcn_readlane(len, src);
      T part = 0;
      for (int off = lane * K; off < wlen; off += 2 * K * kWave) {
        I c[2];
        V v[2];
        T g[2][K];
#pragma unroll
        for (int u = 0; u < 2; ++u) load(base, off + u * K * kWave, c[u], v[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) gather(base, off + u * K * kWave, wlen, c[u], g[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) part += dot(base, off + u * K * kWave, wlen, v[u], g[u]);
      }
      part = wave_total<T>(part);
      if (lane == src) acc[r] = part;
    }
    const int row = row0 + r * NG;
    if (row < nrows && gl == 0 && len <= kRowsWide) y[row] = acc[r];
    wide |= row < nrows && len > kRowsWide;
  }
  if (!__syncthreads_or(wide)) return;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (gl == 0 && row0 + r * NG < nrows && b[r] - a[r] > kRowsWide) s_wide[atomicAdd(&s_nwide, 1)] = row0 + r * NG;
  __syncthreads();
  const int nwide = s_nwide;
  for (int w = 0; w < nwide; ++w) {
    const int r = s_wide[w];
    const int la = pos[r], len = pos[r + 1] - la;
    constexpr int U = 8;  // entries of a thread in flight
    const int whole = len / (U * kBlock);
    const int32_t* rc = crd + la + tid;
    const T* rv = vals + la + tid;
    T part = 0;
    for (int round = 0; round < whole; ++round) {
      int32_t c[U];
      T v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c[u] = rc[u * kBlock];
        v[u] = rv[u * kBlock];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) part += v[u] * x.at(c[u]);
      rc += U * kBlock;
      rv += U * kBlock;
    }
    const int left = len - whole * (U * kBlock) - tid;  // of the row, from this thread's next entry on
    int32_t c[U];
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = 0;  // left unset, they take the whole kernel from 58 registers to 90 (fp64; 36.8 -> 43.6 us)
      v[u] = 0;
      if (u * kBlock < left) {
        c[u] = rc[u * kBlock];
        v[u] = rv[u * kBlock];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u * kBlock < left) part += v[u] * x.at(c[u]);
    part = wave_total<T>(part);
    if (lane == 0) s_part[wave_id()] = part;
    __syncthreads();
    if (tid == 0) {
      T sum = 0;
#pragma unroll
      for (int u = 0; u < kBlock / kWave; ++u) sum += s_part[u];
      y[r] = sum;
    }
    __syncthreads();
  }
}

template <typename T, int G, int R, bool NT, class XP>
__global__ __launch_bounds__(kBlock) void csr_rows_kernel(int nrows, int nnz,
                                                          const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ crd,
                                                          const T* __restrict__ vals, const XP x,
                                                          T* __restrict__ y) {
  csr_rows_block<T, G, R, NT>(xcd_contiguous_block_id(), nrows, nnz, pos, crd, vals, x, y);
}
// One of two candidates (the device has chosen): workgroups take several blocks, since the start of
// 10^5 workgroups that return at once costs 40 us.
template <typename T, int G, int R, class XP>
__global__ __launch_bounds__(kBlock) void csr_rows_if_kernel(int nblocks, int nrows, int nnz,
                                                             const int32_t* __restrict__ pos,
                                                             const int32_t* __restrict__ crd,
                                                             const T* __restrict__ vals, const XP x,
                                                             T* __restrict__ y, const ByRowsIf cond) {
  if (!selected(cond.flags, false)) {
    if (cond.seg_row) find_segment_rows(nrows, pos, cond.nseg, cond.seg_row, y);
    return;
  }
  for (int block = blockIdx.x; block < nblocks; block += gridDim.x) {
    csr_rows_block<T, G, R, true>(xcd_contiguous_block_id(block, nblocks), nrows, nnz, pos, crd, vals, x, y);
    __syncthreads();
  }
}
constexpr int kIfBlocks = 16384;  // a multiple of the XCDs: a workgroup's blocks stay on one

// 256 rows through LDS: their entries, one stretch of the arrays, are read side by side whatever their rows,
// and the products parked in LDS, where a lane adds up its row's. What that saves is accesses to the first-level
// cache, of which it takes one for every 64 bytes of entries; by rows, a group's vectors straddle its lines and
// some lanes are idle: 23.4M accesses against 27.3M (19M entries, 8 to 32 per row, fp32), with that unit busy
// throughout. Worth it for fp32, whose x fits an L2 (the gathers beyond it hide everything else) and whose
// entries do not (from there the row kernel is faster). In us, caches cleared / not, by rows and this way:
//   8 to 32 per row     6.4M 42 / 30 and 42 / 36      12.8M 79 / 73 and 71 / 65       25.6M 181 / 175 and 173 / 168
//                       19M 124 / 118 and 114 / 109   30.4M (x 6.4 MB) 236 / 232 and 236 / 232
//   uniform, mean 10    12.8M 98 / 93 and 92 / 87     25.6M (x 10 MB) 294 / 290 and 292 / 288
//   power law, mean 15 to 20   12.8M 106 / 92 and 101 / 94   14M 146 / 130 and 122 / 111   20M 219 / 198 and 214 / 205
// A sparse or hashed x is looked up for every entry, which idle lanes waste: any such matrix whose entries do not
// stay cached. By rows and this way, 20M entries, a thousandth of x stored: fp64, mean 20, 280 and 214 us sparse,
// 334 and 227 hashed, mean 4 415 and 359, 247 and 195; fp32, mean 20, 245 and 214, 274 and 220 (half of it stored:
// equal to within 5 %; 5M entries, not taken: fp32, mean 4, 79 and 103).
// A block with very long rows (taken from 16 384 entries on instead of 40 960: 115 and 224 us for the power
// laws), and the last, whose vectors would pass the end, go by rows.
constexpr int kStreamPiece = 2048;                      // products in LDS
constexpr int kStreamMost = 160 * kBlock;               // entries of a block
constexpr int kStreamLane = 48;                         // entries of a row that a lane adds up alone, else its wave
constexpr int64_t kStreamXBytes = int64_t(6) << 20;     // an L2 of 4 MB keeps most of it
template <typename T, class XP>
__global__ __launch_bounds__(kBlock) void csr_stream_kernel(int nrows, int nnz, const int32_t* __restrict__ pos,
                                                            const int32_t* __restrict__ crd,
                                                            const T* __restrict__ vals, const XP x,
                                                            T* __restrict__ y) {
  using V = typename Entries<T>::V;
  using I = typename Entries<T>::I;
  constexpr int K = Entries<T>::K, U = kStreamPiece / (K * kBlock), kG = 8;
  __shared__ int32_t s_pos[kBlock + 1];
  __shared__ T s_prod[kStreamPiece];
  const int tid = threadIdx.x, block = xcd_contiguous_block_id(), row0 = block * kBlock;
  for (int q = tid; q <= kBlock; q += kBlock) s_pos[q] = pos[min(row0 + q, nrows)];
  __syncthreads();
  const int e0 = s_pos[0], e1 = s_pos[kBlock];
  if (e1 - e0 > kStreamMost || e1 + K > nnz) {  // uniform
    for (int q = 0; q < kG; ++q) {
      csr_rows_block<T, kG, 1, true>(block * kG + q, nrows, nnz, pos, crd, vals, x, y);
      __syncthreads();
    }
    return;
  }
  const int ra = s_pos[tid], rb = s_pos[tid + 1];
  T acc = 0;
  for (int c0 = e0 / K * K; c0 < e1; c0 += kStreamPiece) {
    const int c1 = min(c0 + kStreamPiece, e1);
    I c[U];
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = c0 + K * (u * kBlock + tid);
      const int q = p < c1 ? p : c0;  // an idle lane reads what the first one reads, and parks what nobody adds
      c[u] = __builtin_nontemporal_load(reinterpret_cast<const I*>(crd + q));
      v[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(vals + q));
    }
    T prod[U][K];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) prod[u][k] = v[u][k] * x.at(c[u][k]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) s_prod[K * (u * kBlock + tid) + k] = prod[u][k];
    __syncthreads();
    const int a = max(ra, c0), e = min(rb, c1);
    const bool big = e - a > kStreamLane;
    for (int q = a; q < (big ? a : e); q += 8) {
      T t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] = s_prod[min(q + k, e - 1) - c0];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc += q + k < e ? t[k] : T(0);
    }
    uint64_t todo = __ballot(big);
    while (todo) {
      const int src = __ffsll(static_cast<long long>(todo)) - 1;
      todo &= todo - 1;
      const int la = __shfl(a, src) - c0, lb = __shfl(e, src) - c0;
      T part = 0;
      for (int q = la + lane_id(); q < lb; q += kWave) part += s_prod[q];
      part = wave_total<T>(part);
      if (lane_id() == src) acc += part;
    }
    __syncthreads();
  }
  if (row0 + tid < nrows) y[row0 + tid] = acc;
}

// By rows, or dealt out evenly in entries? A bound declared on the rows (max_children) decides; else
// the mean row, since a row beyond kRowsWide entries keeps one workgroup busy (0.1 ms per 10^5 entries)
// and few long rows leave the chip idle. In us, by rows / by entries, fp64, even rows and power-law rows:
//   entries   mean 16                mean 64                mean 1024      131 072
//   100 000   4.5 / 8.8, 6.2 / 8.8   4.8 / 8.7, 9.7 / 8.4   9.5 / 9.6
//   1M        13 / 18, 27 / 18       14 / 17, 34 / 18       19 / 17        1277 / 17
//   10M       102 / 115, 159 / 114   107 / 113, 221 / 112   114 / 112      1600 / 110
// (20M entries in one row: 20 ms / 0.17 ms.) Even rows beyond a mean of 32 would gain little by rows,
// skewed ones lose much; up to 2^17 entries, where a launch saved is half the time, twice that mean.
// Fewer than four entries do not fill a vector load. By entries takes a workspace: a caller who was not told
// to need one (no bound declared) and brings none has its rows walked.
constexpr int64_t kRowsMean = kShortRow, kRowsFew = int64_t(1) << 17;
size_t seg_spmv_workspace(int64_t nnz);
static bool csr_use_rows(int64_t nnz, int64_t nrows, int hint, const void* ws, size_t ws_bytes) {
  if (nnz < 4 || nnz >= INT32_MAX || nrows + kBlock >= INT32_MAX) return false;
  if (hint > 0) return hint <= kShortRow;
  if (nnz <= nrows * kRowsMean * (nnz <= kRowsFew ? 2 : 1)) return true;
  return !ws || ws_bytes < seg_spmv_workspace(nnz);
}

template <typename T, class XP>
static spt_status launch_csr_rows(int64_t nnz, int64_t nrows, const int32_t* pos, const int32_t* crd, const T* vals,
                                  const XP x, T* y, hipStream_t s, int64_t ncols = INT64_MAX,
                                  const ByRowsIf* cond = nullptr) {
  // Rows per group at once: two where rows are so short that one leaves a lane with a single load
  // (7 entries per row, 25.6M entries, fp64: 80 -> 70 us), else one. Up to 2^20 entries the chip is
  // not full and waves that hold fewer rows meet fewer long ones: groups twice as wide.
#define SPT_ROWS(G_, R_)                                                                                      \
  do {                                                                                                        \
    const int nb = (int)((nrows + kBlock / G_ * R_ - 1) / (kBlock / G_ * R_));                                \
    if (cond)                                                                                                 \
      hipLaunchKernelGGL((csr_rows_if_kernel<T, G_, R_, XP>), dim3(std::min(nb, kIfBlocks)), dim3(kBlock), 0, \
                         s, nb, (int)nrows, (int)nnz, pos, crd, vals, x, y, *cond);                           \
    else if (large)                                                                                           \
      hipLaunchKernelGGL((csr_rows_kernel<T, G_, R_, true, XP>), dim3(nb), dim3(kBlock), 0, s, (int)nrows,     \
                         (int)nnz, pos, crd, vals, x, y);                                                     \
    else                                                                                                      \
      hipLaunchKernelGGL((csr_rows_kernel<T, G_, R_, false, XP>), dim3(nb), dim3(kBlock), 0, s, (int)nrows,     \
                         (int)nnz, pos, crd, vals, x, y);                                                     \
  } while (0)
  // Entries are read past the caches once the matrix would leave no room for x in them (7 per row,
  // 25.6M entries, fp64: 76 -> 67 us; but 1.6M entries, uniform: 12 -> 14 us).
  const bool large = nnz * (4 + (int64_t)sizeof(T)) > 96000000;
  const bool small = nnz <= (1 << 20);
  const bool two = !small && nnz <= 8 * nrows;
  constexpr bool dense = std::is_same<XP, DenseX<T>>::value;
  if constexpr (sizeof(T) == 4 || !dense) {
    // (its indices pass the end by up to a piece, which must not pass 2^31)
    if (!cond && nnz + 2 * kStreamPiece < INT32_MAX &&
        (dense ? large && nnz >= 8 * nrows && nnz <= kShortRow * nrows && ncols <= kStreamXBytes / (int)sizeof(T)
               : large)) {
      hipLaunchKernelGGL((csr_stream_kernel<T, XP>), dim3((unsigned)((nrows + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                         (int)nrows, (int)nnz, pos, crd, vals, x, y);
      SPT_CHECK_LAUNCH("csr_stream");
      return SPT_OK;
    }
  }
  const int64_t lanes = nnz / Entries<T>::K * (small ? 2 : 1);
  if (lanes <= 2 * nrows) {
    if (two) SPT_ROWS(2, 2);
    else SPT_ROWS(2, 1);
  } else if (lanes <= 4 * nrows) {
    if (two) SPT_ROWS(4, 2);
    else SPT_ROWS(4, 1);
  } else if (lanes <= 8 * nrows) {
    SPT_ROWS(8, 1);
  } else if (lanes <= 16 * nrows) {
    SPT_ROWS(16, 1);
  } else {
    SPT_ROWS(32, 1);
  }
#undef SPT_ROWS
  SPT_CHECK_LAUNCH("csr_rows");
  return SPT_OK;
}

// ---------------------------------------------------------------- unsorted COO
// The fused single loop over all entries of the paper's COO kernel: a scatter into y (Section 4.5, fusing
// iterators). Bound by the atomics in global memory, which one address takes at 12 ns each, the whole of it at
// 20 G a second. A workgroup therefore adds up its 1024 entries in a table of rows in LDS first (the first row
// that meets a slot has it, the others of that slot go straight to y) and then adds each slot to y. In us,
// fp64, against one atomic an entry:
//   entries                        20 000       100 000      400 000      786 000
//   uniform rows                   7.1 / 6.7    8.3 / 8.5     22 / 22      41 / 41
//   power law                       19 / 7.2     24 / 9.7     39 / 23      70 / 48
//   half of them in one row        124 / 6.9    607 / 7.0   2402 / 20    4723 / 30
// (512 entries and 1024 slots: 55 us for the last power law; 2048 and 2048: 43, but 7.5 to 9 us for few entries.)
constexpr int kScatterPerLane = 4, kScatterEntries = kScatterPerLane * kBlock;
constexpr int kScatterSlotBits = 10;
template <typename T>
__global__ __launch_bounds__(kBlock) void coo_atomic_spmv_kernel(
    int nnz, const int32_t* __restrict__ row, const int32_t* __restrict__ col,
    const T* __restrict__ vals, const T* __restrict__ x, T* __restrict__ y) {
  constexpr int kSlots = 1 << kScatterSlotBits;
  __shared__ int32_t s_row[kSlots];
  __shared__ T s_sum[kSlots];
  const int tid = threadIdx.x;
  const int base = blockIdx.x * kScatterEntries;
  int32_t r[kScatterPerLane];
  T prod[kScatterPerLane];
#pragma unroll
  for (int e = 0; e < kScatterPerLane; ++e) {
    const int p = min(base + e * kBlock + tid, nnz - 1);
    r[e] = ld_stream(row + p);
    prod[e] = ld_stream(vals + p) * x[ld_stream(col + p)];
  }
  for (int q = tid; q < kSlots; q += kBlock) {
    s_row[q] = -1;
    s_sum[q] = T(0);
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kScatterPerLane; ++e) {
    if (base + e * kBlock + tid < nnz) {
      const int slot = static_cast<uint32_t>(r[e]) * 2654435769u >> (32 - kScatterSlotBits);
      const int owner = atomicCAS(&s_row[slot], -1, r[e]);
      if (owner == -1 || owner == r[e]) atomicAdd(&s_sum[slot], prod[e]);
      else unsafeAtomicAdd(y + r[e], prod[e]);
    }
  }
  __syncthreads();
  for (int q = tid; q < kSlots; q += kBlock)
    if (s_row[q] >= 0) unsafeAtomicAdd(y + s_row[q], s_sum[q]);
}

// ---------------------------------------------------------------- sorted COO, small
// The whole product in one launch, for matrices whose run time is the launches themselves.
// One wave per 256 consecutive entries (four per lane). The wave that holds a row's first
// entry owns the row: it adds up the row's entries of its own piece with a segmented sum over
// the lanes and, if the row is still open at the end of the piece, keeps reading the entries
// that follow, 64 at a time, until the row changes; entries before a piece's first row start
// belong to an earlier owner and are skipped. Rows without entries lie between the rows of
// two neighbouring entries (or before the first / after the last entry) and are zeroed by the
// thread that sees the gap. No workspace, no atomics, a fixed order of additions.
constexpr int kSmallPiece = 4 * kWave;
constexpr int64_t kSmallCooMaxEntries = 1 << 16;  // worst case (one row holds everything): 1024 read-ahead rounds
constexpr int64_t kSmallCooMaxRows = 1 << 20;     // worst case (all rows empty but one): one wave zeroes them, 16 384 rounds

template <typename T>
__device__ __forceinline__ void zero_rows(T* __restrict__ y, int lo, int hi) {  // rows lo .. hi - 1
  const bool big = hi - lo > 16;
  if (!big)
    for (int r = lo; r < hi; ++r) y[r] = T(0);
  uint64_t todo = __ballot(big);
  while (todo) {  // a long run of empty rows is zeroed by the whole wave
    const int src = __ffsll(static_cast<long long>(todo)) - 1;
    todo &= todo - 1;
    const int l = __shfl(lo, src), h = __shfl(hi, src);
    strided(l, h, lane_id(), kWave, [&](int r) { y[r] = T(0); });
  }
}

template <typename T>
__global__ __launch_bounds__(kWave) void coo_small_spmv_kernel(int nnz, int nrows, const int32_t* __restrict__ row,
                                                               const int32_t* __restrict__ col,
                                                               const T* __restrict__ vals, const T* __restrict__ x,
                                                               T* __restrict__ y) {
  const int lane = lane_id();
  const int base = blockIdx.x * kSmallPiece;
  const int end = min(base + kSmallPiece, nnz);
  const int p0 = base + lane * 4;
  int32_t r[4], c[4];
  T v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool ok = p0 + q < nnz;
    const int p = ok ? p0 + q : nnz - 1;  // beyond the end: the last entry's row again, value 0
    r[q] = row[p];
    c[q] = col[p];
    v[q] = ok ? vals[p] : T(0);
  }
  // the 64 entries after the piece, one per lane: where an open row usually ends
  const int pa = end + lane;
  const bool ahead_ok = pa < nnz;
  int32_t ra = ahead_ok ? row[pa] : -1, ca = ahead_ok ? col[pa] : 0;
  T va = ahead_ok ? vals[pa] : T(0);
  int32_t prev = dpp_move<0x138, 0xf>(-1, r[3]);  // wave_shr:1
  if (lane == 0) prev = base > 0 ? row[base - 1] : -1;
  T prod[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) prod[q] = p0 + q < nnz ? v[q] * x[c[q]] : T(0);
  const T prod_a = ahead_ok ? va * x[ca] : T(0);

  unsigned headmask = 0;
  {
    int32_t a = prev;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool valid = p0 + q < nnz;
      if (valid && r[q] != a) headmask |= 1u << q;
      zero_rows<T>(y, valid && r[q] != a ? a + 1 : 0, valid && r[q] != a ? r[q] : 0);
      if (valid) a = r[q];
    }
    // rows after the last entry of the matrix
    const bool last_entry = p0 <= nnz - 1 && nnz - 1 < p0 + 4;
    zero_rows<T>(y, last_entry ? row[nnz - 1] + 1 : 0, last_entry ? nrows : 0);
  }

  T acc = 0;
  int has_head = 0, last_key = -1;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (headmask & (1u << q)) {
      if (has_head) y[last_key] = acc;  // a row that starts and ends inside this lane
      has_head = 1;
      last_key = r[q];
      acc = 0;
    }
    acc += prod[q];
  }
  SegSum<T> me{has_head, acc, last_key};
  wave_seg_step<0x111, 0xf>(me);
  wave_seg_step<0x112, 0xf>(me);
  wave_seg_step<0x114, 0xf>(me);
  wave_seg_step<0x118, 0xf>(me);
  wave_seg_step<0x142, 0xa>(me);
  wave_seg_step<0x143, 0xc>(me);
  SegSum<T> ex;  // what the lanes before this one add up to
  ex.f = dpp_move<0x138, 0xf>(0, me.f);
  ex.v = dpp_move<0x138, 0xf>(T(0), me.v);
  ex.k = dpp_move<0x138, 0xf>(-1, me.k);
  // the first head of a lane closes the row that was open in the lanes before it; if no lane
  // before holds a head, that row began in an earlier piece and its owner adds these entries
  if (has_head && ex.f) {
    T lead = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (headmask & (1u << q)) break;
      lead += prod[q];
    }
    y[ex.k] = ex.v + lead;
  }
  // the row still open at the end of the piece (inclusive summary of the last lane)
  const int open_f = __shfl(me.f, kWave - 1);
  if (!open_f) return;  // no row starts in this piece
  const int open_row = __shfl(me.k, kWave - 1);
  T sum = __shfl(me.v, kWave - 1);
  bool more = true;
  {
    const bool match = ahead_ok && ra == open_row;
    sum += wave_total<T>(match ? prod_a : T(0));
    more = __ballot(match) == ~uint64_t(0);
  }
  for (int q0 = end + kWave; more; q0 += kWave) {  // a long row: keep reading, 64 entries a round
    const int p = q0 + lane;
    const bool match = p < nnz && row[min(p, nnz - 1)] == open_row;
    const T t = match ? vals[p] * x[col[p]] : T(0);
    sum += wave_total<T>(t);
    more = __ballot(match) == ~uint64_t(0);
  }
  if (lane == 0) y[open_row] = sum;
}

// Ordered COO: one wave per 256 consecutive entries (four per lane, 16-byte loads). The sum
// of a row goes to y from the piece that holds its first entry; what precedes a piece's first row
// start leaves as a carry. ZERO: rows without entries are zeroed by the thread that sees the gap.
// Bound by launches and latency for few entries (200 000 entries, fp64, with a workgroup per 2048
// entries, a fill and a serial fixup: 10.1 us), by the gathers of x and the streams for many.
template <typename T, bool ZERO>
__global__ __launch_bounds__(kBlock) void coo_pieces_kernel(int nnz, int npieces, int nrows,
                                                            const int32_t* __restrict__ row,
                                                            const int32_t* __restrict__ col,
                                                            const T* __restrict__ vals, const T* __restrict__ x,
                                                            T* __restrict__ y, int32_t* __restrict__ carry_key,
                                                            T* __restrict__ carry_val) {
  typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  const int lane = lane_id();
  const int piece = xcd_contiguous_block_id() * (kBlock / kWave) + wave_id();
  if (piece >= npieces) return;
  const int base = piece * kSmallPiece, p0 = base + lane * 4;
  int32_t r[4], c[4];
  T v[4];
  if (base + kSmallPiece <= nnz) {  // uniform
    const I4 rr = __builtin_nontemporal_load(reinterpret_cast<const I4*>(row + p0));
    const I4 cc = __builtin_nontemporal_load(reinterpret_cast<const I4*>(col + p0));
    const V4 vv = __builtin_nontemporal_load(reinterpret_cast<const V4*>(vals + p0));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      r[q] = rr[q];
      c[q] = cc[q];
      v[q] = vv[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = min(p0 + q, nnz - 1);  // beyond the end: the last entry's row again, value 0
      r[q] = row[p];
      c[q] = col[p];
      v[q] = p0 + q < nnz ? vals[p] : T(0);
    }
  }
  int32_t before = -1;
  if (lane == 0 && base > 0) before = row[base - 1];
  T prod[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) prod[q] = x[c[q]];
#pragma unroll
  for (int q = 0; q < 4; ++q) prod[q] = p0 + q < nnz ? v[q] * prod[q] : T(0);
  const int32_t prev = dpp_move<0x138, 0xf>(-1, r[3]);  // wave_shr:1
  if (lane > 0) before = prev;

  T acc = 0, lead = 0;
  bool has_head = false, head_first = false;
  int last_row = -1, a = before;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool head = r[q] != a;
    if (ZERO) zero_rows<T>(y, head ? a + 1 : 0, head ? r[q] : 0);
    if (head) {
      if (has_head) y[last_row] = acc;  // a row that starts and ends inside this lane
      else lead = acc;
      head_first = head_first || q == 0;
      has_head = true;
      last_row = r[q];
      acc = 0;
    }
    acc += prod[q];
    a = r[q];
  }
  if (ZERO && piece == npieces - 1) zero_rows<T>(y, lane == kWave - 1 ? r[3] + 1 : 0, lane == kWave - 1 ? nrows : 0);
  const uint64_t heads = __ballot(has_head);
  const int from = last_lane(heads, false), prev_head = last_lane(heads, true);
  const T sum = wave_marked_sum<T>(acc, from >= 0 ? lane - from : kWave);
  T open = dpp_move<0x138, 0xf>(T(0), sum);  // what is open before this lane
  if (lane == 0) open = T(0);
  const int open_row = __shfl(last_row, max(prev_head, 0));
  if (has_head) {
    if (prev_head >= 0) {
      y[open_row] = open + lead;
    } else {  // what precedes the piece's first row start
      carry_key[piece] = lane == 0 && head_first ? -1 : before;
      carry_val[piece] = open + lead;
    }
  }
  if (lane == kWave - 1) {  // the row still open at the end of the piece
    if (from >= 0) {
      y[has_head ? last_row : open_row] = sum;
    } else {
      carry_key[piece] = r[0];
      carry_val[piece] = sum;
    }
  }
}

// ---------------------------------------------------------------- launchers

// binned scatter for large unordered COO (coo_bin.hip)
template <typename T>
spt_status coo_binned_spmv(int64_t nnz, int64_t nrows, int64_t ncols, const int32_t* row, const int32_t* col,
                           const T* vals, const T* x, T* y, void* ws, size_t ws_bytes,
                           hipStream_t s);
size_t coo_binned_workspace(int dtype, int64_t nnz, int64_t nrows);
// Below this unordered entries are scattered with atomics, from here on they are binned (four launches). The line lies
// where no order of the rows loses; for rows in random order alone it would lie at half of it. In us, scatter / binned:
//   entries                       400 000           600 000           780 000
//                              fp64    fp32      fp64    fp32      fp64    fp32
//   random order, power law   27/23   29/22     41/27   48/24     49/29   59/27
//   random order, uniform     23/24   27/22     31/27   34/24     39/29   45/26
//   ordered, not flagged so    8/24    9/23      9/26   11/24     10/28   12/25
//   half of them in one row   16/35   23/33     23/38   22/36     28/41   35/38
//   CSC, banded               16/27   16/26     20/30   21/28     24/32   25/29
constexpr int64_t kBinnedMinEntries = 3 << 18;

size_t coo_unordered_workspace(int dtype, int64_t nnz, int64_t nrows) {
  return nnz >= kBinnedMinEntries ? coo_binned_workspace(dtype, nnz, nrows) : 256;
}
// The least that a call takes.
static size_t coo_unordered_least(int dtype, int64_t nnz, int64_t nrows) {
  return nnz >= kBinnedMinEntries ? coo_binned_workspace(dtype, nnz, nrows) : 0;
}

constexpr int kSegIPT = 8;

// Ordered COO of more entries: waves that hold 256 each gain nothing over workgroups of 2048 (40M
// entries, fp64, uniform rows 709 against 705 us, power law 664 against 645), and leave more carries.
constexpr int64_t kPiecesMaxEntries = int64_t(1) << 24;
size_t ordered_coo_workspace(int64_t nnz) {
  if (nnz > kPiecesMaxEntries) return seg_spmv_workspace(nnz);
  const int64_t np = (nnz + kSmallPiece - 1) / kSmallPiece;
  return align_up((size_t)np * 4, 256) + align_up((size_t)np * 8, 256) + 256;
}
size_t seg_spmv_workspace(int64_t nnz) {
  const int64_t chunk = (int64_t)kSegIPT * kBlock;
  const int64_t nwg = (nnz + chunk - 1) / chunk;
  return align_up((size_t)nwg * 4, 256) + align_up((size_t)nwg * 8, 256) + 256;
}

template <typename T>
static spt_status launch_fill(T* out, int64_t n, T v, hipStream_t s) {
  if (n <= 0) return SPT_OK;
  const int64_t grid = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(fill_kernel<T>, dim3((unsigned)grid), dim3(kBlock), 0, s, out, n, v);
  SPT_CHECK_LAUNCH("fill");
  return SPT_OK;
}

template <typename T, bool CSR, class XP>
static spt_status launch_seg_x(int64_t nnz, int64_t nrows, const int32_t* pos_or_row,
                               const int32_t* col, const T* vals, const XP x, T* y, void* ws,
                               size_t ws_bytes, hipStream_t s, const uint8_t* select = nullptr,
                               int want = 0) {
  constexpr int CHUNK = kSegIPT * kBlock;
  if (nnz == 0) return launch_fill<T>(y, nrows, T(0), s);
  if (nnz + CHUNK >= INT32_MAX || nrows + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries or rows");
  const int nwg = (int)((nnz + CHUNK - 1) / CHUNK);
  if (ws_bytes < seg_spmv_workspace(nnz) || ws == nullptr)
    return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given",
                seg_spmv_workspace(nnz), ws_bytes);
  Workspace W(ws, ws_bytes);
  int32_t* ckey = W.take<int32_t>(nwg);
  T* cval = W.take<T>(nwg);
  if (!CSR) {
    spt_status st = launch_fill<T>(y, nrows, T(0), s);
    if (st != SPT_OK) return st;
  }
  const bool vec = aligned16(col) && aligned16(vals) && (CSR || aligned16(pos_or_row));
  if (vec)
    hipLaunchKernelGGL((seg_spmv_kernel<T, CSR, kSegIPT, true, XP>), dim3(nwg), dim3(kBlock), 0, s,
                       (int)nnz, (int)nrows, pos_or_row, col, vals, x, y, ckey, cval, select, want);
  else
    hipLaunchKernelGGL((seg_spmv_kernel<T, CSR, kSegIPT, false, XP>), dim3(nwg), dim3(kBlock), 0, s,
                       (int)nnz, (int)nrows, pos_or_row, col, vals, x, y, ckey, cval, select, want);
  SPT_CHECK_LAUNCH("seg_spmv");
  hipLaunchKernelGGL(carry_fixup_kernel<T>, dim3((nwg + kBlock - 1) / kBlock), dim3(kBlock), 0, s,
                     nwg, ckey, cval, y, select, want);
  SPT_CHECK_LAUNCH("carry_fixup");
  return SPT_OK;
}

// Up to kZeroRows rows the pieces zero the rows without entries (worst case, one gap of all rows: one
// wave zeroes them in 4096 rounds), which saves the launch that zeroes all.
constexpr int64_t kZeroRows = 1 << 18;
template <typename T>
static spt_status launch_coo_pieces(int64_t nnz, int64_t nrows, const int32_t* row, const int32_t* col, const T* vals,
                                    const T* x, T* y, void* ws, size_t ws_bytes, hipStream_t s) {
  if (nnz == 0) return launch_fill<T>(y, nrows, T(0), s);
  if (nnz + kSmallPiece >= INT32_MAX || nrows + 1 >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries or rows");
  const int np = (int)((nnz + kSmallPiece - 1) / kSmallPiece);
  if (!ws || ws_bytes < ordered_coo_workspace(nnz))
    return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", ordered_coo_workspace(nnz), ws_bytes);
  Workspace W(ws, ws_bytes);
  int32_t* ckey = W.take<int32_t>(np);
  T* cval = W.take<T>(np);
  const dim3 grid((np + kBlock / kWave - 1) / (kBlock / kWave));
  if (nrows <= kZeroRows) {
    hipLaunchKernelGGL((coo_pieces_kernel<T, true>), grid, dim3(kBlock), 0, s, (int)nnz, np, (int)nrows, row, col, vals, x,
                       y, ckey, cval);
  } else {
    spt_status st = launch_fill<T>(y, nrows, T(0), s);
    if (st != SPT_OK) return st;
    hipLaunchKernelGGL((coo_pieces_kernel<T, false>), grid, dim3(kBlock), 0, s, (int)nnz, np, (int)nrows, row, col, vals, x,
                       y, ckey, cval);
  }
  SPT_CHECK_LAUNCH("coo pieces");
  hipLaunchKernelGGL(carry_fixup_kernel<T>, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, s, np, ckey, cval, y,
                     nullptr, 0);
  SPT_CHECK_LAUNCH("carry_fixup");
  return SPT_OK;
}

template <typename T, bool CSR>
static spt_status launch_seg(int64_t nnz, int64_t nrows, const int32_t* pos_or_row,
                             const int32_t* col, const T* vals, const T* x, T* y, void* ws,
                             size_t ws_bytes, hipStream_t s, const uint8_t* select = nullptr,
                             int want = 0) {
  return launch_seg_x<T, CSR, DenseX<T>>(nnz, nrows, pos_or_row, col, vals, DenseX<T>{x}, y, ws,
                                         ws_bytes, s, select, want);
}

// Large CSR matrices without a declared row bound: which kernel suits is decided on the device. A few workgroups
// look at the entry count of every block of 256 rows and, where x is too large for an L2, at samples of the columns;
// then both candidates are launched, and the one not chosen returns at once (or finds the rows of the other's
// segments). By entries if a block of rows is heavy (60M entries, power law: 0.97 ms against 1.10 by rows), with x
// slice by slice if columns lie scattered. Looking and launching cost some 12 us, which is why only matrices of
// kDynamicMinEntries entries or more (kernel times from 64 us) are looked at.
constexpr int64_t kDynamicMinEntries = int64_t(1) << 25;

// x slice by slice (spmv_slices.hip)? Above, where the choice costs little next to the product; and for ordered COO
// beyond kPiecesMaxEntries, where the one kernel does both (local columns, against a kernel of chunks in LDS: 25M entries,
// fp64 113 / 104 us, fp32 73 / 72; 36M 147 / 148 and 101 / 106). In us, uniform columns, without / with slices, by the size of x:
//   36M entries, fp64, COO   4 MB 257 / 257    6 MB 312 / 264    12 MB 493 / 281   24 MB 606 / 323   48 MB 701 / 404
//                            64 MB 712 / 461   96 MB 770 / 581 (slices of 3.2 MB; as they are now, 35M entries 96 MB 479)
//   36M entries, CSR         fp32 6 MB 272 / 234, 24 MB 593 / 294; fp64 24 MB 597 / 317, 96 MB 795 / 600
//   17M entries, COO         fp64 8 MB 200 / 138; fp32 6.4 MB 155 / 133
//   power law, CSR           fp64, 60M entries, 32 MB 970 / 545; fp32, 35M entries, 9.2 MB 378 / 248
//   local columns, CSR, 36M  a heavy row fp64 171 / 138, fp32 112 / 110; mean row 90 fp64 153 / 111, fp32 94 / 82;
// Not for rows whose declared bound sends them to the row kernel: they are spared the choice, which with local columns
// costs more than it can be made to cost less (by rows at once / chosen; fp64, 36M entries, 12 a row, 117 / 133, 98M 286 / 318;
// fp32 69 / 81 and 180 / 201; waves that go through the rows by themselves, the next ones on their way, 128, 317, 89 and
// 224), though scattered columns then take 556 instead of 313 and 430 instead of 251: who has such declares no bound.
// Takes a larger workspace than the carries of the kernels it replaces; a caller with one of that size has those.
size_t slices_spmv_workspace(int64_t nnz);
ByRowsIf slices_by_rows_if(int64_t nnz, void* ws);
spt_status launch_csr_skew(int64_t nnz, int64_t nrows, const int32_t* pos, uint8_t* flags, hipStream_t s);
template <typename T, bool CSR>
spt_status launch_slices_prepare(int64_t nnz, int64_t nrows, int64_t ncols, const int32_t* pos, const int32_t* col, T* y,
                                 void* ws, hipStream_t s);
template <typename T, bool CSR>
spt_status launch_slices_spmv(int64_t nnz, int64_t ncols, bool rows_may, const int32_t* pos_or_row, const int32_t* col,
                              const T* vals, const T* x, T* y, void* ws, hipStream_t s);
template <typename T>
spt_status launch_segment_rows(int64_t nnz, int64_t nrows, const int32_t* pos, T* y, void* ws, hipStream_t s);

static bool declared_short(int hint) { return hint > 0 && hint <= kShortRow; }
static bool slices_may_pay(bool csr, int64_t nnz, int64_t ncols, int value_bytes) {
  const int64_t x = ncols * value_bytes;
  return nnz >= (csr ? kDynamicMinEntries : kPiecesMaxEntries + 1) && nnz + (1 << 16) < INT32_MAX && x > kSlicesMinX && x <= kSlicesMaxX;
}
// What spt_workspace_bytes answers; the least that a call takes is seg_spmv_workspace and ordered_coo_workspace.
size_t csr_spmv_workspace(const spt_tensor* A) {
  const size_t least = seg_spmv_workspace(A->nvals);
  return !declared_short(A->level[1].max_children) && slices_may_pay(true, A->nvals, A->level[1].N, A->dtype == SPT_F64 ? 8 : 4)
             ? std::max(least, slices_spmv_workspace(A->nvals)) : least;
}
size_t ordered_coo_spmv_workspace(const spt_tensor* A) {
  const size_t least = ordered_coo_workspace(A->nvals);
  return slices_may_pay(false, A->nvals, A->level[1].N, A->dtype == SPT_F64 ? 8 : 4) ? std::max(least, slices_spmv_workspace(A->nvals)) : least;
}

// y = A x, A in CSR, x a sparse vector (compressed level) or a hash map (hashed level).
template <typename T>
static spt_status spmv_sparse_x_typed(const spt_tensor* A, const spt_tensor* X, T* y, void* ws,
                                      size_t ws_bytes, hipStream_t s) {
  const spt_level& L = X->level[0];
  const T* xv = static_cast<const T*>(X->vals);
  const int64_t nnz = A->nvals, N = A->level[0].N;
  const T* vals = static_cast<const T*>(A->vals);
  if (X->nvals >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "spmv: x too large");
  const bool rows = csr_use_rows(nnz, N, A->level[1].max_children, ws, ws_bytes);
  if (L.kind == SPT_HASHED) {
    if (L.M < 1) return fail(SPT_ERR_INVALID_ARG, "spmv: hashed x needs a table width W >= 1");
    if (rows)
      return launch_csr_rows<T, HashX<T>>(nnz, N, A->level[1].pos, A->level[1].crd, vals,
                                            HashX<T>{L.crd, xv, (int)L.M}, y, s);
    return launch_seg_x<T, true, HashX<T>>(nnz, N, A->level[1].pos, A->level[1].crd, vals,
                                           HashX<T>{L.crd, xv, (int)L.M}, y, ws, ws_bytes, s);
  }
  if (rows)
    return launch_csr_rows<T, SparseX<T>>(nnz, N, A->level[1].pos, A->level[1].crd, vals,
                                            SparseX<T>{L.crd, xv, (int)X->nvals}, y, s);
  return launch_seg_x<T, true, SparseX<T>>(nnz, N, A->level[1].pos, A->level[1].crd, vals,
                                           SparseX<T>{L.crd, xv, (int)X->nvals}, y, ws, ws_bytes, s);
}

spt_status spmv_sparse_x_dispatch(const spt_tensor* A, const spt_tensor* X, void* y, void* ws,
                                  size_t ws_bytes, hipStream_t s) {
  if (A->dtype == SPT_F64)
    return spmv_sparse_x_typed<double>(A, X, static_cast<double*>(y), ws, ws_bytes, s);
  return spmv_sparse_x_typed<float>(A, X, static_cast<float*>(y), ws, ws_bytes, s);
}

// y[row[r]] = t[r] for the stored rows of a doubly compressed matrix
template <typename T>
__global__ __launch_bounds__(kBlock) void scatter_rows_kernel(int n, const int32_t* __restrict__ row,
                                                              const T* __restrict__ t,
                                                              T* __restrict__ y) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r < n) y[row[r]] = t[r];
}

spt_status launch_expand_parents(int n, int nparents, const int32_t* pos, int32_t* out, hipStream_t s);

size_t csc_spmv_workspace(const spt_tensor* A) {
  return align_up(static_cast<size_t>(A->nvals) * 4, 256) +
         coo_unordered_workspace(A->dtype, A->nvals, A->level[1].N);
}

static size_t csc_spmv_least(const spt_tensor* A) {
  return align_up(static_cast<size_t>(A->nvals) * 4, 256) + coo_unordered_least(A->dtype, A->nvals, A->level[1].N);
}

size_t dcsr_spmv_workspace(const spt_tensor* A) {
  return align_up(static_cast<size_t>(A->level[1].M) * 8, 256) + seg_spmv_workspace(A->nvals);
}

template <typename T>
static spt_status spmv_typed(Format f, const spt_tensor* A, const T* x, T* y, void* ws,
                             size_t ws_bytes, hipStream_t s) {
  const T* vals = static_cast<const T*>(A->vals);
  switch (f) {
    case Format::DCSR: {
      // (compressed, compressed): the column level is a CSR over the stored rows only, so
      // the CSR kernels produce one sum per stored row, which is then placed at the row's
      // coordinate in the zero-filled y (row coordinates are unique: no two sums collide)
      const int64_t N = A->level[0].N, stored = A->level[1].M;
      spt_status st = launch_fill<T>(y, N, T(0), s);
      if (st != SPT_OK || stored == 0) return st;
      if (stored >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 stored rows");
      if (!ws || ws_bytes < dcsr_spmv_workspace(A))
        return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given",
                    dcsr_spmv_workspace(A), ws_bytes);
      Workspace W(ws, ws_bytes);
      T* t = reinterpret_cast<T*>(W.take<double>(stored));
      char* rest = static_cast<char*>(ws) + W.used;
      const int hint = A->level[1].max_children;
      if (csr_use_rows(A->nvals, stored, hint, rest, ws_bytes - W.used))
        st = launch_csr_rows<T>(A->nvals, stored, A->level[1].pos, A->level[1].crd, vals, DenseX<T>{x}, t, s,
                                A->level[1].N);
      else
        st = launch_seg<T, true>(A->nvals, stored, A->level[1].pos, A->level[1].crd, vals, x, t, rest,
                                 ws_bytes - W.used, s);
      if (st != SPT_OK) return st;
      hipLaunchKernelGGL(scatter_rows_kernel<T>, dim3(static_cast<unsigned>((stored + kBlock - 1) / kBlock)),
                         dim3(kBlock), 0, s, static_cast<int>(stored), A->level[0].crd, t, y);
      SPT_CHECK_LAUNCH("scatter rows");
      return SPT_OK;
    }
    case Format::CSR: {
      const int hint = A->level[1].max_children;
      const int64_t nnz = A->nvals, N = A->level[0].N;
      const int32_t *pos = A->level[1].pos, *crd = A->level[1].crd;
      const int64_t M = A->level[1].N;
      const bool rows = csr_use_rows(nnz, N, hint, ws, ws_bytes);
      if (!declared_short(hint) && slices_may_pay(true, nnz, M, sizeof(T)) && ws && ws_bytes >= slices_spmv_workspace(nnz) && N + kBlock < INT32_MAX) {
        const ByRowsIf cond = slices_by_rows_if(nnz, ws);
        spt_status st = launch_slices_prepare<T, true>(nnz, N, M, pos, crd, y, ws, s);
        if (st == SPT_OK)
          st = rows ? launch_csr_rows<T>(nnz, N, pos, crd, vals, DenseX<T>{x}, y, s, M, &cond)
                    : launch_segment_rows<T>(nnz, N, pos, y, ws, s);
        return st == SPT_OK ? launch_slices_spmv<T, true>(nnz, M, rows, pos, crd, vals, x, y, ws, s) : st;
      }
      if (!rows) return launch_seg<T, true>(nnz, N, pos, crd, vals, x, y, ws, ws_bytes, s);
      if (hint > 0 || nnz < kDynamicMinEntries) return launch_csr_rows<T>(nnz, N, pos, crd, vals, DenseX<T>{x}, y, s, M);
      if (!ws || ws_bytes < seg_spmv_workspace(nnz))
        return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", seg_spmv_workspace(nnz),
                    ws_bytes);
      // the flags live in the last 256 bytes of the workspace, behind the carries
      uint8_t* select = static_cast<uint8_t*>(ws) + seg_spmv_workspace(nnz) - 256;
      const ByRowsIf cond{select, nullptr, 0};
      spt_status st = launch_csr_skew(nnz, N, pos, select, s);
      if (st == SPT_OK) st = launch_csr_rows<T>(nnz, N, pos, crd, vals, DenseX<T>{x}, y, s, M, &cond);
      return st == SPT_OK ? launch_seg<T, true>(nnz, N, pos, crd, vals, x, y, ws, ws_bytes, s, select, 1) : st;
    }
    case Format::CSC: {
      // (dense columns, compressed rows): the entries lie in column order, which makes the
      // matrix a COO whose row coordinates are unordered and whose column coordinates are
      // implicit in pos. The columns are written out once, then the entries are binned by row
      // like any unordered COO; x is read in ascending order on the way.
      const int64_t nnz = A->nvals, N = A->level[1].N, M = A->level[0].N;
      if (nnz >= INT32_MAX || M + 1 >= INT32_MAX)
        return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries or columns");
      if (nnz == 0) return launch_fill<T>(y, N, T(0), s);
      if (!ws || ws_bytes < csc_spmv_least(A))
        return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", csc_spmv_least(A), ws_bytes);
      Workspace W(ws, ws_bytes);
      int32_t* cols = W.take<int32_t>(nnz);
      spt_status st = launch_expand_parents((int)nnz, (int)M, A->level[1].pos, cols, s);
      if (st != SPT_OK) return st;
      char* rest = static_cast<char*>(ws) + W.used;
      if (nnz >= kBinnedMinEntries)  // (no columns to speak of: they ascend)
        return coo_binned_spmv<T>(nnz, N, 0, A->level[1].crd, cols, vals, x, y, rest, ws_bytes - W.used, s);
      st = launch_fill<T>(y, N, T(0), s);
      if (st != SPT_OK) return st;
      hipLaunchKernelGGL(coo_atomic_spmv_kernel<T>, dim3((unsigned)((nnz + kScatterEntries - 1) / kScatterEntries)),
                         dim3(kBlock), 0, s, (int)nnz, A->level[1].crd, cols, vals, x, y);
      SPT_CHECK_LAUNCH("coo_atomic_spmv");
      return SPT_OK;
    }
    case Format::COO2: {
      const int64_t nnz = A->nvals, N = A->level[0].N;
      if ((A->level[0].flags & SPT_ORDERED) && nnz > 0 && nnz <= kSmallCooMaxEntries && N <= kSmallCooMaxRows) {
        hipLaunchKernelGGL(coo_small_spmv_kernel<T>, dim3((unsigned)((nnz + kSmallPiece - 1) / kSmallPiece)),
                           dim3(kWave), 0, s, (int)nnz, (int)N, A->level[0].crd, A->level[1].crd, vals, x, y);
        SPT_CHECK_LAUNCH("coo_small_spmv");
        return SPT_OK;
      }
      if ((A->level[0].flags & SPT_ORDERED) && slices_may_pay(false, nnz, A->level[1].N, sizeof(T)) && ws &&
          ws_bytes >= slices_spmv_workspace(nnz)) {
        spt_status st = launch_slices_prepare<T, false>(nnz, N, A->level[1].N, nullptr, A->level[1].crd, y, ws, s);
        return st == SPT_OK ? launch_slices_spmv<T, false>(nnz, A->level[1].N, false, A->level[0].crd, A->level[1].crd, vals, x, y, ws, s) : st;
      }
      if ((A->level[0].flags & SPT_ORDERED) && nnz <= kPiecesMaxEntries)
        return launch_coo_pieces<T>(nnz, N, A->level[0].crd, A->level[1].crd, vals, x, y, ws, ws_bytes, s);
      if (A->level[0].flags & SPT_ORDERED)
        return launch_seg<T, false>(nnz, N, A->level[0].crd, A->level[1].crd, vals, x, y, ws, ws_bytes, s);
      if (nnz >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "spmv: more than 2^31 entries");
      if (nnz >= kBinnedMinEntries)
        return coo_binned_spmv<T>(nnz, N, A->level[1].N, A->level[0].crd, A->level[1].crd, vals, x, y, ws, ws_bytes,
                                  s);
      spt_status st = launch_fill<T>(y, N, T(0), s);
      if (st != SPT_OK || nnz == 0) return st;
      hipLaunchKernelGGL(coo_atomic_spmv_kernel<T>, dim3((unsigned)((nnz + kScatterEntries - 1) / kScatterEntries)),
                         dim3(kBlock), 0, s, (int)nnz, A->level[0].crd, A->level[1].crd, vals, x,
                         y);
      SPT_CHECK_LAUNCH("coo_atomic_spmv");
      return SPT_OK;
    }
    case Format::DIA: {
      const int64_t K = A->level[0].N, N = A->level[1].N, M = A->level[1].M;
      if (N == 0) return SPT_OK;
      if (K >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "spmv: too many diagonals");
      if (K == 0) return launch_fill<T>(y, N, T(0), s);
      constexpr int R = Entries<T>::K;
      if (M == 0) return launch_fill<T>(y, N, T(0), s);
      if (N >= R) {
        const int64_t lanes = (N + R - 1) / R;
        const dim3 grid((unsigned)((lanes + kBlock - 1) / kBlock));
        const int32_t* off = A->level[1].offset;
#define SPT_DIA_CASE(KT)                                                                                       \
  case KT:                                                                                                     \
    hipLaunchKernelGGL((dia_spmv_vec_kernel<T, KT>), grid, dim3(kBlock), 0, s, N, M, (int)K, off, vals, x, y); \
    break;
        switch (K <= 16 ? (int)K : 0) {
          SPT_DIA_CASE(1) SPT_DIA_CASE(2) SPT_DIA_CASE(3) SPT_DIA_CASE(4) SPT_DIA_CASE(5)
          SPT_DIA_CASE(6) SPT_DIA_CASE(7) SPT_DIA_CASE(8) SPT_DIA_CASE(9) SPT_DIA_CASE(10)
          SPT_DIA_CASE(11) SPT_DIA_CASE(12) SPT_DIA_CASE(13) SPT_DIA_CASE(14) SPT_DIA_CASE(15)
          SPT_DIA_CASE(16)
          default:
            hipLaunchKernelGGL((dia_spmv_vec_kernel<T, 0>), grid, dim3(kBlock), 0, s, N, M, (int)K, off, vals, x, y);
        }
#undef SPT_DIA_CASE
      } else {
        hipLaunchKernelGGL(dia_spmv_kernel<T>, dim3((unsigned)((N + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, N, M, (int)K, A->level[1].offset, vals, x, y);
      }
      SPT_CHECK_LAUNCH("dia_spmv");
      return SPT_OK;
    }
    case Format::ELL: {
      const int64_t Wd = A->level[0].N, N = A->level[1].N;
      if (N == 0) return SPT_OK;
      if (Wd >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "spmv: ELL width too large");
      constexpr int R = Entries<T>::K;
      if (Wd == 0 || A->level[2].N == 0) return launch_fill<T>(y, N, T(0), s);
      if (N >= R) {
        const int64_t waves = (N + kWave * R - 1) / (kWave * R);
        if (waves >= kEllWaves || Wd <= 8)
          hipLaunchKernelGGL((ell_spmv_vec_kernel<T, 1>), dim3((unsigned)((waves + 3) / 4)), dim3(kBlock), 0, s, N,
                             (int)Wd, A->level[2].crd, vals, x, y);
        else
          hipLaunchKernelGGL((ell_spmv_vec_kernel<T, 4>), dim3((unsigned)waves), dim3(kBlock), 0, s, N, (int)Wd,
                             A->level[2].crd, vals, x, y);
      } else {
        hipLaunchKernelGGL(ell_spmv_kernel<T>, dim3((unsigned)((N + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, N, (int)Wd, A->level[2].crd, vals, x, y);
      }
      SPT_CHECK_LAUNCH("ell_spmv");
      return SPT_OK;
    }
    default:
      return fail(SPT_ERR_UNSUPPORTED, "spmv: the tensor is not a CSR, COO, DIA or ELL matrix");
  }
}

// out[r] = sum over p in [pos[r], pos[r+1]) of vals[p] * x[crd[p]]: CSR SpMV, and
// equally TTV on the bottom level of a CSF tensor (rows = fibers).
spt_status csr_rows_reduce(int dtype, int64_t nnz, int64_t nrows, const int32_t* pos,
                           const int32_t* crd, const void* vals, const void* x, void* out,
                           void* ws, size_t ws_bytes, hipStream_t s) {
  // By entries: fibre lengths of a skewed tensor are far from their mean (hundreds of entries in the first
  // slices, single ones elsewhere). Few entries, where one launch is what counts, by rows if fibres are short on
  // average (50 000 entries, fp64: 7.4 instead of 11 us; 1M skewed ones take longer).
  if (nnz < (1 << 19) && csr_use_rows(nnz, nrows, 0, ws, ws_bytes)) {
    if (dtype == SPT_F64)
      return launch_csr_rows<double>(nnz, nrows, pos, crd, static_cast<const double*>(vals),
                                     DenseX<double>{static_cast<const double*>(x)}, static_cast<double*>(out), s);
    return launch_csr_rows<float>(nnz, nrows, pos, crd, static_cast<const float*>(vals),
                                  DenseX<float>{static_cast<const float*>(x)}, static_cast<float*>(out), s);
  }
  if (dtype == SPT_F64)
    return launch_seg<double, true>(nnz, nrows, pos, crd, static_cast<const double*>(vals),
                                    static_cast<const double*>(x), static_cast<double*>(out), ws,
                                    ws_bytes, s);
  return launch_seg<float, true>(nnz, nrows, pos, crd, static_cast<const float*>(vals),
                                 static_cast<const float*>(x), static_cast<float*>(out), ws, ws_bytes,
                                 s);
}

// ---- array-of-structs COO (Section 5.2): (row, col) pairs in one array ----

__global__ __launch_bounds__(kBlock) void split_pairs_kernel(int64_t n, const int32_t* __restrict__ rc,
                                                             int32_t* __restrict__ row,
                                                             int32_t* __restrict__ col) {
  const int64_t p = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (p >= n) return;
  row[p] = rc[2 * p];  // the two loads of a lane share 8 bytes, a wave reads 512 contiguous bytes
  col[p] = rc[2 * p + 1];
}

static size_t aos_pairs_bytes(const spt_tensor* A) { return 2 * align_up(static_cast<size_t>(A->nvals) * 4, 256); }
static size_t coo_least_workspace(const spt_tensor* A) {
  return (A->level[0].flags & SPT_ORDERED) ? ordered_coo_workspace(A->nvals)
                                           : coo_unordered_least(A->dtype, A->nvals, A->level[0].N);
}

size_t aos_coo_spmv_workspace(const spt_tensor* A) {
  return aos_pairs_bytes(A) + ((A->level[0].flags & SPT_ORDERED) ? ordered_coo_spmv_workspace(A)
                                                                 : coo_unordered_workspace(A->dtype, A->nvals, A->level[0].N));
}

// The least that spt_spmv takes where that is less than `query`, what spt_workspace_bytes answers.
bool is_aos_coo_matrix(const spt_tensor* T);
size_t spmv_least_workspace(Format f, const spt_tensor* A, size_t query) {
  if (f == Format::Unsupported && is_aos_coo_matrix(A)) return std::min(query, aos_pairs_bytes(A) + coo_least_workspace(A));
  if (f == Format::CSR) return std::min(query, seg_spmv_workspace(A->nvals));
  if (f == Format::COO2) return std::min(query, coo_least_workspace(A));
  if (f == Format::CSC) return std::min(query, csc_spmv_least(A));
  return query;
}

spt_status spmv_dispatch(Format f, const spt_tensor* A, const void* x, void* y, void* ws,
                         size_t ws_bytes, hipStream_t s);

// The pairs are split into a row and a column array in the workspace (8 bytes read and 8
// written per entry), then the COO kernels run on those.
spt_status aos_coo_spmv_dispatch(const spt_tensor* A, const void* x, void* y, void* ws,
                                 size_t ws_bytes, hipStream_t s) {
  const int64_t nnz = A->nvals;
  const size_t need = aos_pairs_bytes(A) + coo_least_workspace(A);
  if (nnz > 0 && (!ws || ws_bytes < need))
    return fail(SPT_ERR_WORKSPACE, "spmv: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  spt_tensor S = *A;
  S.level[0].crd_stride = S.level[1].crd_stride = 1;
  size_t used = 0;
  if (nnz > 0) {
    Workspace W(ws, ws_bytes);
    int32_t* row = W.take<int32_t>(nnz);
    int32_t* col = W.take<int32_t>(nnz);
    used = W.used;
    hipLaunchKernelGGL(split_pairs_kernel, dim3(static_cast<unsigned>((nnz + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, nnz, A->level[0].crd, row, col);
    SPT_CHECK_LAUNCH("split pairs");
    S.level[0].crd = row;
    S.level[1].crd = col;
  }
  return spmv_dispatch(Format::COO2, &S, x, y, ws ? static_cast<char*>(ws) + used : nullptr,
                       ws_bytes > used ? ws_bytes - used : 0, s);
}

spt_status spmv_dispatch(Format f, const spt_tensor* A, const void* x, void* y, void* ws,
                         size_t ws_bytes, hipStream_t s) {
  if (A->dtype == SPT_F64)
    return spmv_typed<double>(f, A, static_cast<const double*>(x), static_cast<double*>(y), ws,
                              ws_bytes, s);
  return spmv_typed<float>(f, A, static_cast<const float*>(x), static_cast<float*>(y), ws,
                           ws_bytes, s);
}

}  // namespace spt
