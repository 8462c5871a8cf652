// SpMV on CSR and ordered COO whose columns lie anywhere in an x that no L2 holds: x is gathered slice by slice.
//
// Entry after entry, such gathers miss L2, and the fabric brings 64 G lines of 128 bytes a second, whatever is
// used of them (60M entries, 4M columns, fp64: 57M lines, 0.95 ms). Here every compute unit holds 40 960 entries
// (fp32: 65 536) at a time, 40 per lane, in registers, and the chip sweeps over x in slices of 3.2 MB, which an L2 of 4 MB holds:
// in each, the entries whose column lies in it fetch their x, all others wait. A line of x is then brought to an
// XCD once per 1.3M of its entries instead of once per entry: 0.55 ms.
//  * The waves of a workgroup meet after each slice; the workgroups of an XCD keep together by themselves, since
//    the first to enter a slice wait for lines that the others then find. (Without the meeting 0.95 ms, the oldest
//    waves run ahead; with a barrier across the XCD before the sweep 0.71, with one between slices slower still.)
//  * Segments of 256 entries are dealt out across the matrix: a row of 10^5 entries lies in a few slices, and
//    workgroups of consecutive entries would drift apart (0.86 ms; 2048 consecutive entries per wave: 0.73).
//  * The number of workgroups is a multiple of the compute units, one of them to each (128 registers a lane): with
//    as many as there are full ones, the last round took as long as the others (0.71 against 0.68 ms).
//  * An offset's register becomes half of its value's, so that 40 entries fit where 32 with both did (8 rounds over x
//    become 6). Where that saves no rounds, lanes keep the 32 (slices_of_many); larger x have larger slices (slices_of).
// Bound by the address unit (a load with a few lanes takes it some 20 clocks), then the lines.
#include <algorithm>

#include "carry.hpp"
#include "common.hpp"
#include "slices.hpp"
#include "wavescan.hpp"

namespace spt {

constexpr int kSliceWaves = kSliceBlock / kWave;
constexpr int kFewSegments = kFewEntries / 4;
// Segments of a wave, each a vector of four entries per lane; and as many of them as have their row starts in LDS at a time (CSR).
template <typename T, bool MANY>
constexpr int kSegments = MANY ? kInPlace<T> / 4 : kFewSegments;
template <typename T, bool MANY>
constexpr int kRowBatch = MANY && sizeof(T) == 8 ? 6 : 8;

// What precedes the product, kChoiceFlags workgroups.
// CSR: does a block of kSkewRows rows hold more than 1 / kSkewShare of all entries? By rows, the kernel would end on
// the workgroup of one long row (10^5 entries keep it busy for about 0.1 ms). COO: y = 0.
// Both: do columns lie scattered? Each wave looks at a window of 256 entries: they do if they lie in 16 or more of
// 64 equal parts of x (random columns in about 63, seven diagonals in at most 14), and in parts of 4.4 MB or more, which no
// L2 holds. (Columns anywhere in a third of x that moves on with the row, without / with slices, in us: 2.7 MB, fp32, 36M
// entries, CSR 194 / 232, COO 228 / 260, 100M 557 / 589 and 599 / 696; 4 MB, fp32, 36M, 237 / 248 and 271 / 275; 4.8 MB, fp64,
// 36M, 294 / 279 and 312 / 292; 5.3 MB, fp32, 60M, 445 / 427 and 487 / 468, fp64, 100M, 811 / 734 and 860 / 776.)
// A window without a descending column lies inside a row and tells nothing: a long row's columns ascend slowly, and yet each is another line.
constexpr int kSkewShare = 1536, kSkewRows = 256, kScattered = 16;
constexpr int64_t kSpread = 4400000;
template <typename T, bool CSR>
__global__ __launch_bounds__(kSliceBlock) void slices_prepare_kernel(int nnz, int nrows, int ncols, int least_parts,
                                                                     const int32_t* __restrict__ pos,
                                                                     const int32_t* __restrict__ col, T* __restrict__ y,
                                                                     uint8_t* __restrict__ flags) {
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  __shared__ int s_heavy, s_tell, s_scattered;
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id(), b = blockIdx.x;
  if (tid == 0) s_heavy = s_tell = s_scattered = 0;
  __syncthreads();
  I4 c = 0;
  const bool look = col && nnz >= kSegment;  // uniform
  if (look) {
    const int64_t at = static_cast<int64_t>(nnz - kSegment) * (b * kSliceWaves + w) / (kChoiceFlags * kSliceWaves);
    c = *reinterpret_cast<const I4*>(col + at + lane * 4);
  }
  if (CSR) {
    const int nblocks = (nrows + kSkewRows - 1) / kSkewRows;
    bool heavy = false;
    for (int k = b * kSliceBlock + tid; k < nblocks; k += kChoiceFlags * kSliceBlock) {
      const int64_t e = pos[min((k + 1) * kSkewRows, nrows)] - pos[k * kSkewRows];
      heavy |= e * kSkewShare > nnz;
    }
    if (heavy) s_heavy = 1;
  } else {
    constexpr int R = 16 / sizeof(T);
    typedef T V __attribute__((ext_vector_type(R), aligned(sizeof(T))));
    for (int64_t e = (static_cast<int64_t>(b) * kSliceBlock + tid) * R; e < nrows; e += static_cast<int64_t>(kChoiceFlags) * kSliceBlock * R) {
      if (e + R <= nrows) *reinterpret_cast<V*>(y + e) = V(T(0));
      else
        for (int64_t q = e; q < nrows; ++q) y[q] = T(0);
    }
  }
  if (look) {
    const float parts = 64.0f / ncols;
    uint64_t in = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) in |= uint64_t{1} << min(static_cast<int>(c[q] * parts), 63);
    const int32_t left = __shfl_up(c[3], 1);
    const bool down = c[1] < c[0] || c[2] < c[1] || c[3] < c[2] || (lane > 0 && c[0] < left);
    const bool tells = __ballot(down) != 0;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) in |= __shfl_xor(in, d);
    if (lane == 0 && tells) {
      atomicAdd(&s_tell, 1);
      if (__popcll(in) >= least_parts) atomicAdd(&s_scattered, 1);
    }
  }
  __syncthreads();
  if (tid == 0) flags[b] = (s_heavy ? kChoiceHeavy : 0) | (2 * s_scattered > s_tell ? kChoiceScattered : 0) | (s_tell ? kChoiceTells : 0);
}

// Row starts of the segments where the row kernel is no candidate.
template <typename T>
__global__ __launch_bounds__(kBlock) void segment_rows_kernel(int nrows, const int32_t* __restrict__ pos, int nseg,
                                                              int32_t* __restrict__ seg_row, T* __restrict__ y) {
  find_segment_rows(nrows, pos, nseg, seg_row, y);
}

// The sums of a segment's rows, in registers: the segment that holds a row's first entry stores the row's sum, what
// precedes the first row start leaves as carry number `seg`. A lane has the entries lane * 4 .. lane * 4 + 3, those from
// `left_over` on do not count. rows: COO, their rows; CSR, the rows that start at them, or -1. cut: the row that
// the segment's start cuts. Fixed order of additions: bit-reproducible.
template <typename T, bool CSR, class V4, class I4>
__device__ __forceinline__ void reduce_segment(int seg, int left_over, int cut, const V4& v, const T* got, const I4& rows,
                                               T* __restrict__ y, int32_t* __restrict__ carry_key, T* __restrict__ carry_val) {
  const int lane = lane_id();
  int32_t before = cut;
  if (!CSR) {
    const int32_t left = dpp_move<0x138, 0xf>(-1, rows[3]);  // wave_shr:1
    if (lane > 0) before = left;
  }
  T acc = 0, lead = 0;
  bool has_head = false, head_first = false;
  int last_row = -1;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t r = rows[q];
    if (CSR ? r >= 0 : r != before) {
      if (has_head) y[last_row] = acc;  // a row that starts and ends inside this lane
      else lead = acc;
      head_first = head_first || q == 0;
      has_head = true;
      last_row = r;
      acc = 0;
    }
    acc += lane * 4 + q < left_over ? v[q] * got[q] : T(0);
    before = r;
  }
  const uint64_t marks = __ballot(has_head);
  const int from = last_lane(marks, false), prev_head = last_lane(marks, true);
  const T sum = wave_marked_sum<T>(acc, from >= 0 ? lane - from : kWave);
  T open = dpp_move<0x138, 0xf>(T(0), sum);  // what is open before this lane
  if (lane == 0) open = T(0);
  const int open_row = __shfl(last_row, max(prev_head, 0));
  if (has_head) {
    if (prev_head >= 0) {
      y[open_row] = open + lead;
    } else {  // what precedes the segment's first row start
      carry_key[seg] = lane == 0 && head_first ? -1 : cut;
      carry_val[seg] = open + lead;
    }
  }
  if (lane == kWave - 1) {  // the row still open at the end of the segment
    if (from >= 0) {
      y[has_head ? last_row : open_row] = sum;
    } else {
      carry_key[seg] = cut;
      carry_val[seg] = sum;
    }
  }
}

// CSR, for a segment with more than kMany row starts (mostly of rows without entries): the row of each entry is looked up
// in rows l .. h - 1, which start in it. from: its first entry.
constexpr int kMany = 256;
__device__ __forceinline__ void look_up_rows(int l, int h, int from, int nnz, const int32_t* __restrict__ pos, int32_t* heads) {
  const int lane = lane_id();
  int r[4], end[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    r[q] = l - 1;
    end[q] = h;
  }
  for (int span = h - l + 1; span > 1; span = (span + 1) / 2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int mid = r[q] + (end[q] - r[q]) / 2;
      if (mid > r[q]) {
        if (pos[mid] - from <= lane * 4 + q) r[q] = mid;
        else end[q] = mid;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (r[q] >= l && lane * 4 + q < nnz - from && pos[r[q]] - from == lane * 4 + q) heads[lane * 4 + q] = r[q];
}

// Columns that do not lie scattered (the device's choice): x is gathered as the entries come, and kCus workgroups go
// through the segments in order, an eighth of them on each XCD (a stretch to each workgroup: ordered COO, 60M, fp64
// 256 us, fp32 174). A wave waits for no other, and has the gathers of the next segment and the columns of the one after
// that on their way while it adds up one (gathers when their turn comes: up to 4 % longer). Bound by memory, 4.2 TB/s.
// Whole call, local columns, in us, with all entries of a wave at once as for slices / a kernel of chunks in LDS without
// a choice before it / this way:
//   entries              18M              25M               36M               40M               50M              74M
//   COO, fp64        84 / 81 / 80   112 / 113 / 104   156 / 148 / 148   175 / 164 / 166   214 / 202 / 202   296 / 275 / 280
//   COO, fp32        64 / 55 / 57    82 / 73 / 72     115 / 102 / 106   128 / 113 / 115   158 / 141 / 139   212 / 182 / 178
//   CSR, a heavy row,                                 148 / 171 / 138   161 / 191 / 150   193 / 231 / 181   253 / 309 / 228
//     fp64 and fp32                                   116 / 112 / 110   125 / 124 / 115   146 / 149 / 133   184 / 193 / 157
template <typename T, bool CSR>
__device__ __forceinline__ void segments_in_order(int nnz, int nseg, const int32_t* __restrict__ pos_or_row,
                                                  const int32_t* __restrict__ col, const T* __restrict__ vals,
                                                  const T* __restrict__ x, T* __restrict__ y, const int32_t* __restrict__ seg_row,
                                                  int32_t* __restrict__ carry_key, T* __restrict__ carry_val, int32_t* heads) {
  typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  if (blockIdx.x >= kCus) return;
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  // an XCD has an eighth of the segments, its workgroups side by side
  constexpr int kStep = kCus / kXcds * kSliceWaves;
  const int per = (nseg + kXcds - 1) / kXcds, xcd = blockIdx.x % kXcds, limit = min((xcd + 1) * per, nseg);
  struct Entries {
    I4 r;           // COO: rows
    V4 v;
    T got[4];
    int32_t prior;  // COO: row of the entry before the segment
    int lo, hi;     // CSR: the rows that start in the segment,
    int a, b;       // and where the first 64 of them begin and end
  };
  const auto load_columns = [&](int seg) {
    const int64_t p = static_cast<int64_t>(seg) * kSegment;
    I4 c;
    if (p + kSegment <= nnz) {  // uniform
      c = __builtin_nontemporal_load(reinterpret_cast<const I4*>(col + p + lane * 4));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) c[q] = p + lane * 4 + q < nnz ? col[p + lane * 4 + q] : 0;  // beyond the end: not counted
    }
    return c;
  };
  const auto load_bounds = [&](int seg, Entries& e) {
    e.lo = seg_row[seg];
    e.hi = seg_row[seg + 1];
  };
  const auto gather = [&](const I4& c, Entries& e) {
#pragma unroll
    for (int q = 0; q < 4; ++q) e.got[q] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(x) + static_cast<uint32_t>(c[q]) * sizeof(T));
  };
  const auto load = [&](int seg, Entries& e) {
    const int64_t p = static_cast<int64_t>(seg) * kSegment;
    if (p + kSegment <= nnz) {  // uniform
      e.v = __builtin_nontemporal_load(reinterpret_cast<const V4*>(vals + p + lane * 4));
      if (!CSR) e.r = __builtin_nontemporal_load(reinterpret_cast<const I4*>(pos_or_row + p + lane * 4));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t at = p + lane * 4 + q < nnz ? p + lane * 4 + q : nnz - 1;
        e.v[q] = vals[at];
        if (!CSR) e.r[q] = pos_or_row[at];
      }
    }
    if (CSR) {
      const int r = min(e.lo + lane, max(e.hi - 1, e.lo));  // (no row: nothing behind the end of pos is read)
      e.a = pos_or_row[r];
      e.b = pos_or_row[min(r + 1, max(e.hi, e.lo))];
    } else {
      e.prior = seg > 0 ? pos_or_row[p - 1] : -1;
    }
  };
  int seg = xcd * per + static_cast<int>(blockIdx.x) / kXcds * kSliceWaves + w;
  if (seg >= limit) return;
  Entries now{}, next{};
  I4 c = load_columns(seg);  // of the segment that is gathered next
  if (CSR) load_bounds(seg, now);
  gather(c, now);
  load(seg, now);
  if (seg + kStep < limit) {
    c = load_columns(seg + kStep);
    if (CSR) load_bounds(seg + kStep, next);
  }
  for (; seg < limit; seg += kStep) {
    const int after = seg + kStep;
    Entries later{};
    if (after < limit) {  // uniform
      gather(c, next);
      load(after, next);
      if (after + kStep < limit) {
        c = load_columns(after + kStep);
        if (CSR) load_bounds(after + kStep, later);
      }
    }
    I4 rows = now.r;
    if (CSR) {
      *reinterpret_cast<I4*>(heads + lane * 4) = I4(-1);
      wave_lds_order();
      const int base = seg * kSegment;
      if (now.hi - now.lo > kMany) {
        look_up_rows(now.lo, now.hi, base, nnz, pos_or_row, heads);
      } else {
        if (now.lo + lane < now.hi && now.b > now.a) heads[now.a - base] = now.lo + lane;
        for (int r = now.lo + kWave + lane; r < now.hi; r += kWave) {
          const int a = pos_or_row[r], b = pos_or_row[r + 1];
          if (b > a) heads[a - base] = r;
        }
      }
      wave_lds_order();
      rows = *reinterpret_cast<const I4*>(heads + lane * 4);
      wave_lds_order();
    }
    reduce_segment<T, CSR>(seg, nnz - seg * kSegment, CSR ? now.lo - 1 : now.prior, now.v, now.got, rows, y, carry_key,
                           carry_val);
    now = next;
    next = later;
  }
}

// x slice by slice, all segments of a wave at once. CSR: the rows that start in a segment are entered at their first entry
// in LDS.
template <typename T, bool CSR, bool MANY>
__global__ __launch_bounds__(kSliceBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void slices_spmv_kernel(
    int nnz, int nseg, int nslices, int slice, bool rows_may, const int32_t* __restrict__ pos_or_row, const int32_t* __restrict__ col,
    const T* __restrict__ vals, const T* __restrict__ x, T* __restrict__ y, const int32_t* __restrict__ seg_row,
    int32_t* __restrict__ carry_key, T* __restrict__ carry_val, const uint8_t* __restrict__ flags) {
  constexpr int V = kSegments<T, MANY>, B = kRowBatch<T, MANY>;
  typedef T V4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  extern __shared__ __attribute__((aligned(16))) int32_t s_rows[];  // CSR: the row that starts at an entry, or -1
  const int choice = read_choice(flags);
  if (rows_may && choice == kByRows) return;
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  int32_t* heads = s_rows + w * (B * kSegment);
  if (choice != kBySlices) {
    segments_in_order<T, CSR>(nnz, nseg, pos_or_row, col, vals, x, y, seg_row, carry_key, carry_val, heads);
    return;
  }
  // segment of vector j: first + j * step, none from nseg on
  const int step = kSliceWaves * gridDim.x, first = w * gridDim.x + blockIdx.x;

  T got[4 * V];
  uint32_t offset[4 * V];
  constexpr uint32_t kNowhere = 0xFFFFFFFFu;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const int seg = first + j * step;
    const int64_t p = static_cast<int64_t>(seg) * kSegment;
    if (seg < nseg && p + kSegment <= nnz) {  // uniform
      const I4 c = __builtin_nontemporal_load(reinterpret_cast<const I4*>(col + p + lane * 4));
#pragma unroll
      for (int q = 0; q < 4; ++q) offset[4 * j + q] = static_cast<uint32_t>(c[q]) * sizeof(T);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t e = p + lane * 4 + q;
        offset[4 * j + q] = seg < nseg && e < nnz ? static_cast<uint32_t>(col[e]) * sizeof(T) : kNowhere;
      }
    }
  }
  if constexpr (MANY) {
#pragma unroll
    for (int k = 0; k < 4 * V; ++k) {
      if constexpr (sizeof(T) == 8) got[k] = __hiloint2double(0, static_cast<int>(offset[k]));
      else got[k] = __uint_as_float(offset[k]);
    }
    SliceGatherInPlace<T>::run(x, nslices, slice, got);
  } else {
#pragma unroll
    for (int k = 0; k < 4 * V; ++k) got[k] = 0;
    SliceGather<T, 4 * V>::run(x, nslices, slice, offset, got);
  }

  // Segments whose values (COO: and rows) are on their way at a time. Next to 40 gathered doubles there is room for those of
  // two, as long as entries are counted in 32 bits (in 64, a lane's four places took eight registers and 2 others went through
  // scratch memory), of COO for those of one (with two, 6 and 2 registers). 60M entries, x of 32 MB, us, with scratch memory / one / two:
  // CSR, power law 543 / 545 / 541, even rows 528 / 518 / 522; COO 543 / 537 /  -, 560 / 553 /  -.
  constexpr int kBatch = sizeof(T) == 8 ? (MANY && !CSR ? 1 : 2) : 4;
  static_assert(B % kBatch == 0 && V % kBatch == 0, "");
  int r_first = 0;  // CSR, in lane l: the first row that starts in segment l / L of those in LDS
  constexpr int L = kWave / B;  // lanes that enter the rows of a segment
#pragma unroll
  for (int h = 0; h < V; h += kBatch) {
    if (CSR && h % B == 0) {
      const int j = lane / L, seg = first + (h + j) * step, base = seg * kSegment;
      const bool live = j < B && h + j < V && seg < nseg;
      const int lo = live ? seg_row[seg] : 0, hi = live ? seg_row[seg + 1] : 0;
#pragma unroll
      for (int u = 0; u < B; ++u) *reinterpret_cast<I4*>(heads + u * kSegment + lane * 4) = I4(-1);
      wave_lds_order();  // other lanes enter rows over what a lane has cleared
      const bool many = hi - lo > kMany;
      if (!many) {
        for (int r = lo + lane % L; r < hi; r += L) {
          const int a = pos_or_row[r], b = pos_or_row[r + 1];
          if (b > a) heads[j * kSegment + a - base] = r;
        }
      }
      uint64_t todo = __ballot(many && lane % L == 0);
      while (todo) {
        const int src = __ffsll(static_cast<long long>(todo)) - 1;
        todo &= todo - 1;
        look_up_rows(__builtin_amdgcn_readlane(lo, src), __builtin_amdgcn_readlane(hi, src), __builtin_amdgcn_readlane(base, src), nnz,
                     pos_or_row, heads + __builtin_amdgcn_readlane(j, src) * kSegment);
      }
      wave_lds_order();  // and other lanes again read them
      r_first = lo;
    }
    V4 v[kBatch];
    I4 rows[kBatch];
    int32_t prior[kBatch];  // COO: row of the entry before the segment
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int seg = first + (h + j) * step;
      const int64_t p = static_cast<int64_t>(seg) * kSegment;
      if (seg < nseg && p + kSegment <= nnz) {  // uniform
        v[j] = __builtin_nontemporal_load(reinterpret_cast<const V4*>(vals + p + lane * 4));
        if (!CSR) rows[j] = __builtin_nontemporal_load(reinterpret_cast<const I4*>(pos_or_row + p + lane * 4));
      } else if (seg < nseg) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t e = p + lane * 4 + q;
          v[j][q] = e < nnz ? vals[e] : T(0);
          if (!CSR) rows[j][q] = pos_or_row[e < nnz ? e : nnz - 1];
        }
      }
      if (!CSR) prior[j] = seg > 0 && seg < nseg ? pos_or_row[p - 1] : -1;
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int seg = first + (h + j) * step;
      if (seg >= nseg) break;  // uniform
      if (CSR) rows[j] = *reinterpret_cast<const I4*>(heads + (h + j) % B * kSegment + lane * 4);
      reduce_segment<T, CSR>(seg, nnz - seg * kSegment,
                             CSR ? __builtin_amdgcn_readlane(r_first, (h + j) % B * L) - 1 : prior[j], v[j], got + 4 * (h + j), rows[j], y,
                             carry_key, carry_val);
    }
    if (CSR) wave_lds_order();  // the next batch clears what lanes have read
  }
}

struct SlicesWorkspace {
  int nseg;
  uint8_t* flags;
  int32_t *seg_row, *carry_key;
  void* carry_val;
  size_t bytes;
  SlicesWorkspace(int64_t nnz, void* ws) {
    nseg = (int)((nnz + kSegment - 1) / kSegment);
    Workspace W(ws, 0);
    flags = W.take<uint8_t>(kChoiceFlags);
    seg_row = W.take<int32_t>((size_t)nseg + 1);
    carry_key = W.take<int32_t>(nseg);
    carry_val = W.take<double>(nseg);
    bytes = W.used;
  }
};
size_t slices_spmv_workspace(int64_t nnz) { return SlicesWorkspace(nnz, nullptr).bytes; }
ByRowsIf slices_by_rows_if(int64_t nnz, void* ws) {
  const SlicesWorkspace W(nnz, ws);
  return {W.flags, W.seg_row, W.nseg};
}
template <typename T>
spt_status launch_segment_rows(int64_t nnz, int64_t nrows, const int32_t* pos, T* y, void* ws, hipStream_t s) {
  const SlicesWorkspace W(nnz, ws);
  hipLaunchKernelGGL(segment_rows_kernel<T>, dim3((unsigned)std::min<int64_t>((nrows + kBlock - 1) / kBlock, 4096)),
                     dim3(kBlock), 0, s, (int)nrows, pos, W.nseg, W.seg_row, y);
  SPT_CHECK_LAUNCH("segment rows");
  return SPT_OK;
}

template <typename T, bool CSR>
spt_status launch_slices_prepare(int64_t nnz, int64_t nrows, int64_t ncols, const int32_t* pos, const int32_t* col, T* y,
                                 void* ws, hipStream_t s) {
  const SlicesWorkspace W(nnz, ws);
  const int64_t x = ncols * (int64_t)sizeof(T);
  const int least_parts = (int)std::max<int64_t>(kScattered, (64 * kSpread + x - 1) / x);
  hipLaunchKernelGGL((slices_prepare_kernel<T, CSR>), dim3(kChoiceFlags), dim3(kSliceBlock), 0, s, (int)nnz, (int)nrows,
                     (int)ncols, least_parts, pos, col, y, W.flags);
  SPT_CHECK_LAUNCH("slices prepare");
  return SPT_OK;
}
// Only whether a block of rows is heavy, CSR.
spt_status launch_csr_skew(int64_t nnz, int64_t nrows, const int32_t* pos, uint8_t* flags, hipStream_t s) {
  hipLaunchKernelGGL((slices_prepare_kernel<float, true>), dim3(kChoiceFlags), dim3(kSliceBlock), 0, s, (int)nnz, (int)nrows, 1, 0,
                     pos, nullptr, nullptr, flags);
  SPT_CHECK_LAUNCH("csr skew");
  return SPT_OK;
}
template <typename T, bool CSR>
spt_status launch_slices_spmv(int64_t nnz, int64_t ncols, bool rows_may, const int32_t* pos_or_row, const int32_t* col,
                              const T* vals, const T* x, T* y, void* ws, hipStream_t s) {
  const SlicesWorkspace W(nnz, ws);
  const bool many = slices_of_many<T>(nnz, ncols, CSR);
  const int per = kSliceWaves * (many ? kSegments<T, true> : kFewSegments);
  const int nslices = slices_of(ncols, sizeof(T), int64_t(per) * kSegment * kCus);
  const uint32_t slice = (uint32_t)((ncols + nslices - 1) / nslices * sizeof(T));
  const int grid = ((W.nseg + per - 1) / per + kCus - 1) / kCus * kCus;
  T* cval = static_cast<T*>(W.carry_val);
  const int lds = CSR ? kSliceWaves * kSegment * 4 * (many ? kRowBatch<T, true> : kRowBatch<T, false>) : 0;
#define SPT_SLICES_SPMV(MANY_)                                                                                        \
  hipLaunchKernelGGL((slices_spmv_kernel<T, CSR, MANY_>), dim3(grid), dim3(kSliceBlock), lds, s, (int)nnz, W.nseg,     \
                     nslices, (int)slice, rows_may, pos_or_row, col, vals, x, y, W.seg_row, W.carry_key, cval, W.flags)
  if (many) SPT_SLICES_SPMV(true);
  else SPT_SLICES_SPMV(false);
#undef SPT_SLICES_SPMV
  SPT_CHECK_LAUNCH("slices_spmv");
  hipLaunchKernelGGL((carry_fixup_kernel<T, 16>), dim3((W.nseg + kBlock - 1) / kBlock), dim3(kBlock), 0, s, W.nseg, W.carry_key, cval,
                     y, rows_may ? W.flags : nullptr, 1);
  SPT_CHECK_LAUNCH("carry_fixup");
  return SPT_OK;
}
#define SPT_SLICES(T, C)                                                                                              \
  template spt_status launch_slices_prepare<T, C>(int64_t, int64_t, int64_t, const int32_t*, const int32_t*, T*,       \
                                                  void*, hipStream_t);                                                \
  template spt_status launch_slices_spmv<T, C>(int64_t, int64_t, bool, const int32_t*, const int32_t*, const T*,      \
                                               const T*, T*, void*, hipStream_t);
template spt_status launch_segment_rows<double>(int64_t, int64_t, const int32_t*, double*, void*, hipStream_t);
template spt_status launch_segment_rows<float>(int64_t, int64_t, const int32_t*, float*, void*, hipStream_t);
SPT_SLICES(double, true) SPT_SLICES(double, false) SPT_SLICES(float, true) SPT_SLICES(float, false)
#undef SPT_SLICES

}  // namespace spt
