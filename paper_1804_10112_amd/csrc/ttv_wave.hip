// TTV A_ij = sum_k B_ijk c_k (Section 5.3): COO, and CSF tensors of many entries. In pieces of 256
// entries per wave; for large tensors the vector c is held in LDS.
//
// Every stored entry gathers one c_k. With c in global memory those gathers, not the
// streams of coordinates and values, set the pace (they hit L2, but a wave's 64 distinct
// lines take several clocks each through the vector memory path). Here one workgroup of
// sixteen waves stays on every compute unit, copies c (as much of it as fits) into LDS once,
// and its waves then walk through the entries on their own, 256 consecutive entries (four
// per lane, one 16-byte load per array) at a time, two such pieces in flight:
//   - products with c from LDS (entries whose k lies beyond the cached part read global c);
//   - fibre heads: COO compares (i, j) with the entry before; CSF marks the entries at which
//     the fibres of the piece begin (from pos of the bottom level) in a wave-private strip
//     of LDS;
//   - a segmented sum over the wave in registers (lane movement inside the vector ALU), no
//     workgroup barrier anywhere in the loop, so a wave waiting for memory never holds up
//     another.
// Output: the piece that holds a fibre's first entry
// stores the fibre's (possibly partial) sum; what precedes the first head of a piece leaves
// as carry number `piece` and is added afterwards (carry_fixup_kernel), in a fixed order:
// results are bit-reproducible.
// Measured on 50M entries in 8.1M fibres, fp32, c of 50 000 values (78 % / 61 % of it cached):
// COO 229 us in all, call after call on the same operands (count of the heads 40, their offsets 5, this kernel 185, carries
// 5; 248 us where operands change from call to call), CSF 157 us (workgroups of 2048 entries
// with c in global memory: 324 and 357 us). Left out
// after measuring: eight entries per lane (a lane's two 16-byte loads then lie 32 bytes apart:
// 263 / 174 us, against 214 / 158 then), four pieces in flight instead of two or the next two loaded ahead (no change), results
// put in order in LDS before they are stored (dense fibres 12 % faster, skewed tensors 2 to 5 % slower). What remains is the serial
// instruction stream of a wave: sixteen waves per compute unit is all that one workgroup, which
// the single copy of c forces, can provide.
#include "carry.hpp"
#include "common.hpp"
#include "scan.hpp"
#include "segreduce.hpp"
#include "search.hpp"
#include "wavescan.hpp"

namespace spt {

constexpr int kBig = 1024;                    // threads per workgroup
constexpr int kBigWaves = kBig / kWave;
constexpr int kEPL = 4;                       // consecutive entries per lane
constexpr int kPiece = kEPL * kWave;          // entries of one piece
constexpr int kNP = 2;                        // pieces a wave has in flight per step
constexpr int kCooCacheBytes = 152 * 1024;    // LDS set aside for c (COO: nothing else lives there)
constexpr int kCsfCacheBytes = 120 * 1024;    // CSF: next to 32 KiB of fibre marks

template <typename T>
__device__ __forceinline__ T ld_nt(const T* p) {
  return __builtin_nontemporal_load(p);
}

typedef int32_t int4v __attribute__((ext_vector_type(4)));

// Four consecutive values as 16-byte loads.
__device__ __forceinline__ void load4(const float* p, float (&v)[4]) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 q = ld_nt(reinterpret_cast<const f4*>(p));
  v[0] = q[0], v[1] = q[1], v[2] = q[2], v[3] = q[3];
}
__device__ __forceinline__ void load4(const double* p, double (&v)[4]) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const d2 a = ld_nt(reinterpret_cast<const d2*>(p)), b = ld_nt(reinterpret_cast<const d2*>(p) + 1);
  v[0] = a[0], v[1] = a[1], v[2] = b[0], v[3] = b[1];
}
__device__ __forceinline__ void load4(const int32_t* p, int32_t (&v)[4]) {
  const int4v q = ld_nt(reinterpret_cast<const int4v*>(p));
  v[0] = q[0], v[1] = q[1], v[2] = q[2], v[3] = q[3];
}

// Four consecutive values of any alignment.
template <typename E>
__device__ __forceinline__ void load_any(const E* p, E (&v)[4]) {
  typedef E V4 __attribute__((ext_vector_type(4), aligned(sizeof(E))));
  const V4 q = __builtin_nontemporal_load(reinterpret_cast<const V4*>(p));
  v[0] = q[0], v[1] = q[1], v[2] = q[2], v[3] = q[3];
}

// kEPL consecutive values or coordinates, 16 bytes per load.
template <typename E>
__device__ __forceinline__ void load_lane(const E* p, E (&v)[kEPL]) {
#pragma unroll
  for (int h = 0; h < kEPL / 4; ++h) {
    E q[4];
    load4(p + 4 * h, q);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[4 * h + r] = q[r];
  }
}

// The workgroup copies c[0 .. cached) into LDS.
template <typename T>
__device__ __forceinline__ void stage_vector(T* s_c, const T* __restrict__ c, int cached) {
  constexpr int U = 8;  // loads in flight per thread: the copy is one round trip per U * kBig values
  int q = threadIdx.x;
  for (; q + (U - 1) * kBig < cached; q += U * kBig) {
    T t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = c[q + u * kBig];
#pragma unroll
    for (int u = 0; u < U; ++u) s_c[q + u * kBig] = t[u];
  }
  for (; q < cached; q += kBig) s_c[q] = c[q];
  __syncthreads();
}

// c_k: from LDS below `cached`, from global memory beyond. ALL: everything is cached.
template <typename T, bool ALL>
__device__ __forceinline__ void gather_lane(const T* s_c, const T* __restrict__ c, int cached,
                                            const int32_t (&k)[kEPL], T (&g)[kEPL]) {
#pragma unroll
  for (int r = 0; r < kEPL; ++r) g[r] = s_c[ALL ? k[r] : min(k[r], cached - 1)];
  if (!ALL) {
#pragma unroll
    for (int r = 0; r < kEPL; ++r)
      if (k[r] >= cached) g[r] = c[k[r]];
  }
}

// The last piece: nothing is added for lanes beyond the last entry, whose c may be infinite (their value is 0).
template <typename T>
__device__ __forceinline__ void drop_beyond(int p0, int nnz, T (&g)[kEPL]) {
#pragma unroll
  for (int r = 0; r < kEPL; ++r)
    if (p0 + r >= nnz) g[r] = T(0);
}

// A lane holds the products p[0 .. kEPL) of its consecutive entries; bit r of headmask says
// that a fibre starts at entry r, key[r] is then that fibre's index in the output.
// Stores the sums of the fibres that start in this piece, and the piece's carry.
template <typename T>
__device__ __forceinline__ void wave_fibre_sums(const T (&p)[kEPL], unsigned headmask, const int (&key)[kEPL],
                                                int carry_idx, int piece, T* __restrict__ out_v,
                                                int32_t* __restrict__ carry_key, T* __restrict__ carry_val) {
  const int lane = lane_id();
  T acc = 0, lead = 0;
  int has_head = 0, last_key = -1;
#pragma unroll
  for (int r = 0; r < kEPL; ++r) {
    if (headmask & (1u << r)) {
      if (!has_head) {
        lead = acc;
        has_head = 1;
      } else {
        out_v[last_key] = acc;
      }
      last_key = key[r];
      acc = 0;
    }
    acc += p[r];
  }
  SegSum<T> me{has_head, acc, last_key};
  wave_seg_step<0x111, 0xf>(me);  // row_shr:1, 2, 4, 8: scan inside each row of 16 lanes
  wave_seg_step<0x112, 0xf>(me);
  wave_seg_step<0x114, 0xf>(me);
  wave_seg_step<0x118, 0xf>(me);
  wave_seg_step<0x142, 0xa>(me);  // row_bcast:15 into rows 1 and 3
  wave_seg_step<0x143, 0xc>(me);  // row_bcast:31 into rows 2 and 3
  SegSum<T> ex;  // what the lanes before this one add up to
  ex.f = dpp_move<0x138, 0xf>(0, me.f);  // wave_shr:1
  ex.v = dpp_move<0x138, 0xf>(T(0), me.v);
  ex.k = dpp_move<0x138, 0xf>(-1, me.k);
  if (lane == 0) ex = SegSum<T>{0, T(0), -1};
  if (has_head) {
    const T total = ex.v + lead;
    if (ex.f) {
      out_v[ex.k] = total;
    } else {  // first head of the piece: what precedes it continues an earlier piece
      carry_key[piece] = (lane == 0 && (headmask & 1u)) ? -1 : carry_idx;
      carry_val[piece] = total;
    }
  }
  if (lane == kWave - 1) {  // the fibre still open at the end of the piece
    if (has_head) {
      out_v[last_key] = acc;
    } else if (ex.f) {
      out_v[ex.k] = ex.v + acc;
    } else {  // no head in the whole piece: everything is carry
      carry_key[piece] = carry_idx;
      carry_val[piece] = ex.v + acc;
    }
  }
}

// ================================================================ COO
// piece_off[piece] = (i, j) fibre starts in the pieces before among the workgroup's, group_off[workgroup] = in all of
// them. Bound by reading i and j; i is ordered, so where it is the same before and at the end of a piece
// it need not be read. A wave has the loads of its pieces in flight together: four, of many entries eight (whole call,
// fp32, with four / eight: 12M entries 57 / 59 us, 24M 127 / 127, 26M 133 / 134, 50M 238 / 229 (this kernel 52 / 40, since then 34), 50M of
// one entry to a fibre 501 / 494; 16: 62, 130 and, 50M, 245).
// SELF (few pieces): one piece for a wave, piece_off[piece] = the starts in it.
constexpr int kLogGroup = 4, kLogGroupMany = 5, kManyPieces = 96 * 1024;
template <bool VEC, bool SELF, int LOG_GROUP>
__global__ __launch_bounds__(kBlock) void ttv_piece_heads_kernel(int nnz, int npieces,
                                                                 const int32_t* __restrict__ ci,
                                                                 const int32_t* __restrict__ cj,
                                                                 int32_t* __restrict__ piece_off,
                                                                 int32_t* __restrict__ group_off) {
  constexpr int kPieces = SELF ? kBlock / kWave : 1 << LOG_GROUP, OWN = kPieces / (kBlock / kWave);
  __shared__ int s_heads[kPieces];
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
  int32_t i[OWN][kEPL], j[OWN][kEPL], bi[OWN], bj[OWN], ei[OWN];
  int base[OWN];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    base[u] = min(static_cast<int>(blockIdx.x) * kPieces + w * OWN + u, npieces - 1) * kPiece;
    const int p0 = base[u] + lane * kEPL, before = max(base[u] - 1, 0);
    if (VEC && base[u] + kPiece <= nnz) {  // uniform
      load_lane(cj + p0, j[u]);
    } else {
#pragma unroll
      for (int r = 0; r < kEPL; ++r) j[u][r] = cj[min(p0 + r, nnz - 1)];  // beyond the end: the last entry again, never a head
    }
    if (u == 0) {
      bi[u] = ci[before];
      bj[u] = cj[before];
    }
  }
  // the pieces of a wave lie in one slice, most of them: one look at i for all (a look at both ends of each piece takes a
  // line of i per KB: 50M entries 43 us, so 34)
  const bool one = bi[0] == ci[min(base[OWN - 1] + kPiece, nnz) - 1];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int p0 = base[u] + lane * kEPL;
    if (u > 0) {
      bj[u] = __builtin_amdgcn_readlane(j[u - 1][kEPL - 1], kWave - 1);  // (the piece before; of pieces beyond the end, not stored)
      bi[u] = one ? bi[0] : ci[max(base[u] - 1, 0)];
    }
    ei[u] = one ? bi[0] : ci[min(base[u] + kPiece, nnz) - 1];
    if (bi[u] == ei[u]) {  // uniform
#pragma unroll
      for (int r = 0; r < kEPL; ++r) i[u][r] = bi[u];
    } else if (VEC && base[u] + kPiece <= nnz) {
      load_lane(ci + p0, i[u]);
    } else {
#pragma unroll
      for (int r = 0; r < kEPL; ++r) i[u][r] = ci[min(p0 + r, nnz - 1)];
    }
  }
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    int32_t pi = dpp_move<0x138, 0xf>(bi[u], i[u][kEPL - 1]), pj = dpp_move<0x138, 0xf>(bj[u], j[u][kEPL - 1]);  // wave_shr:1
    if (base[u] == 0 && lane == 0) pi = pj = -1;
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
      cnt += __popcll(__ballot(i[u][r] != pi || j[u][r] != pj));
      pi = i[u][r];
      pj = j[u][r];
    }
    const int piece = blockIdx.x * kPieces + w * OWN + u;
    if (SELF) {
      if (lane == 0 && piece < npieces) piece_off[piece] = cnt;
      return;
    }
    if (lane == 0) s_heads[w * OWN + u] = piece < npieces ? cnt : 0;
  }
  __syncthreads();
  if (w == 0) {
    const int heads = lane < kPieces ? s_heads[lane] : 0, upto = wave_inclusive_sum(heads);
    const int piece = blockIdx.x * kPieces + lane;
    if (lane < kPieces && piece < npieces) piece_off[piece] = upto - heads;
    if (lane == kPieces - 1) group_off[blockIdx.x] = upto;
  }
}

// The heads of the groups become those of the groups before, in one workgroup (50M entries: 4 us; a scan over all
// pieces takes 11 in two launches).
__global__ __launch_bounds__(1024) void ttv_group_off_kernel(int ngroups, int32_t* __restrict__ group_off) {
  block_exclusive_scan<1024>(group_off, ngroups, 0);
}

// One output entry per fibre, at index group_off + piece_off[piece] + rank of the fibre's head inside
// the piece (append order = ascending (i, j), Section 3.4).
template <typename T, bool VEC, bool ALL>
__global__ __launch_bounds__(kBig) void ttv_coo_wave_kernel(
    int nnz, int npieces, const int32_t* __restrict__ ci, const int32_t* __restrict__ cj,
    const int32_t* __restrict__ ck, const T* __restrict__ vals, const T* __restrict__ c, int cached,
    const int32_t* __restrict__ piece_off, const int32_t* __restrict__ group_off, int log_group, int32_t* __restrict__ out_i, int32_t* __restrict__ out_j,
    T* __restrict__ out_v, int64_t* __restrict__ out_nnz, int32_t* __restrict__ carry_key,
    T* __restrict__ carry_val) {
  __shared__ T s_c[kCooCacheBytes / sizeof(T)];
  stage_vector(s_c, c, cached);
  const int lane = lane_id();
  const int stride = gridDim.x * kBigWaves;
  // piece number = step * (all waves of the grid) + wave: in one step the grid reads one
  // contiguous stretch of every array. A wave has kNP pieces in flight: all their loads are
  // issued before the first is used.
  // the piece number is the same in all lanes: held in a scalar register, what is indexed by it
  // alone (piece_off, the entry before the piece) is fetched by scalar loads
  for (int piece0 = __builtin_amdgcn_readfirstlane(blockIdx.x * kBigWaves + wave_id()); piece0 < npieces;
       piece0 += kNP * stride) {
    int32_t i[kNP][kEPL], j[kNP][kEPL], k[kNP][kEPL], pi[kNP], pj[kNP], first[kNP];
    T v[kNP][kEPL];
#pragma unroll
    for (int u = 0; u < kNP; ++u) {
      const int piece = min(piece0 + u * stride, npieces - 1);  // beyond the end: the last piece again, not stored
      const int p0 = piece * kPiece + lane * kEPL;
      const int before = max(piece * kPiece - 1, 0);  // only lane 0 uses it
      pi[u] = ci[before];
      pj[u] = cj[before];
      if (VEC && (piece + 1) * kPiece <= nnz) {  // uniform
        load_lane(cj + p0, j[u]);
        load_lane(ck + p0, k[u]);
        load_lane(vals + p0, v[u]);
        if (pi[u] == ci[piece * kPiece + kPiece - 1]) {
#pragma unroll
          for (int r = 0; r < kEPL; ++r) i[u][r] = pi[u];
        } else {
          load_lane(ci + p0, i[u]);
        }
      } else {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
          const bool ok = p0 + r < nnz;
          const int p = ok ? p0 + r : nnz - 1;  // beyond the end: the last entry's fibre, value 0
          i[u][r] = ci[p];
          j[u][r] = cj[p];
          k[u][r] = ck[p];
          v[u][r] = ok ? vals[p] : T(0);
        }
      }
      first[u] = piece_off[piece] + group_off[piece >> log_group];
    }
#pragma unroll
    for (int u = 0; u < kNP; ++u) {
      const int piece = piece0 + u * stride;
      if (piece >= npieces) break;
      int32_t qi = __shfl_up(i[u][kEPL - 1], 1), qj = __shfl_up(j[u][kEPL - 1], 1);
      if (lane == 0) {
        qi = piece > 0 ? pi[u] : -1;
        qj = piece > 0 ? pj[u] : -1;
      }
      T g[kEPL];
      gather_lane<T, ALL>(s_c, c, cached, k[u], g);
      if ((piece + 1) * kPiece > nnz) drop_beyond(piece * kPiece + lane * kEPL, nnz, g);  // uniform
      unsigned headmask = 0;
#pragma unroll
      for (int r = 0; r < kEPL; ++r) {
        if (i[u][r] != qi || j[u][r] != qj) headmask |= 1u << r;
        qi = i[u][r];
        qj = j[u][r];
      }
      const int cnt = __popc(headmask);
      const int upto = first[u] + wave_inclusive_sum(cnt);
      int next_idx = upto - cnt;
      // the number of fibres of the result: where the last piece's last head lands, plus one
      if (piece == npieces - 1 && lane == kWave - 1 && out_nnz) *out_nnz = upto;
      int key[kEPL];
      T p[kEPL];
#pragma unroll
      for (int r = 0; r < kEPL; ++r) {
        p[r] = v[u][r] * g[r];
        key[r] = next_idx;
        if (headmask & (1u << r)) {
          out_i[next_idx] = i[u][r];
          out_j[next_idx] = j[u][r];
          ++next_idx;
        }
      }
      wave_fibre_sums<T>(p, headmask, key, first[u] - 1, piece, out_v, carry_key, carry_val);
    }
  }
}

// The same with c in global memory and a wave per piece. SELF: piece_off holds the pieces' head counts,
// which every workgroup adds up as far as its pieces.
template <typename T, bool SELF>
__global__ __launch_bounds__(kBlock) void ttv_coo_piece_kernel(
    int nnz, int npieces, const int32_t* __restrict__ ci, const int32_t* __restrict__ cj,
    const int32_t* __restrict__ ck, const T* __restrict__ vals, const T* __restrict__ c,
    const int32_t* __restrict__ piece_off, const int32_t* __restrict__ group_off, int log_group, int32_t* __restrict__ out_i, int32_t* __restrict__ out_j,
    T* __restrict__ out_v, int64_t* __restrict__ out_nnz, int32_t* __restrict__ carry_key,
    T* __restrict__ carry_val) {
  constexpr int kWaves = kBlock / kWave;
  __shared__ int s_before[kWaves];
  const int lane = lane_id(), piece0 = blockIdx.x * kWaves;
  const int piece = __builtin_amdgcn_readfirstlane(min(piece0 + wave_id(), npieces - 1));  // beyond the end: the last piece again, not stored
  const int base = piece * kPiece, p0 = base + lane * kEPL;
  int32_t i[kEPL], j[kEPL], k[kEPL];
  T v[kEPL];
  if (base + kPiece <= nnz) {  // uniform
    load_any(ck + p0, k);
    load_any(vals + p0, v);
    load_any(cj + p0, j);
    const int32_t slice = ci[max(base - 1, 0)];
    if (slice == ci[base + kPiece - 1]) {
#pragma unroll
      for (int r = 0; r < kEPL; ++r) i[r] = slice;
    } else {
      load_any(ci + p0, i);
    }
  } else {
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
      const int p = min(p0 + r, nnz - 1);  // beyond the end: the last entry's fibre, value 0
      i[r] = ci[p];
      j[r] = cj[p];
      k[r] = ck[p];
      v[r] = p0 + r < nnz ? vals[p] : T(0);
    }
  }
  int32_t qi = -1, qj = -1;
  if (lane == 0 && base > 0) {
    qi = ci[base - 1];
    qj = cj[base - 1];
  }
  T g[kEPL];
#pragma unroll
  for (int r = 0; r < kEPL; ++r) g[r] = c[k[r]];
  if (base + kPiece > nnz) drop_beyond(p0, nnz, g);  // uniform
  int first;  // results before the piece
  if (SELF) {
    int before = 0;
    for (int t = threadIdx.x; t < piece0; t += kBlock) before += piece_off[t];
    before = wave_inclusive_sum(before);
    if (lane == kWave - 1) s_before[wave_id()] = before;
    __syncthreads();
    first = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) first += s_before[w];
    for (int w = piece0; w < piece; ++w) first += piece_off[w];
  } else {
    first = piece_off[piece] + group_off[piece >> log_group];
  }
  if (piece0 + wave_id() >= npieces) return;
  const int32_t ui = dpp_move<0x138, 0xf>(-1, i[kEPL - 1]), uj = dpp_move<0x138, 0xf>(-1, j[kEPL - 1]);  // wave_shr:1
  if (lane > 0) {
    qi = ui;
    qj = uj;
  }
  unsigned headmask = 0;
#pragma unroll
  for (int r = 0; r < kEPL; ++r) {
    if (i[r] != qi || j[r] != qj) headmask |= 1u << r;
    qi = i[r];
    qj = j[r];
  }
  const int cnt = __popc(headmask), upto = first + wave_inclusive_sum(cnt);
  if (piece == npieces - 1 && lane == kWave - 1 && out_nnz) *out_nnz = upto;
  int next = upto - cnt, key[kEPL];
  T p[kEPL];
#pragma unroll
  for (int r = 0; r < kEPL; ++r) {
    p[r] = v[r] * g[r];
    key[r] = next;
    if (headmask & (1u << r)) {
      out_i[next] = i[r];
      out_j[next] = j[r];
      ++next;
    }
  }
  wave_fibre_sums<T>(p, headmask, key, first - 1, piece, out_v, carry_key, carry_val);
}

// ================================================================ CSF
// Empty fibres. A group of kGap of them is zeroed here, a thread looks at each; what is not a whole group, by the piece it
// lies in (enter_fibres). 1M entries with 1M empty fibres in one gap,
// fp64: 4270 us all by that piece, 33 so. (Every 100th of 60M fibres with an entry: 366 us fibre after fibre, 257 with the
// starts of 256 on their way at a time.)
constexpr int kLogGap = 10, kGap = 1 << kLogGap;
template <typename T>
__device__ __forceinline__ void zero_gaps(int group, int nfib, const int32_t* __restrict__ pos, T* __restrict__ out_v) {
  constexpr int K = 16 / sizeof(T);
  typedef T V __attribute__((ext_vector_type(K), aligned(sizeof(T))));
  const bool empty = group < nfib >> kLogGap && pos[group << kLogGap] == pos[(group + 1) << kLogGap];
  for (uint64_t todo = __ballot(empty); todo; todo &= todo - 1) {
    const int64_t from = static_cast<int64_t>(__builtin_amdgcn_readlane(group, __ffsll(static_cast<long long>(todo)) - 1)) << kLogGap;
#pragma unroll
    for (int q = 0; q < kGap; q += kWave * K) *reinterpret_cast<V*>(out_v + from + q + lane_id() * K) = V(T(0));
  }
}
// The fibres f_lo .. f_hi - 1 of the piece that begins at entry `base`, by a wave: those with entries, at most kPiece, are
// entered in `mark`, and empty ones zeroed. After kGap empty ones in a row the next with entries is searched for.
template <typename T>
__device__ __forceinline__ void enter_fibres(int f_lo, int f_hi, int base, const int32_t* __restrict__ pos, int32_t* mark,
                                             T* __restrict__ out_v) {
  const int lane = lane_id(), n = f_hi - f_lo;  // (f_hi may be close to 2^31: no sum passes it)
  const auto enter = [&](int f, int a, int b) {
    if (b > a) mark[a - base] = f;
    else out_v[f] = T(0);
  };
  if (n <= 4 * kGap) {
    for (int q = lane; q < n; q += kWave) enter(f_lo + q, pos[f_lo + q], pos[f_lo + q + 1]);
    return;
  }
  const auto zero = [&](int f, int count) {
    for (int k = lane; k < count; k += kWave) out_v[f + k] = T(0);
  };
  int empty = 0;
  constexpr int U = 4;
  for (int q = 0; q < n;) {
    int a[U], b[U];
    bool any = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f_lo + q + min(u * kWave + lane, n - q - 1);
      a[u] = pos[f];
      b[u] = pos[f + 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u * kWave + lane < n - q) enter(f_lo + q + u * kWave + lane, a[u], b[u]);
      any = any || b[u] > a[u];  // (beyond the end: of the last fibre)
    }
    q += min(U * kWave, n - q);
    empty = __ballot(any) != 0 ? 0 : empty + U * kWave;
    if (empty >= kGap && q < n) {
      const int f = f_lo + q, at = pos[f];  // the last fibre that begins there has entries, or is the end
      const int next = group_last_true<kWave>(f, static_cast<int64_t>(f_hi) + 1, [&](int p) { return pos[p] <= at; });
      const int head = min(-f & (kGap - 1), next - f), tail = min(next & (kGap - 1), next - f - head);
      zero(f, head);
      zero(next - tail, tail);
      q = next - f_lo;
      empty = 0;
    }
  }
}

// first[piece] = first fibre that starts at or after the piece's first entry (piece ==
// npieces: the number of fibres, so that the last piece also covers trailing empty fibres).
// count (may be null) receives the number of values of the result, one per fibre.
// W lanes per search: it waits for its probes, and eight lanes need a third of the steps (12 000 pieces: 1.3 us
// less); with 60 000 pieces and more their number counts.
constexpr int kFewPieces = 32768;
// Workgroups from `search` on look for gaps.
template <int W, typename T>
__global__ __launch_bounds__(kBlock) void ttv_piece_fibres_kernel(int search, int npieces, int nfib,
                                                                  const int32_t* __restrict__ pos,
                                                                  int32_t* __restrict__ first,
                                                                  int64_t* __restrict__ count, T* __restrict__ out_v) {
  if (static_cast<int>(blockIdx.x) >= search) {
    zero_gaps<T>((blockIdx.x - search) * kBlock + threadIdx.x, nfib, pos, out_v);
    return;
  }
  const int t = blockIdx.x * kBlock + threadIdx.x, piece = t / W;
  if (t == 0 && count) *count = nfib;
  if (piece > npieces) return;
  const int target = piece * kPiece;
  int lo = 0, hi = nfib + 1;
  if (piece == npieces) {
    lo = nfib;
  } else if (W > 1) {
    lo = group_last_true<W>(0, static_cast<int64_t>(hi) + 1, [&](int q) { return q == 0 || pos[q - 1] < target; });
  } else {
    while (lo < hi) {
      const int mid = lo + ((hi - lo) >> 1);
      if (pos[mid] < target) lo = mid + 1; else hi = mid;
    }
  }
  if (t % W == 0) first[piece] = min(lo, nfib);
}

// out_v[f] = sum over the entries of fibre f (dense over the fibres, zero for empty ones).
template <typename T, bool VEC, bool ALL>
__global__ __launch_bounds__(kBig) void ttv_csf_wave_kernel(
    int nnz, int npieces, const int32_t* __restrict__ first, const int32_t* __restrict__ pos,
    const int32_t* __restrict__ ck, const T* __restrict__ vals, const T* __restrict__ c, int cached,
    T* __restrict__ out_v, int32_t* __restrict__ carry_key, T* __restrict__ carry_val) {
  __shared__ T s_c[kCsfCacheBytes / sizeof(T)];
  // fibre that starts at an entry of one of the wave's pieces, or -1
  __shared__ int32_t s_mark[kBigWaves][kNP][kPiece];
  stage_vector(s_c, c, cached);
  const int lane = lane_id();
#pragma unroll
  for (int u = 0; u < kNP; ++u)
#pragma unroll
    for (int r = 0; r < kEPL; ++r) s_mark[wave_id()][u][lane * kEPL + r] = -1;
  const int stride = gridDim.x * kBigWaves;
  for (int piece0 = __builtin_amdgcn_readfirstlane(blockIdx.x * kBigWaves + wave_id()); piece0 < npieces;
       piece0 += kNP * stride) {
    wave_lds_order();  // the marks are cleared
    int32_t k[kNP][kEPL], f_lo[kNP], f_hi[kNP];
    T v[kNP][kEPL];
#pragma unroll
    for (int u = 0; u < kNP; ++u) {
      const int piece = min(piece0 + u * stride, npieces - 1);  // beyond the end: the last piece again, not stored
      const int p0 = piece * kPiece + lane * kEPL;
      // fibres first[piece] .. first[piece + 1] - 1 start inside this piece (or are empty)
      f_lo[u] = first[piece];
      f_hi[u] = first[piece + 1];
      if (VEC && p0 + kEPL <= nnz) {
        load_lane(ck + p0, k[u]);
        load_lane(vals + p0, v[u]);
      } else {
#pragma unroll
        for (int r = 0; r < kEPL; ++r) {
          const bool ok = p0 + r < nnz;
          k[u][r] = ok ? ck[p0 + r] : 0;
          v[u][r] = ok ? vals[p0 + r] : T(0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kNP; ++u) {
      const int piece = piece0 + u * stride;
      if (piece >= npieces) break;
      enter_fibres<T>(f_lo[u], f_hi[u], piece * kPiece, pos, s_mark[wave_id()][u], out_v);
    }
#pragma unroll
    for (int u = 0; u < kNP; ++u) {
      const int piece = piece0 + u * stride;
      if (piece >= npieces) break;
      int32_t* mark = s_mark[wave_id()][u];
      T g[kEPL];
      gather_lane<T, ALL>(s_c, c, cached, k[u], g);
      if ((piece + 1) * kPiece > nnz) drop_beyond(piece * kPiece + lane * kEPL, nnz, g);  // uniform
      wave_lds_order();
      int key[kEPL];
      unsigned headmask = 0;
      T p[kEPL];
#pragma unroll
      for (int r = 0; r < kEPL; ++r) {
        key[r] = mark[lane * kEPL + r];
        if (key[r] >= 0) headmask |= 1u << r;
        p[r] = v[u][r] * g[r];
      }
      wave_lds_order();
#pragma unroll
      for (int r = 0; r < kEPL; ++r)
        if (key[r] >= 0) mark[lane * kEPL + r] = -1;
      wave_fibre_sums<T>(p, headmask, key, f_lo[u] - 1, piece, out_v, carry_key, carry_val);
    }
  }
}

// The same with c in global memory and a wave per piece.
template <typename T>
__global__ __launch_bounds__(kBlock) void ttv_csf_piece_kernel(
    int nnz, int npieces, const int32_t* __restrict__ first, const int32_t* __restrict__ pos,
    const int32_t* __restrict__ ck, const T* __restrict__ vals, const T* __restrict__ c, T* __restrict__ out_v,
    int32_t* __restrict__ carry_key, T* __restrict__ carry_val) {
  __shared__ int32_t s_mark[kBlock / kWave][kPiece];
  const int lane = lane_id();
  const int piece = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / kWave) + wave_id());
  if (piece >= npieces) return;
  const int base = piece * kPiece, p0 = base + lane * kEPL;
  int32_t k[kEPL], *mark = s_mark[wave_id()];
  T v[kEPL], g[kEPL];
  const int f_lo = first[piece], f_hi = first[piece + 1];
  if (base + kPiece <= nnz) {  // uniform
    load_any(ck + p0, k);
    load_any(vals + p0, v);
  } else {
#pragma unroll
    for (int r = 0; r < kEPL; ++r) {
      const bool ok = p0 + r < nnz;
      k[r] = ok ? ck[p0 + r] : 0;
      v[r] = ok ? vals[p0 + r] : T(0);
    }
  }
#pragma unroll
  for (int r = 0; r < kEPL; ++r) mark[lane * kEPL + r] = -1;
#pragma unroll
  for (int r = 0; r < kEPL; ++r) g[r] = c[k[r]];
  if (base + kPiece > nnz) drop_beyond(p0, nnz, g);  // uniform
  wave_lds_order();
  enter_fibres<T>(f_lo, f_hi, base, pos, mark, out_v);
  wave_lds_order();
  int key[kEPL];
  unsigned headmask = 0;
  T p[kEPL];
#pragma unroll
  for (int r = 0; r < kEPL; ++r) {
    key[r] = mark[lane * kEPL + r];
    if (key[r] >= 0) headmask |= 1u << r;
    p[r] = v[r] * g[r];
  }
  wave_fibre_sums<T>(p, headmask, key, f_lo - 1, piece, out_v, carry_key, carry_val);
}

// ================================================================ host
static int compute_units() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// COO tensors of up to 1.5M entries leave c in global memory, since staging it in every compute unit costs
// 8 us, and add up the pieces' counts themselves, since making offsets of them is a launch of its own; up to 2.75M where
// most of the gathers would go past the staged part of c anyway, fp64 with a c of more than 1.5 times that; up to 3M where
// nothing of c is staged (2.2M, c of 90 000, fp64 31.8 / 32.8). In us, so / as beyond (400 000 entries 12 / 14, 1.2M 19 / 23):
//   entries, c                        1.6M         2M           2.5M         3M
//   fp32, 30 000, skewed              20.0 / 18.7  23.0 / 18.8  27.4 / 23.8  31.1 / 24.4
//   fp32, 60 000, every one a fibre   24.7 / 25.8  29.1 / 28.0  35.7 / 39.1  41.7 / 40.8
//   fp64, 20 000, skewed              21.1 / 20.6  23.8 / 21.5  28.8 / 27.1  33.0 / 27.8
//     "           every one a fibre   27.3 / 27.8  30.8 / 29.3  37.1 / 38.4  42.4 / 39.7
//   fp64, 30 000, skewed              22.5 / 24.4  25.6 / 24.9  30.8 / 31.8  35.4 / 32.5
//     "           every one a fibre   28.4 / 30.5  32.8 / 33.3  39.5 / 43.1  45.5 / 45.1
//   fp64, 60 000, skewed              24.5 / 27.3  28.0 / 28.6  33.5 / 37.4  38.6 / 38.9
//     "           every one a fibre   28.8 / 33.3  33.6 / 35.5  40.9 / 47.3  47.3 / 48.9
constexpr int kSelfPieces = 6144;

static int64_t pieces_of(int64_t nnz) { return (nnz + kPiece - 1) / kPiece; }

// CSF tensors of fewer entries are reduced as CSR rows, in one launch where fibres are short (300 000 entries: 7 to 9 us,
// as pieces 10 to 11; 700 000: 15 to 16, 12 to 13), and so are those of a longer c: its gathers go beyond L2, and chunks
// of 2048 entries have more of them in flight. 15M entries, two to a fibre, as rows / as pieces, fp64: c of 100 000
// 136 / 126, 300 000 142 / 137, 900 000 190 / 209, 10M 314 / 350; fp32: 100 000 98 / 98, 300 000 113 / 104 (3M entries
// 27.4 / 29.5), 10M 287 / 302.
bool ttv_csf_applies(int64_t nnz, int64_t nfib, int64_t K, int dtype) {
  return nnz >= (int64_t(1) << 19) && nnz + kPiece < INT32_MAX && nfib + 1 < INT32_MAX &&
         K <= (dtype == SPT_F64 ? 300000 : 1 << 17);
}

// c is staged in LDS from here on. CSF, c of 10 000, as pieces with c in global memory / staged: 700 000 entries, fp32
// 11.5 / 12.0 us, fp64 12.6 / 12.8; 1.5M 13.5 / 13.0, 16.2 / 15.3; 15M 68 / 43, 98 / 55. (COO: the table below.)
constexpr int64_t kCsfStagedEntries = int64_t(1) << 20;

// Tensors whose last dimension is so long that less than a quarter of c fits the cache leave c in global memory: their
// gathers go there anyway, and without staging more waves are in flight for them. (CSF, fp64, c of 90 000, reduced as
// CSR rows / as pieces: 3M entries, skewed 44 / 28 us, every one a fibre 47 / 37; 15M 143 / 104, 177 / 142.)
bool ttv_wave_applies(int64_t nnz, int64_t K, int dtype) {
  const int64_t vsz = dtype == SPT_F64 ? 8 : 4;
  return nnz >= (int64_t(1) << 19) && nnz + kPiece < INT32_MAX && K * vsz <= 4 * (int64_t)kCsfCacheBytes;
}

size_t ttv_coo_workspace(int64_t nnz) {
  const int64_t np = pieces_of(nnz);
  return 3 * align_up((size_t)np * 4, 256) + align_up((size_t)np * 8, 256) + 256;
}
size_t ttv_csf_wave_workspace(int64_t nnz) {
  const int64_t np = pieces_of(nnz);
  return align_up((size_t)(np + 1) * 4, 256) + align_up((size_t)np * 4, 256) + align_up((size_t)np * 8, 256) + 256;
}

static bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <typename T>
spt_status ttv_coo(int64_t nnz64, int64_t K, const int32_t* ci, const int32_t* cj, const int32_t* ck,
                   const T* vals, const T* c, int32_t* out_i, int32_t* out_j, T* out_v, int64_t* out_nnz,
                   void* ws, size_t ws_bytes, hipStream_t s) {
  if (nnz64 + kPiece >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "ttv: more than 2^31 entries");
  const int nnz = (int)nnz64;
  const int np = (int)pieces_of(nnz64);
  if (!ws || ws_bytes < ttv_coo_workspace(nnz64))
    return fail(SPT_ERR_WORKSPACE, "ttv: workspace of %zu bytes needed, %zu given", ttv_coo_workspace(nnz64), ws_bytes);
  Workspace W(ws, ws_bytes);
  const bool wave = ttv_wave_applies(nnz64, K, sizeof(T) == 8 ? SPT_F64 : SPT_F32);
  const bool past = sizeof(T) == 8 && K * 2 * static_cast<int64_t>(sizeof(T)) > 3 * kCooCacheBytes;
  const bool self = np <= (!wave ? 2 * kSelfPieces : past ? kSelfPieces / 4 * 7 : kSelfPieces);
  const int log_group = np >= kManyPieces ? kLogGroupMany : kLogGroup;
  const unsigned groups = (unsigned)(((np - 1) >> log_group) + 1);
  int32_t* group_off = W.take<int32_t>(groups);
  int32_t* off = W.take<int32_t>(np);
  int32_t* ckey = W.take<int32_t>(np);
  T* cval = W.take<T>(np);
  const bool vec = al16(ci) && al16(cj) && al16(ck) && al16(vals);
  const unsigned grid4 = (unsigned)((np + kBlock / kWave - 1) / (kBlock / kWave));
#define SPT_TTV_HEADS(VEC_, SELF_, LOG_)                                                                             \
  hipLaunchKernelGGL((ttv_piece_heads_kernel<VEC_, SELF_, LOG_>), dim3(SELF_ ? grid4 : groups), dim3(kBlock), 0, s, \
                     nnz, np, ci, cj, off, group_off)
  if (self && vec) SPT_TTV_HEADS(true, true, kLogGroup);
  else if (self) SPT_TTV_HEADS(false, true, kLogGroup);
  else if (vec && log_group == kLogGroup) SPT_TTV_HEADS(true, false, kLogGroup);
  else if (vec) SPT_TTV_HEADS(true, false, kLogGroupMany);
  else if (log_group == kLogGroup) SPT_TTV_HEADS(false, false, kLogGroup);
  else SPT_TTV_HEADS(false, false, kLogGroupMany);
#undef SPT_TTV_HEADS
  SPT_CHECK_LAUNCH("ttv piece heads");
  if (self) {
    hipLaunchKernelGGL((ttv_coo_piece_kernel<T, true>), dim3(grid4), dim3(kBlock), 0, s, nnz, np, ci, cj, ck, vals, c,
                       off, group_off, log_group, out_i, out_j, out_v, out_nnz, ckey, cval);
    SPT_CHECK_LAUNCH("ttv coo pieces");
  } else {
    hipLaunchKernelGGL(ttv_group_off_kernel, dim3(1), dim3(1024), 0, s, (int)groups, group_off);
    SPT_CHECK_LAUNCH("ttv group offsets");
    if (wave) {
      const int cached = (int)std::min<int64_t>(K, kCooCacheBytes / sizeof(T));
      const bool all = cached == K;
      const unsigned grid = (unsigned)std::min<int64_t>(compute_units(), (np + kBigWaves - 1) / kBigWaves);
#define SPT_TTV_COO(VEC_, ALL_)                                                                                    \
  hipLaunchKernelGGL((ttv_coo_wave_kernel<T, VEC_, ALL_>), dim3(grid), dim3(kBig), 0, s, nnz, np, ci, cj, ck, vals, \
                     c, cached, off, group_off, log_group, out_i, out_j, out_v, out_nnz, ckey, cval)
      if (vec && all) SPT_TTV_COO(true, true);
      else if (vec) SPT_TTV_COO(true, false);
      else if (all) SPT_TTV_COO(false, true);
      else SPT_TTV_COO(false, false);
#undef SPT_TTV_COO
    } else {
      hipLaunchKernelGGL((ttv_coo_piece_kernel<T, false>), dim3(grid4), dim3(kBlock), 0, s, nnz, np, ci, cj, ck, vals,
                         c, off, group_off, log_group, out_i, out_j, out_v, out_nnz, ckey, cval);
    }
    SPT_CHECK_LAUNCH("ttv coo");
  }
  hipLaunchKernelGGL(carry_fixup_kernel<T>, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, s, np, ckey, cval,
                     out_v, nullptr, 0);
  SPT_CHECK_LAUNCH("ttv carry_fixup");
  return SPT_OK;
}

template <typename T>
spt_status ttv_csf_wave(int64_t nnz64, int64_t nfib, int64_t K, const int32_t* pos, const int32_t* ck,
                        const T* vals, const T* c, T* out_v, int64_t* out_count, void* ws, size_t ws_bytes,
                        hipStream_t s) {
  const int nnz = (int)nnz64;
  const int np = (int)pieces_of(nnz64);
  if (nfib + 1 >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "ttv: more than 2^31 fibres");
  if (!ws || ws_bytes < ttv_csf_wave_workspace(nnz64))
    return fail(SPT_ERR_WORKSPACE, "ttv: workspace of %zu bytes needed, %zu given", ttv_csf_wave_workspace(nnz64),
                ws_bytes);
  Workspace W(ws, ws_bytes);
  int32_t* first = W.take<int32_t>(np + 1);
  int32_t* ckey = W.take<int32_t>(np);
  T* cval = W.take<T>(np);
  const int gaps = nfib > 4 * kGap ? (int)(((nfib >> kLogGap) + kBlock - 1) / kBlock) : 0;
#define SPT_TTV_FIRST(W_)                                                                                            \
  do {                                                                                                               \
    const int search = (int)(((int64_t)(np + 1) * W_ + kBlock - 1) / kBlock);                                        \
    hipLaunchKernelGGL((ttv_piece_fibres_kernel<W_, T>), dim3(search + gaps), dim3(kBlock), 0, s, search, np, (int)nfib, pos, \
                       first, out_count, out_v);                                                                     \
  } while (0)
  if (np <= kFewPieces) SPT_TTV_FIRST(8);
  else SPT_TTV_FIRST(1);
#undef SPT_TTV_FIRST
  SPT_CHECK_LAUNCH("ttv piece fibres");
  if (nnz64 >= kCsfStagedEntries && ttv_wave_applies(nnz64, K, sizeof(T) == 8 ? SPT_F64 : SPT_F32)) {
    const bool vec = al16(ck) && al16(vals);
    const int cached = (int)std::min<int64_t>(K, kCsfCacheBytes / sizeof(T));
    const bool all = cached == K;
    const unsigned grid = (unsigned)std::min<int64_t>(compute_units(), (np + kBigWaves - 1) / kBigWaves);
#define SPT_TTV_CSF(VEC_, ALL_)                                                                                   \
  hipLaunchKernelGGL((ttv_csf_wave_kernel<T, VEC_, ALL_>), dim3(grid), dim3(kBig), 0, s, nnz, np, first, pos, ck, \
                     vals, c, cached, out_v, ckey, cval)
    if (vec && all) SPT_TTV_CSF(true, true);
    else if (vec) SPT_TTV_CSF(true, false);
    else if (all) SPT_TTV_CSF(false, true);
    else SPT_TTV_CSF(false, false);
#undef SPT_TTV_CSF
  } else {
    hipLaunchKernelGGL(ttv_csf_piece_kernel<T>, dim3((np + kBlock / kWave - 1) / (kBlock / kWave)), dim3(kBlock), 0, s, nnz,
                       np, first, pos, ck, vals, c, out_v, ckey, cval);
  }
  SPT_CHECK_LAUNCH("ttv csf wave");
  hipLaunchKernelGGL(carry_fixup_kernel<T>, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, s, np, ckey, cval,
                     out_v, nullptr, 0);
  SPT_CHECK_LAUNCH("ttv carry_fixup");
  return SPT_OK;
}

template spt_status ttv_coo<float>(int64_t, int64_t, const int32_t*, const int32_t*, const int32_t*,
                                        const float*, const float*, int32_t*, int32_t*, float*, int64_t*, void*,
                                        size_t, hipStream_t);
template spt_status ttv_coo<double>(int64_t, int64_t, const int32_t*, const int32_t*, const int32_t*,
                                         const double*, const double*, int32_t*, int32_t*, double*, int64_t*, void*,
                                         size_t, hipStream_t);
template spt_status ttv_csf_wave<float>(int64_t, int64_t, int64_t, const int32_t*, const int32_t*, const float*,
                                        const float*, float*, int64_t*, void*, size_t, hipStream_t);
template spt_status ttv_csf_wave<double>(int64_t, int64_t, int64_t, const int32_t*, const int32_t*, const double*,
                                         const double*, double*, int64_t*, void*, size_t, hipStream_t);

}  // namespace spt
