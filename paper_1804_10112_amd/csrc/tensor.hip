// SpDM and TTM on ordered COO and on CSF (paper Sections 5.2, 5.3), and which kernels TTV runs, gfx950.
//
// Both reduce runs of consecutive stored entries that share leading
// coordinates -- the GPU form of the paper's deduplication / iterator chaining
// over ordered non-unique levels (Section 4.3): (i,j) fibres for TTM, rows
// for SpDM. Work is split evenly over stored entries; a run cut by a split
// leaves a carry that a follow-up kernel adds in a fixed order (no atomics).
#include <algorithm>

#include "carry.hpp"
#include "common.hpp"
#include "scan.hpp"
#include "segreduce.hpp"

namespace spt {

spt_status csr_rows_reduce(int dtype, int64_t nnz, int64_t nrows, const int32_t* pos,
                           const int32_t* crd, const void* vals, const void* x, void* out,
                           void* ws, size_t ws_bytes, hipStream_t s);
size_t seg_spmv_workspace(int64_t nnz);

template <typename T>
__device__ __forceinline__ T ldg_stream(const T* p) {
  return __builtin_nontemporal_load(p);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fill_t_kernel(T* __restrict__ out, int64_t n, T value) {
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) out[i] = value;
}

// ================================================================ fibres of a COO tensor (TTM)

constexpr int kTtvIPT = 8;
constexpr int kTtvChunk = kTtvIPT * kBlock;

// heads[w] = number of (i,j) fiber starts among the entries of chunk w.
// VEC: 16-byte coordinate loads (needs 16-byte aligned ci, cj).
template <bool VEC>
__global__ __launch_bounds__(kBlock) void ttv_count_kernel(int nnz, const int32_t* __restrict__ ci,
                                                           const int32_t* __restrict__ cj,
                                                           int32_t* __restrict__ heads) {
  const int base = blockIdx.x * kTtvChunk;
  int cnt = 0;
  if (VEC) {
    typedef int32_t i4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < kTtvIPT / 4; ++q) {
      const int p0 = base + (q * kBlock + threadIdx.x) * 4;
      if (p0 + 4 <= nnz) {
        const i4 a = ldg_stream(reinterpret_cast<const i4*>(ci + p0));
        const i4 b = ldg_stream(reinterpret_cast<const i4*>(cj + p0));
        int pa = -1, pb = -1;
        if (p0 > 0) {
          pa = ci[p0 - 1];
          pb = cj[p0 - 1];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          cnt += (a[r] != pa || b[r] != pb) ? 1 : 0;
          pa = a[r];
          pb = b[r];
        }
      } else {
        for (int p = p0; p < nnz && p < p0 + 4; ++p)
          cnt += (p == 0 || ci[p] != ci[p - 1] || cj[p] != cj[p - 1]) ? 1 : 0;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < kTtvIPT; ++k) {
      const int p = base + k * kBlock + threadIdx.x;
      if (p < nnz) cnt += (p == 0 || ci[p] != ci[p - 1] || cj[p] != cj[p - 1]) ? 1 : 0;
    }
  }
  int total;
  block_inclusive_sum(cnt, &total);
  if (threadIdx.x == 0) heads[blockIdx.x] = total;
}

__global__ void ttv_total_kernel(int nchunks, const int32_t* __restrict__ heads,
                                 const int32_t* __restrict__ off, int64_t* __restrict__ out_nnz) {
  if (threadIdx.x == 0 && blockIdx.x == 0)
    *out_nnz = nchunks > 0 ? (int64_t)off[nchunks - 1] + heads[nchunks - 1] : 0;
}

// ================================================================ SpDM
//
// A_ij = sum_k B_ik C_kj, B an ordered COO matrix (or the entries of a tensor under fibre numbers, TTM).
// G lanes (32 or 64) work on one stored entry at a time, lane gl owning output
// column jt*G + gl; a workgroup has 256/G such groups, each walking kEPG
// consecutive entries and keeping the running row sum in a register. Entry
// coordinates are loaded G at a time (coalesced) and broadcast with shuffles;
// the factor rows C[k,:] are gathered as contiguous G-wide rows.
// LEVEL2 = the same reduction applied to the (key, vector) carries of level 1.
enum { MT_LEVEL2 = 1, MT_SPDM = 3 };
// entries walked by one group of lanes: the carry level is small and wants parallelism instead
template <int MODE> struct Epg { static constexpr int value = MODE == MT_LEVEL2 ? 32 : 128; };
constexpr int kU = 8;  // entries whose factor rows are in flight together

template <typename T, int G>
struct SpdmShared {
  T lead[kBlock / G][G];
  T tail[kBlock / G][G];
  int has_head[kBlock / G];
  int first_close[kBlock / G];
  int last_key[kBlock / G];
  int empty[kBlock / G];
};


// Broadcast of lane (addr / 4)'s value through the LDS crossbar.
__device__ __forceinline__ int32_t bperm(int addr, int32_t v) { return __builtin_amdgcn_ds_bpermute(addr, v); }
__device__ __forceinline__ float bperm(int addr, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double bperm(int addr, double v) {
  const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
  const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
  return __hiloint2double(hi, lo);
}

// FAST: the factor matrix is addressed with 32-bit byte offsets formed by one 24-bit
// multiply-add (host-checked: dimensions and J * sizeof(T) below 2^23, matrices below 4 GiB),
// and no load of the batch sits behind a branch: a batch slot beyond the group's entries
// repeats the last entry, a lane beyond column J reads column J - 1 (neither is ever stored).
// The 64-bit multiply-adds and the per-entry branches of the general path cost more vector
// instructions than the arithmetic itself.
template <typename T, int G, int MODE, bool FAST>
__global__ __launch_bounds__(kBlock) void spdm_rows_kernel(
    int n, int J,
    const int32_t* __restrict__ ci, const int32_t* __restrict__ ck, const T* __restrict__ vals,
    const T* __restrict__ Cm,
    // LEVEL2 input
    const int32_t* __restrict__ in_key, const T* __restrict__ in_vec,
    T* __restrict__ A, int32_t* __restrict__ carry_key, T* __restrict__ carry_vec, bool dealt) {
  constexpr int NG = kBlock / G;
  constexpr int kEPG = Epg<MODE>::value;
  constexpr int CHUNK = NG * kEPG;
  __shared__ SpdmShared<T, G> sh;
  // SpDM closes a row every few entries. A store issued between two batches of gathers
  // makes the next batch wait for the store's acknowledgement (loads and stores retire
  // through one counter), so closed rows are parked in LDS and written out in bursts.
  constexpr int kRowBuf = 16;
  __shared__ T s_rowv[MODE == MT_SPDM ? NG : 1][MODE == MT_SPDM ? kRowBuf : 1][G];
  __shared__ int s_rowk[MODE == MT_SPDM ? NG : 1][MODE == MT_SPDM ? kRowBuf : 1];
  int nbuf = 0;

  const int tid = threadIdx.x;
  const int g = tid / G, gl = tid % G;
  const int j = blockIdx.y * G + gl;
  const bool jok = j < J;
  // FAST: byte address of lane 0 of this lane's group for the broadcasts, bytes per factor
  // row and this lane's byte offset inside a row
  const int half_base = 4 * (lane_id() & ~(G - 1));
  const uint32_t jbytes = static_cast<uint32_t>(J) * sizeof(T);
  const uint32_t joff = static_cast<uint32_t>(min(j, J - 1)) * sizeof(T);
  // a tensor's chunks are dealt out to the XCDs in turn: its fibres are long in the first slices and single entries
  // in the last, which in one piece keep one XCD busy longest (50M entries, K = 32: 1.63 -> 1.24 ms)
  const int chunk = dealt ? static_cast<int>(blockIdx.x) : xcd_contiguous_block_id();
  const int chunk_base = chunk * CHUNK;
  const int chunk_end = min(chunk_base + CHUNK, n);

  // ---- group walk
  const int g0 = chunk_base + g * kEPG;
  const int g1 = min(g0 + kEPG, chunk_end);
  T acc = 0, lead = 0;
  int has_head = 0, first_close = -1;
  int cur = -1;
  // cur = row of the entry just before this group's first entry (-1: there is none)
  if (g0 < g1) {
    if (MODE == MT_SPDM) cur = g0 > 0 ? ci[g0 - 1] : -1;
    if (MODE == MT_LEVEL2) cur = g0 > 0 ? in_key[g0 - 1] : -1;
  }

  for (int b0 = g0; b0 < g1; b0 += G) {
    const int p_l = b0 + gl;
    int32_t ri = 0, rk = 0;
    T rv = 0;
    if (p_l < g1) {
      if (MODE == MT_SPDM) {
        ri = ldg_stream(ci + p_l);
        rk = ldg_stream(ck + p_l);
        rv = ldg_stream(vals + p_l);
      } else {
        ri = in_key[p_l];
      }
    }
    const int cntb = min(G, g1 - b0);
    // kU entries at a time: first issue all their factor-row loads (they are
    // independent, so the cache latency is paid once per batch, not per entry),
    // then run the segment logic over the batch in order.
    for (int s0 = 0; s0 < cntb; s0 += kU) {
      int ii[kU];
      T fa[kU], vv[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int sidx = s0 + u;  // < G because kU divides G
        const bool live = sidx < cntb;
        vv[u] = T(1);
        if (FAST && MODE != MT_LEVEL2) {
          const int addr = half_base + 4 * min(sidx, cntb - 1);
          ii[u] = bperm(addr, ri);
          const int k = bperm(addr, rk);
          vv[u] = bperm(addr, rv);
          fa[u] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(Cm) + (__umul24(k, jbytes) + joff));
          continue;
        }
        ii[u] = __shfl(ri, sidx, G);
        if (MODE == MT_LEVEL2) {
          fa[u] = (live && jok) ? in_vec[(int64_t)(b0 + sidx) * J + j] : T(0);
        } else {
          const int k = __shfl(rk, sidx, G);
          vv[u] = __shfl(rv, sidx, G);
          fa[u] = (live && jok) ? Cm[(int64_t)k * J + j] : T(0);
        }
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        if (s0 + u < cntb) {
          const int i = ii[u];
          if (i != cur) {
            if (!has_head) {
              lead = acc;
              has_head = 1;
              first_close = cur;
            } else if (cur >= 0) {
              if (MODE == MT_SPDM) {
                s_rowv[g][nbuf][gl] = acc;
                if (gl == 0) s_rowk[g][nbuf] = cur;
                ++nbuf;
              } else if (jok) {
                if (MODE == MT_LEVEL2) A[(int64_t)cur * J + j] += acc;
                else A[(int64_t)cur * J + j] = acc;
              }
            }
            acc = 0;
            cur = i;
          }
          if (MODE == MT_SPDM) acc += vv[u] * fa[u];
          else acc += fa[u];
        }
      }
      if (MODE == MT_SPDM && nbuf > kRowBuf - kU) {
        for (int r = 0; r < nbuf; ++r)
          if (jok) __builtin_nontemporal_store(s_rowv[g][r][gl], &A[(int64_t)s_rowk[g][r] * J + j]);
        nbuf = 0;
      }
    }
  }
  if (MODE == MT_SPDM) {
    for (int r = 0; r < nbuf; ++r)
      if (jok) __builtin_nontemporal_store(s_rowv[g][r][gl], &A[(int64_t)s_rowk[g][r] * J + j]);
  }

  sh.lead[g][gl] = lead;
  sh.tail[g][gl] = acc;
  if (gl == 0) {
    sh.has_head[g] = has_head;
    sh.first_close[g] = first_close;
    sh.last_key[g] = cur;
    sh.empty[g] = g0 >= g1;
  }
  __syncthreads();

  // ---- resolve the NG group summaries in order (threads of group 0)
  if (g == 0) {
    T run = 0;
    bool seen = false, carried = false;
    int last = -1;
    for (int q = 0; q < NG; ++q) {
      if (sh.empty[q]) continue;
      if (sh.has_head[q]) {
        const T total = run + sh.lead[q][gl];
        const int key = sh.first_close[q];
        if (seen) {
          if (jok && key >= 0) {
            if (MODE == MT_LEVEL2) A[(int64_t)key * J + j] += total;
            else A[(int64_t)key * J + j] = total;
          }
        } else {  // precedes the first head of the chunk: carry (key < 0: nothing precedes)
          if (jok) carry_vec[(int64_t)chunk * J + j] = total;
          if (gl == 0 && blockIdx.y == 0) carry_key[chunk] = key < 0 ? -1 : key;
          carried = true;
        }
        run = sh.tail[q][gl];
        seen = true;
      } else {
        run += sh.tail[q][gl];
      }
      last = sh.last_key[q];
    }
    if (seen) {
      if (jok && last >= 0) {
        if (MODE == MT_LEVEL2) A[(int64_t)last * J + j] += run;
        else A[(int64_t)last * J + j] = run;
      }
    } else if (!carried) {
      if (jok) carry_vec[(int64_t)chunk * J + j] = run;
      if (gl == 0 && blockIdx.y == 0) carry_key[chunk] = last;
    }
  }
}

// Adds the remaining (key, vector) carries into A, one thread per (carry, j);
// the thread at the start of a run of equal keys adds the whole run in order.
template <typename T>
__global__ __launch_bounds__(kBlock) void vec_carry_fixup_kernel(int n, int J,
                                                                 const int32_t* __restrict__ key,
                                                                 const T* __restrict__ vec,
                                                                 T* __restrict__ A) {
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= (int64_t)n * J) return;
  const int w = (int)(idx / J), j = (int)(idx % J);
  const int32_t kk = key[w];
  if (kk < 0) return;
  if (w > 0 && key[w - 1] == kk) return;
  double s = 0;
  for (int u = w; u < n && key[u] == kk; ++u) s += (double)vec[(int64_t)u * J + j];
  A[(int64_t)kk * J + j] = (T)((double)A[(int64_t)kk * J + j] + s);
}

static int spdm_group(int J) { return J <= 32 ? 32 : 64; }
static int spdm_chunk(int J, int mode) {
  return (kBlock / spdm_group(J)) * (mode == MT_LEVEL2 ? Epg<MT_LEVEL2>::value : Epg<MT_SPDM>::value);
}

size_t spdm_workspace(const spt_tensor* B, int32_t J) {
  if (J < 1) J = 1;
  const int64_t chunk = spdm_chunk(J, MT_SPDM), chunk2 = spdm_chunk(J, MT_LEVEL2);
  const int64_t n1 = (B->nvals + chunk - 1) / chunk;
  const int64_t n2 = (n1 + chunk2 - 1) / chunk2;
  return align_up((size_t)n1 * 4, 256) + align_up((size_t)n1 * J * 8, 256) +
         align_up((size_t)n2 * 4, 256) + align_up((size_t)n2 * J * 8, 256) + 256;
}

// rows_override / cols_override: row and column index per stored entry taken
// from these arrays instead of B's first two levels, and no zero fill of A (every output row
// then has at least one entry, and rows with entries are stored, not accumulated).
template <typename T, int G, bool FAST>
static spt_status spdm_launch(const spt_tensor* B, const T* Cm, int J, T* A, void* ws, size_t ws_bytes,
                              hipStream_t s, const int32_t* rows_override, const int32_t* cols_override) {
  const int CHUNK = spdm_chunk(J, MT_SPDM), CHUNK2 = spdm_chunk(J, MT_LEVEL2);
  const int64_t I = B->level[0].N;
  const int64_t nnz64 = B->nvals;
  if (nnz64 + CHUNK >= INT32_MAX || I * J >= ((int64_t)1 << 38))
    return fail(SPT_ERR_UNSUPPORTED, "spdm: matrix too large");
  if (I * J > 0 && !rows_override) {
    hipLaunchKernelGGL(fill_t_kernel<T>, dim3((unsigned)((I * J + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, A, I * J, T(0));
    SPT_CHECK_LAUNCH("spdm fill");
  }
  const int nnz = (int)nnz64;
  if (nnz == 0) return SPT_OK;
  if (!ws || ws_bytes < spdm_workspace(B, J))
    return fail(SPT_ERR_WORKSPACE, "spdm: workspace of %zu bytes needed, %zu given", spdm_workspace(B, J), ws_bytes);
  const int n1 = (nnz + CHUNK - 1) / CHUNK;
  const int n2 = (n1 + CHUNK2 - 1) / CHUNK2;
  Workspace W(ws, ws_bytes);
  int32_t* key1 = W.take<int32_t>(n1);
  T* vec1 = W.take<T>((size_t)n1 * J);
  int32_t* key2 = W.take<int32_t>(n2);
  T* vec2 = W.take<T>((size_t)n2 * J);
  const unsigned jt = (unsigned)((J + G - 1) / G);
  const spt_level* L = B->level;
  hipLaunchKernelGGL((spdm_rows_kernel<T, G, MT_SPDM, FAST>), dim3(n1, jt), dim3(kBlock), 0, s, nnz, J,
                     rows_override ? rows_override : L[0].crd, cols_override ? cols_override : L[1].crd,
                     static_cast<const T*>(B->vals), Cm, nullptr, nullptr, A, key1, vec1, rows_override != nullptr);
  SPT_CHECK_LAUNCH("spdm");
  hipLaunchKernelGGL((spdm_rows_kernel<T, G, MT_LEVEL2, false>), dim3(n2, jt), dim3(kBlock), 0, s, n1, J,
                     nullptr, nullptr, nullptr, nullptr, key1, vec1, A, key2, vec2, false);
  SPT_CHECK_LAUNCH("spdm level 2");
  const int64_t tot = (int64_t)n2 * J;
  hipLaunchKernelGGL(vec_carry_fixup_kernel<T>, dim3((unsigned)((tot + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, n2, J, key2, vec2, A);
  SPT_CHECK_LAUNCH("spdm fixup");
  return SPT_OK;
}

template <typename T>
static spt_status spdm_typed(const spt_tensor* B, const void* C, int J, void* A, void* ws, size_t ws_bytes,
                             hipStream_t s, const int32_t* rows_override = nullptr,
                             const int32_t* cols_override = nullptr) {
  const T* Cm = static_cast<const T*>(C);
  // 32-bit factor addressing: every coordinate and the row size below 2^23 (one 24-bit multiply),
  // the factor matrix below 4 GiB
  int64_t big = 0;  // the largest dimension bounds every coordinate that indexes a factor row
  for (int k = 0; k < B->nlevels; ++k) big = std::max(big, B->level[k].N);
  const int64_t rowb = (int64_t)J * (int64_t)sizeof(T);
  const bool fast = big < (1 << 23) && rowb < (1 << 23) && big * rowb < ((int64_t)1 << 32);
  T* out = static_cast<T*>(A);
  if (spdm_group(J) == 32)
    return fast ? spdm_launch<T, 32, true>(B, Cm, J, out, ws, ws_bytes, s, rows_override, cols_override)
                : spdm_launch<T, 32, false>(B, Cm, J, out, ws, ws_bytes, s, rows_override, cols_override);
  return fast ? spdm_launch<T, 64, true>(B, Cm, J, out, ws, ws_bytes, s, rows_override, cols_override)
              : spdm_launch<T, 64, false>(B, Cm, J, out, ws, ws_bytes, s, rows_override, cols_override);
}

// SpDM A = B C (Section 5.2, Figure 11): B an ordered COO matrix, C and A dense row-major.
spt_status spdm_dispatch(const spt_tensor* B, const void* C, int32_t J, void* A_out, void* ws,
                         size_t ws_bytes, hipStream_t s) {
  if (!(B->level[0].flags & SPT_ORDERED))
    return fail(SPT_ERR_UNSUPPORTED, "spdm: the row level of B must be ordered");
  if (B->dtype == SPT_F64) return spdm_typed<double>(B, C, J, A_out, ws, ws_bytes, s);
  return spdm_typed<float>(B, C, J, A_out, ws, ws_bytes, s);
}

// ================================================================ TTV dispatch

__global__ void set_i64_kernel(int64_t* out, int64_t v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = v;
}

// ================================================================ TTM
//
// A_ijk = sum_l B_ijl C_kl (Section 5.3): every (i,j) fibre of B yields one dense fibre of K
// values, A[f, :] = sum over the fibre's entries of B_ijl * C[:, l]. With the fibre index as
// row and l as column this is the sparse-times-dense reduction of SpDM against C transposed,
// so TTM = (fibre index per entry) + (C transposed into the workspace) + the SpDM kernels.

// COO: fid[p] = index of the (i,j) fibre of entry p; the thread holding a fibre's first
// entry appends its coordinates (append order = ascending (i,j)). Chunks as in ttv_count_kernel.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void fiber_ids_kernel(int nnz, const int32_t* __restrict__ ci,
                                                           const int32_t* __restrict__ cj,
                                                           const int32_t* __restrict__ chunk_off,
                                                           int32_t* __restrict__ fid,
                                                           int32_t* __restrict__ out_i,
                                                           int32_t* __restrict__ out_j) {
  typedef int32_t i4 __attribute__((ext_vector_type(4)));
  static_assert(kTtvIPT == 8, "two 16-byte loads per array and thread");
  const int p0 = blockIdx.x * kTtvChunk + threadIdx.x * kTtvIPT;
  int32_t li[kTtvIPT], lj[kTtvIPT];
  int32_t qi = -1, qj = -1;
  if (p0 > 0 && p0 < nnz) {
    qi = ci[p0 - 1];
    qj = cj[p0 - 1];
  }
  const bool full = VEC && p0 + kTtvIPT <= nnz;
  if (full) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const i4 a = *reinterpret_cast<const i4*>(ci + p0 + 4 * h);
      const i4 b = *reinterpret_cast<const i4*>(cj + p0 + 4 * h);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        li[4 * h + r] = a[r];
        lj[4 * h + r] = b[r];
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < kTtvIPT; ++k) {
      li[k] = p0 + k < nnz ? ci[p0 + k] : -1;
      lj[k] = p0 + k < nnz ? cj[p0 + k] : -1;
    }
  }
  unsigned headmask = 0;
#pragma unroll
  for (int k = 0; k < kTtvIPT; ++k) {
    if (p0 + k < nnz && (li[k] != qi || lj[k] != qj)) headmask |= 1u << k;
    qi = li[k];
    qj = lj[k];
  }
  const int cnt = __popc(headmask);
  int total;
  int running = chunk_off[blockIdx.x] + block_inclusive_sum(cnt, &total) - cnt - 1;
  int32_t lf[kTtvIPT];
#pragma unroll
  for (int k = 0; k < kTtvIPT; ++k) {
    if (headmask & (1u << k)) {
      ++running;
      out_i[running] = li[k];
      out_j[running] = lj[k];
    }
    lf[k] = running;
  }
  if (full) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      i4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = lf[4 * h + r];
      *reinterpret_cast<i4*>(fid + p0 + 4 * h) = v;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kTtvIPT; ++k)
      if (p0 + k < nnz) fid[p0 + k] = lf[k];
  }
}

// CSF: the fibre of entry p is the position f of level 1 with pos2[f] <= p < pos2[f+1].
__global__ __launch_bounds__(kBlock) void expand_fiber_ids_kernel(int nfib,
                                                                  const int32_t* __restrict__ pos2,
                                                                  int32_t* __restrict__ fid) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= nfib) return;
  const int a = pos2[f], b = pos2[f + 1];
  for (int p = a; p < b; ++p) fid[p] = f;
}

// CSF: a fibre without entries (a compressed level may hold empty segments) still owns K
// output values; no entry ever writes them, so they are set to zero here. One lane per
// (fibre, k) pair would read pos2 K times: a lane tests one fibre and the rare hit loops.
template <typename T>
__global__ __launch_bounds__(kBlock) void zero_empty_fibres_kernel(int nfib, int K,
                                                                   const int32_t* __restrict__ pos2,
                                                                   T* __restrict__ out) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= nfib || pos2[f + 1] > pos2[f]) return;
  for (int k = 0; k < K; ++k) out[(int64_t)f * K + k] = T(0);
}

// Ct[l * K + k] = C[k * L + l]
template <typename T>
__global__ __launch_bounds__(kBlock) void transpose_kernel(int K, int64_t L, const T* __restrict__ C,
                                                           T* __restrict__ Ct) {
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= L * K) return;
  const int64_t l = idx / K;
  const int k = (int)(idx % K);
  Ct[idx] = C[(int64_t)k * L + l];
}

size_t ttm_workspace(Format f, const spt_tensor* B, int32_t K) {
  if (K < 1) K = 1;
  const int64_t nnz = B->nvals, L = B->level[2].N;
  size_t n = align_up((size_t)nnz * 4, 256) + align_up((size_t)L * K * 8, 256) +
             spdm_workspace(B, K);
  if (f == Format::COO3) {
    const int64_t nch = (nnz + kTtvChunk - 1) / kTtvChunk;
    n += 2 * align_up((size_t)nch * 4, 256) + scan_workspace(nch);
  }
  return n + 256;
}

template <typename T>
static spt_status ttm_typed(Format f, const spt_tensor* B, const T* C, int K, int32_t* out_i,
                            int32_t* out_j, T* out_v, int64_t* out_nfib, void* ws, size_t ws_bytes,
                            hipStream_t s) {
  const int64_t nnz64 = B->nvals, L = B->level[2].N;
  if (nnz64 + kTtvChunk >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "ttm: more than 2^31 entries");
  const int nnz = (int)nnz64;
  if (nnz == 0) {
    if (out_nfib) {
      hipLaunchKernelGGL(set_i64_kernel, dim3(1), dim3(kWave), 0, s, out_nfib, (int64_t)0);
      SPT_CHECK_LAUNCH("ttm set count");
    }
    return SPT_OK;
  }
  if (!ws || ws_bytes < ttm_workspace(f, B, K))
    return fail(SPT_ERR_WORKSPACE, "ttm: workspace of %zu bytes needed, %zu given",
                ttm_workspace(f, B, K), ws_bytes);
  Workspace W(ws, ws_bytes);
  int32_t* fid = W.take<int32_t>(nnz);
  T* Ct = W.take<T>((size_t)L * K);
  if (f == Format::COO3) {
    const int nch = (nnz + kTtvChunk - 1) / kTtvChunk;
    int32_t* heads = W.take<int32_t>(nch);
    int32_t* off = W.take<int32_t>(nch);
    int32_t* scan_tmp = reinterpret_cast<int32_t*>(W.take<char>(scan_workspace(nch)));
    const int32_t *ci = B->level[0].crd, *cj = B->level[1].crd;
    const bool vec = ((reinterpret_cast<uintptr_t>(ci) | reinterpret_cast<uintptr_t>(cj)) & 15) == 0;
    if (vec) hipLaunchKernelGGL(ttv_count_kernel<true>, dim3(nch), dim3(kBlock), 0, s, nnz, ci, cj, heads);
    else hipLaunchKernelGGL(ttv_count_kernel<false>, dim3(nch), dim3(kBlock), 0, s, nnz, ci, cj, heads);
    SPT_CHECK_LAUNCH("ttm count");
    spt_status st = device_scan_i32<false>(heads, off, nch, scan_tmp, s);
    if (st != SPT_OK) return st;
    hipLaunchKernelGGL(ttv_total_kernel, dim3(1), dim3(kWave), 0, s, nch, heads, off, out_nfib);
    SPT_CHECK_LAUNCH("ttm total");
    if (vec)  // fid comes from the 256-byte aligned workspace
      hipLaunchKernelGGL(fiber_ids_kernel<true>, dim3(nch), dim3(kBlock), 0, s, nnz, ci, cj, off, fid,
                         out_i, out_j);
    else
      hipLaunchKernelGGL(fiber_ids_kernel<false>, dim3(nch), dim3(kBlock), 0, s, nnz, ci, cj, off, fid,
                         out_i, out_j);
    SPT_CHECK_LAUNCH("ttm fiber ids");
  } else {
    const int64_t nfib = B->level[2].M;
    if (nfib + 1 >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "ttm: tensor too large");
    if (out_nfib) {
      hipLaunchKernelGGL(set_i64_kernel, dim3(1), dim3(kWave), 0, s, out_nfib, nfib);
      SPT_CHECK_LAUNCH("ttm set count");
    }
    hipLaunchKernelGGL(expand_fiber_ids_kernel, dim3((unsigned)((nfib + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, (int)nfib, B->level[2].pos, fid);
    SPT_CHECK_LAUNCH("ttm expand fibre ids");
    hipLaunchKernelGGL(zero_empty_fibres_kernel<T>, dim3((unsigned)((nfib + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, (int)nfib, K, B->level[2].pos, out_v);
    SPT_CHECK_LAUNCH("ttm zero empty fibres");
  }
  hipLaunchKernelGGL(transpose_kernel<T>, dim3((unsigned)((L * K + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, K, L, C, Ct);
  SPT_CHECK_LAUNCH("ttm transpose");
  void* rest = static_cast<char*>(ws) + W.used;
  return spdm_typed<T>(B, Ct, K, out_v, rest, ws_bytes - W.used, s, fid,
                         B->level[2].crd);
}

spt_status ttm_dispatch(Format f, const spt_tensor* B, const void* C, int32_t K, int32_t* out_crd0,
                        int32_t* out_crd1, void* out_vals, int64_t* out_nfib_dev, void* ws,
                        size_t ws_bytes, hipStream_t s) {
  for (int k = 0; k < 3; ++k)
    if (!(B->level[k].flags & SPT_ORDERED))
      return fail(SPT_ERR_UNSUPPORTED, "ttm: every level of B must be ordered");
  if (B->dtype == SPT_F64)
    return ttm_typed<double>(f, B, static_cast<const double*>(C), K, out_crd0, out_crd1,
                             static_cast<double*>(out_vals), out_nfib_dev, ws, ws_bytes, s);
  return ttm_typed<float>(f, B, static_cast<const float*>(C), K, out_crd0, out_crd1,
                          static_cast<float*>(out_vals), out_nfib_dev, ws, ws_bytes, s);
}

// ttv_wave.hip
bool ttv_csf_applies(int64_t nnz, int64_t nfib, int64_t K, int dtype);
bool ttv_wave_applies(int64_t nnz, int64_t K, int dtype);
size_t ttv_coo_workspace(int64_t nnz);
size_t ttv_csf_wave_workspace(int64_t nnz);
template <typename T>
spt_status ttv_coo(int64_t nnz, int64_t K, const int32_t* ci, const int32_t* cj, const int32_t* ck,
                   const T* vals, const T* c, int32_t* out_i, int32_t* out_j, T* out_v, int64_t* out_nnz,
                   void* ws, size_t ws_bytes, hipStream_t s);
template <typename T>
spt_status ttv_csf_wave(int64_t nnz, int64_t nfib, int64_t K, const int32_t* pos, const int32_t* ck,
                        const T* vals, const T* c, T* out_v, int64_t* out_count, void* ws, size_t ws_bytes,
                        hipStream_t s);

size_t ttv_workspace(Format f, const spt_tensor* B) {
  if (f == Format::COO3) return ttv_coo_workspace(B->nvals);
  return ttv_csf_applies(B->nvals, B->level[2].M, B->level[2].N, B->dtype) ? ttv_csf_wave_workspace(B->nvals)
                                                                           : seg_spmv_workspace(B->nvals);
}

spt_status ttv_dispatch(Format f, const spt_tensor* B, const void* c, int32_t* out_crd0,
                        int32_t* out_crd1, void* out_vals, int64_t* out_nnz_dev, void* ws,
                        size_t ws_bytes, hipStream_t s) {
  for (int k = 0; k < 3; ++k)
    if (!(B->level[k].flags & SPT_ORDERED))
      return fail(SPT_ERR_UNSUPPORTED, "ttv: every level of B must be ordered");
  if (f == Format::CSF3) {
    // The bottom level is a compressed level over the fibers: the same row
    // reduction as CSR SpMV with rows = fibers and x = c.
    const int64_t nfib = B->level[2].M;
    // (with less workspace than pieces take, a tensor of a long c is reduced as rows all the same)
    if (ttv_csf_applies(B->nvals, nfib, B->level[2].N, B->dtype) &&
        (ttv_wave_applies(B->nvals, B->level[2].N, B->dtype) ||
         (ws && ws_bytes >= ttv_csf_wave_workspace(B->nvals)))) {  // writes the count itself
      if (B->dtype == SPT_F64)
        return ttv_csf_wave<double>(B->nvals, nfib, B->level[2].N, B->level[2].pos, B->level[2].crd,
                                    static_cast<const double*>(B->vals), static_cast<const double*>(c),
                                    static_cast<double*>(out_vals), out_nnz_dev, ws, ws_bytes, s);
      return ttv_csf_wave<float>(B->nvals, nfib, B->level[2].N, B->level[2].pos, B->level[2].crd,
                                 static_cast<const float*>(B->vals), static_cast<const float*>(c),
                                 static_cast<float*>(out_vals), out_nnz_dev, ws, ws_bytes, s);
    }
    if (out_nnz_dev) {
      hipLaunchKernelGGL(set_i64_kernel, dim3(1), dim3(kWave), 0, s, out_nnz_dev, nfib);
      SPT_CHECK_LAUNCH("ttv set count");
    }
    return csr_rows_reduce(B->dtype, B->nvals, nfib, B->level[2].pos, B->level[2].crd, B->vals, c,
                           out_vals, ws, ws_bytes, s);
  }
  if (B->nvals == 0) {
    hipLaunchKernelGGL(set_i64_kernel, dim3(1), dim3(kWave), 0, s, out_nnz_dev, (int64_t)0);
    SPT_CHECK_LAUNCH("ttv set count");
    return SPT_OK;
  }
  const int32_t *ci = B->level[0].crd, *cj = B->level[1].crd, *ck = B->level[2].crd;
  if (B->dtype == SPT_F64)
    return ttv_coo<double>(B->nvals, B->level[2].N, ci, cj, ck, static_cast<const double*>(B->vals),
                           static_cast<const double*>(c), out_crd0, out_crd1, static_cast<double*>(out_vals),
                           out_nnz_dev, ws, ws_bytes, s);
  return ttv_coo<float>(B->nvals, B->level[2].N, ci, cj, ck, static_cast<const float*>(B->vals),
                        static_cast<const float*>(c), out_crd0, out_crd1, static_cast<float*>(out_vals),
                        out_nnz_dev, ws, ws_bytes, s);
}

}  // namespace spt
