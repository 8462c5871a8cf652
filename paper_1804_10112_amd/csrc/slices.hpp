// Gathers from a vector that no L2 holds, slice by slice, in registers.
#pragma once
#include "common.hpp"

namespace spt {

// An x that an L2 holds need not be cut; beyond some 150 MB the passes cost more than the lines.
constexpr int64_t kSlicesMinX = 6000000, kSlicesMaxX = 128000000, kSliceBytes = 3200000;

constexpr int kSegment = 4 * kWave;  // consecutive entries that a wave reduces at a time

// The row kernel as one of two candidates: where the choice is made, and what it leaves behind for the other if
// it is not chosen (seg_row, or null).
struct ByRowsIf {
  const uint8_t* flags;
  int32_t* seg_row;
  int nseg;
};

// seg_row[s] = the first row that starts at or after entry s * kSegment, for s = 0 .. nseg - 1; seg_row[nseg] = nrows.
// Rows without entries are zeroed in y. By all workgroups of kBlock threads.
template <typename T>
__device__ __forceinline__ void find_segment_rows(int nrows, const int32_t* __restrict__ pos, int nseg,
                                                  int32_t* __restrict__ seg_row, T* __restrict__ y) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    seg_row[0] = 0;
    seg_row[nseg] = nrows;
  }
  for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * kBlock; r0 < nrows; r0 += static_cast<int64_t>(gridDim.x) * kBlock) {
    const int64_t r = r0 + threadIdx.x;
    int s = 0, last = -1;
    if (r < nrows) {
      const int a = pos[r], b = pos[r + 1];
      if (a == b) y[r] = T(0);
      s = a / kSegment + 1;
      last = min(b / kSegment, nseg - 1);
    }
    const bool far = last - s >= 8;
    if (!far)
      for (int q = s; q <= last; ++q) seg_row[q] = static_cast<int>(r) + 1;
    uint64_t todo = __ballot(far);
    while (todo) {  // a long row: the whole wave
      const int src = __ffsll(static_cast<long long>(todo)) - 1;
      todo &= todo - 1;
      const int s0 = __builtin_amdgcn_readlane(s, src), s1 = __builtin_amdgcn_readlane(last, src);
      const int after = __builtin_amdgcn_readlane(static_cast<int>(r), src) + 1;
      for (int t = s0 + lane_id(); t <= s1; t += kWave) seg_row[t] = after;
    }
  }
}

// got[k] = the value at byte offset at[k] of x, where that lies inside n slices of `bytes`; left alone where it
// lies beyond. A lane has N offsets; each slice in turn, the loads of those that fall into it are issued, all
// others masked off, and the workgroup meets before the next slice, so that what its waves ask for at a time
// lies in one slice of x. All waves of the workgroup call.
// Written out because of what the compiler makes of the same loop: a load under a mask into a register that
// holds something goes through a copy and a wait, and 32 of them spill (1.2 to 1.9 ms for what takes 0.5 here).
// A load no lane needs is jumped over: it would keep the address unit busy for some 20 clocks.
// What is written while offsets are still to be read is marked so (&): no operand may share its register.
template <typename T, int N>
struct SliceGather;

#define SPT_EACH10(M, A) M(A##0) M(A##1) M(A##2) M(A##3) M(A##4) M(A##5) M(A##6) M(A##7) M(A##8) M(A##9)
#define SPT_ONE_TO_NINE(M) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9)
#define SPT_EACH32(M) M(0) SPT_ONE_TO_NINE(M) SPT_EACH10(M, 1) SPT_EACH10(M, 2) M(30) M(31)
#define SPT_GATHER_RESULT(K) [g##K] "+&v"(got[K]),
#define SPT_GATHER_OFFSET(K) [a##K] "v"(at[K]),
#define SPT_GATHER_LOAD(WIDTH, K)                  \
  "s_mov_b64 exec, %[all]\n\t"                     \
  "v_subrev_u32 %[rel], %[lo], %[a" #K "]\n\t"     \
  "v_cmpx_gt_u32 vcc, %[bytes], %[rel]\n\t"        \
  "s_cbranch_execz 1f\n\t"                         \
  "global_load_" WIDTH " %[g" #K "], %[a" #K "], %[x]\n" \
  "1:\n\t"
#define SPT_GATHER_LOAD1(K) SPT_GATHER_LOAD("dword", K)
#define SPT_GATHER_LOAD2(K) SPT_GATHER_LOAD("dwordx2", K)
#define SPT_SLICE_GATHER(T, N, LOAD)                                                                              \
  template <>                                                                                                     \
  struct SliceGather<T, N> {                                                                                      \
    static __device__ __forceinline__ void run(const T* x, int n, uint32_t bytes, const uint32_t (&at)[N],        \
                                               T (&got)[N]) {                                                     \
      uint32_t lo, rel;                                                                                           \
      uint64_t all;                                                                                               \
      asm volatile("s_mov_b64 %[all], exec\n\t"                                                                   \
                   "s_mov_b32 %[lo], 0\n"                                                                         \
                   "0:\n\t" SPT_EACH##N(LOAD)                                                                     \
                   "s_mov_b64 exec, %[all]\n\t"                                                                   \
                   "s_barrier\n\t"                                                                                \
                   "s_add_u32 %[lo], %[lo], %[bytes]\n\t"                                                         \
                   "s_sub_u32 %[n], %[n], 1\n\t"                                                                  \
                   "s_cmp_lg_u32 %[n], 0\n\t"                                                                     \
                   "s_cbranch_scc1 0b\n\t"                                                                        \
                   "s_waitcnt vmcnt(0)"                                                                           \
                   : SPT_EACH##N(SPT_GATHER_RESULT)[n] "+&s"(n), [lo] "=&s"(lo), [all] "=&s"(all), [rel] "=&v"(rel) \
                   : SPT_EACH##N(SPT_GATHER_OFFSET)[bytes] "s"(bytes), [x] "s"(x)                                 \
                   : "vcc", "scc", "memory");                                                                     \
    }                                                                                                             \
  };
SPT_SLICE_GATHER(double, 32, SPT_GATHER_LOAD2)
SPT_SLICE_GATHER(float, 32, SPT_GATHER_LOAD1)

}  // namespace spt
