// Gathers from a vector that no L2 holds, slice by slice, in registers.
#pragma once
#include <algorithm>

#include "common.hpp"

namespace spt {

// An x that an L2 holds need not be cut. The upper line lies where passes over slices of 3.2 MB came to cost about what
// the lines did. With the larger slices of slices_of it is cautious: 60M entries, x of 126 MB sliced, fp64 810 and fp32 645 us,
// of 130 MB not sliced 1231 and 1190.
constexpr int64_t kSlicesMinX = 6000000, kSlicesMaxX = 128000000;

// Slices of an x, of which an XCD gathers `entries` / kXcds entries at a time (`entries`: of all). A slice that an L2
// holds next to what streams through it, 3.2 MB, where a line of x serves several of them; where it serves fewer, a miss more
// or less counts less than one more slice to go through: up to 5.6 MB. Whole product of 60M entries (40M: marked), uniform
// columns, with slices of 3.2 / 4.2 / 5.4 / 7 MB, us:
//   x, MB             32 (power law)          48 (40M)               64                     96                    120
//   fp64      547 / 573 / 627 /  -     432 / 415 / 420 / 474  721 / 671 / 657 / 706  938 / 817 / 778 / 796  1094 / 953 / 877 / 860
//   fp32                                                       584 / 590 / 632 / 701                        728 / 734 / 736 / 781
inline int slices_of(int64_t ncols, int64_t value, int64_t entries) {
  const int64_t x = ncols * value;
  const double of_a_line = static_cast<double>(entries) / kXcds / (static_cast<double>(x) / 128);
  const int64_t bytes = static_cast<int64_t>(3200000 * std::min(std::max(4.5 / of_a_line, 1.0), 1.75));
  return static_cast<int>((x + bytes - 1) / bytes);
}

// A workgroup of the sliced product on every compute unit; entries to a lane, of one kernel and of the other.
constexpr int kSliceBlock = 1024, kCus = 256, kFewEntries = 32;
template <typename T>
constexpr int kInPlace = sizeof(T) == 8 ? 40 : 64;

// Do the lanes hold kInPlace entries or 32? The chip goes over x in rounds of what all lanes hold; a round of more entries
// looks at more registers in every slice, filled or not, and each round brings the lines of x. So what counts is
// how many registers all rounds look at, and, where the two kernels are about equal in that, whether the lines of fewer
// rounds are many. 32 entries to a lane / kInPlace, us (rounds):
//   COO, fp64, x, MB     8          16          32          64         126
//     21M (3, 3)     169 / 174   180 / 188   208 / 221   256 / 268   319 / 333
//     26M (4, 3)     212 / 210   227 / 222   264 / 256   328 / 305   404 / 389
//     33M (4, 4)     263 / 268   279 / 285   315 / 329   386 / 394   481 / 502
//     38M (5, 4)     294 / 306   314 / 322   359 / 363   457 / 439   559 / 556
//     51M (7, 5)     396 / 396   424 / 415   493 / 472   644 / 573   760 / 725
//     56M (7, 6)     432 / 439   459 / 463   529 / 529   687 / 646   823 / 814
//     75M (9, 8)     570 / 623   606 / 654   700 / 730   919 / 901  1077 / 1132
//   CSR, fp64: 34M (5, 4) 256 / 261, 276 / 278, 322 / 322, 399 / 385; 47M (6, 5) 345 / 341, 368 / 360, 424 / 415, 528 / 502
//   COO, fp32 (whose kernel of more entries has no slower looks): 18M (3, 2) 142 / 148, 155 / 158, 180 / 183, 232 / 222; 28M
//     (4, 2) 212 / 209, 229 / 220, 263 / 241, 345 / 286; 51M (7, 4) 373 / 371, 414 / 394, 483 / 445, 650 / 537
// (COO, fp64, 18M (3, 2), x of 8 MB 148 / 150: three rounds over little.)
template <typename T>
inline bool slices_of_many(int64_t nnz, int64_t ncols, bool csr) {
  const auto rounds = [&](int entries) { return (nnz - 1) / (int64_t(kSliceBlock) * kCus * entries) + 1; };
  const int64_t x = ncols * static_cast<int64_t>(sizeof(T)), few = rounds(kFewEntries) * kFewEntries, many = rounds(kInPlace<T>) * kInPlace<T>;
  if (sizeof(T) == 4) return many * 4 <= few * 5 || x > 36000000;
  if (many < few) return csr || x > 12000000 || rounds(kFewEntries) > 3;
  return many * 25 <= few * 27 && x > (csr ? 12000000 : 40000000);
}

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

// The same with more entries to a lane: got[k] holds the byte offset of entry k in its first 32 bits, and the value takes
// its place, in the registers from v48 on, which are named here since an operand's first half has no name. What is still
// to be gathered is kept as a bit per entry: a register may look like an offset once its load has been issued, or be
// read while the load is on its way, in lanes whose bit is cleared. An offset beyond every slice is left as it is.
template <typename T>
struct SliceGatherInPlace;

// (entry, its bit, of which register, the registers of its value)
#define SPT_PLACES_double(M) \
  M(0, 0x1, 0, 48, 49) M(1, 0x2, 0, 50, 51) M(2, 0x4, 0, 52, 53) M(3, 0x8, 0, 54, 55) M(4, 0x10, 0, 56, 57) M(5, 0x20, 0, 58, 59) \
   M(6, 0x40, 0, 60, 61) M(7, 0x80, 0, 62, 63) M(8, 0x100, 0, 64, 65) M(9, 0x200, 0, 66, 67) M(10, 0x400, 0, 68, 69) M(11, 0x800, 0, 70, 71) \
   M(12, 0x1000, 0, 72, 73) M(13, 0x2000, 0, 74, 75) M(14, 0x4000, 0, 76, 77) M(15, 0x8000, 0, 78, 79) M(16, 0x10000, 0, 80, 81) M(17, 0x20000, 0, 82, 83) \
   M(18, 0x40000, 0, 84, 85) M(19, 0x80000, 0, 86, 87) M(20, 0x100000, 0, 88, 89) M(21, 0x200000, 0, 90, 91) M(22, 0x400000, 0, 92, 93) M(23, 0x800000, 0, 94, 95) \
   M(24, 0x1000000, 0, 96, 97) M(25, 0x2000000, 0, 98, 99) M(26, 0x4000000, 0, 100, 101) M(27, 0x8000000, 0, 102, 103) M(28, 0x10000000, 0, 104, 105) M(29, 0x20000000, 0, 106, 107) \
   M(30, 0x40000000, 0, 108, 109) M(31, 0x80000000, 0, 110, 111) M(32, 0x1, 1, 112, 113) M(33, 0x2, 1, 114, 115) M(34, 0x4, 1, 116, 117) M(35, 0x8, 1, 118, 119) \
   M(36, 0x10, 1, 120, 121) M(37, 0x20, 1, 122, 123) M(38, 0x40, 1, 124, 125) M(39, 0x80, 1, 126, 127)
#define SPT_PLACES_float(M) \
  M(0, 0x1, 0, 48, 48) M(1, 0x2, 0, 49, 49) M(2, 0x4, 0, 50, 50) M(3, 0x8, 0, 51, 51) M(4, 0x10, 0, 52, 52) M(5, 0x20, 0, 53, 53) \
   M(6, 0x40, 0, 54, 54) M(7, 0x80, 0, 55, 55) M(8, 0x100, 0, 56, 56) M(9, 0x200, 0, 57, 57) M(10, 0x400, 0, 58, 58) M(11, 0x800, 0, 59, 59) \
   M(12, 0x1000, 0, 60, 60) M(13, 0x2000, 0, 61, 61) M(14, 0x4000, 0, 62, 62) M(15, 0x8000, 0, 63, 63) M(16, 0x10000, 0, 64, 64) M(17, 0x20000, 0, 65, 65) \
   M(18, 0x40000, 0, 66, 66) M(19, 0x80000, 0, 67, 67) M(20, 0x100000, 0, 68, 68) M(21, 0x200000, 0, 69, 69) M(22, 0x400000, 0, 70, 70) M(23, 0x800000, 0, 71, 71) \
   M(24, 0x1000000, 0, 72, 72) M(25, 0x2000000, 0, 73, 73) M(26, 0x4000000, 0, 74, 74) M(27, 0x8000000, 0, 75, 75) M(28, 0x10000000, 0, 76, 76) M(29, 0x20000000, 0, 77, 77) \
   M(30, 0x40000000, 0, 78, 78) M(31, 0x80000000, 0, 79, 79) M(32, 0x1, 1, 80, 80) M(33, 0x2, 1, 81, 81) M(34, 0x4, 1, 82, 82) M(35, 0x8, 1, 83, 83) \
   M(36, 0x10, 1, 84, 84) M(37, 0x20, 1, 85, 85) M(38, 0x40, 1, 86, 86) M(39, 0x80, 1, 87, 87) M(40, 0x100, 1, 88, 88) M(41, 0x200, 1, 89, 89) \
   M(42, 0x400, 1, 90, 90) M(43, 0x800, 1, 91, 91) M(44, 0x1000, 1, 92, 92) M(45, 0x2000, 1, 93, 93) M(46, 0x4000, 1, 94, 94) M(47, 0x8000, 1, 95, 95) \
   M(48, 0x10000, 1, 96, 96) M(49, 0x20000, 1, 97, 97) M(50, 0x40000, 1, 98, 98) M(51, 0x80000, 1, 99, 99) M(52, 0x100000, 1, 100, 100) M(53, 0x200000, 1, 101, 101) \
   M(54, 0x400000, 1, 102, 102) M(55, 0x800000, 1, 103, 103) M(56, 0x1000000, 1, 104, 104) M(57, 0x2000000, 1, 105, 105) M(58, 0x4000000, 1, 106, 106) M(59, 0x8000000, 1, 107, 107) \
   M(60, 0x10000000, 1, 108, 108) M(61, 0x20000000, 1, 109, 109) M(62, 0x40000000, 1, 110, 110) M(63, 0x80000000, 1, 111, 111)
#define SPT_PLACE_OPERAND_double(K, BIT, W, LO, HI) "+{v[" #LO ":" #HI "]}"(got[K]),
#define SPT_PLACE_OPERAND_float(K, BIT, W, LO, HI) "+{v" #LO "}"(got[K]),
#define SPT_PLACE_LOAD_double(LO, HI) "global_load_dwordx2 v[" #LO ":" #HI "], v" #LO ", %[x]\n"
#define SPT_PLACE_LOAD_float(LO, HI) "global_load_dword v" #LO ", v" #LO ", %[x]\n"
#define SPT_PLACE_STEP(T, K, BIT, W, LO, HI)       \
  "s_mov_b64 exec, %[all]\n\t"                     \
  "v_and_b32 %[bit], " #BIT ", %[todo" #W "]\n\t"  \
  "v_subrev_u32 %[rel], %[lo], v" #LO "\n\t"       \
  "v_cmpx_gt_u32 vcc, %[bytes], %[rel]\n\t"        \
  "v_cmpx_ne_u32 vcc, 0, %[bit]\n\t"               \
  "s_cbranch_execz 1f\n\t"                         \
  "v_xor_b32 %[todo" #W "], " #BIT ", %[todo" #W "]\n\t" SPT_PLACE_LOAD_##T(LO, HI) \
  "1:\n\t"
#define SPT_PLACE_STEP_double(K, BIT, W, LO, HI) SPT_PLACE_STEP(double, K, BIT, W, LO, HI)
#define SPT_PLACE_STEP_float(K, BIT, W, LO, HI) SPT_PLACE_STEP(float, K, BIT, W, LO, HI)
#define SPT_GATHER_IN_PLACE(T)                                                                                    \
  template <>                                                                                                     \
  struct SliceGatherInPlace<T> {                                                                                  \
    static __device__ __forceinline__ void run(const T* x, int n, uint32_t bytes, T (&got)[kInPlace<T>]) {        \
      uint32_t lo, rel, bit, todo0 = ~0u, todo1 = ~0u;                                                            \
      uint64_t all;                                                                                               \
      asm volatile("s_mov_b64 %[all], exec\n\t"                                                                   \
                   "s_mov_b32 %[lo], 0\n"                                                                         \
                   "0:\n\t" SPT_PLACES_##T(SPT_PLACE_STEP_##T)                                                    \
                   "s_mov_b64 exec, %[all]\n\t"                                                                   \
                   "s_barrier\n\t"                                                                                \
                   "s_add_u32 %[lo], %[lo], %[bytes]\n\t"                                                         \
                   "s_sub_u32 %[n], %[n], 1\n\t"                                                                  \
                   "s_cmp_lg_u32 %[n], 0\n\t"                                                                     \
                   "s_cbranch_scc1 0b\n\t"                                                                        \
                   "s_waitcnt vmcnt(0)"                                                                           \
                   : SPT_PLACES_##T(SPT_PLACE_OPERAND_##T)[n] "+&s"(n), [lo] "=&s"(lo), [all] "=&s"(all),         \
                     [rel] "=&v"(rel), [bit] "=&v"(bit), [todo0] "+&v"(todo0), [todo1] "+&v"(todo1)                \
                   : [bytes] "s"(bytes), [x] "s"(x)                                                               \
                   : "vcc", "scc", "memory");                                                                     \
    }                                                                                                             \
  };
SPT_GATHER_IN_PLACE(double)
SPT_GATHER_IN_PLACE(float)

}  // namespace spt
