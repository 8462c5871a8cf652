// Digits of the COO->CSR sort and of the binned COO SpMV, and the sort's histogram of them per tile.
#pragma once
#include "common.hpp"

namespace spt {

constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;
constexpr int kSortIPT = 16;
constexpr int kSortTile = kSortIPT * kBlock;  // 4096 records per workgroup
constexpr int kWaves = kBlock / kWave;

inline int bits_for(int64_t dim) {
  int b = 1;
  while (b < 31 && ((int64_t)1 << b) < dim) ++b;
  return b;
}

__device__ __forceinline__ int digit_of(int32_t key, int shift) {
  return ((uint32_t)key >> shift) & (kRadix - 1);
}

// A key's place among 256 equal stretches of a dimension (binning by rows): digit d begins at first(d).
struct StretchDigit {
  uint32_t mult;  // 2^32 * 256 / extent
  explicit StretchDigit(int64_t extent) {
    const uint64_t m = (uint64_t{kRadix} << 32) / static_cast<uint64_t>(extent > 0 ? extent : 1);
    mult = m > 0xFFFFFFFFu ? 0xFFFFFFFFu : static_cast<uint32_t>(m);
  }
  __host__ __device__ __forceinline__ int64_t first(int d) const {
    return static_cast<int64_t>(((static_cast<uint64_t>(d) << 32) + mult - 1) / mult);
  }
  int64_t most() const { return static_cast<int64_t>(((uint64_t{1} << 32) + mult - 1) / mult); }  // of one digit
  __device__ __forceinline__ int of(int32_t key) const { return __umulhi(static_cast<uint32_t>(key), mult); }
};

// The lanes of `among` whose eight bits are those of this one. What differs is gathered with a bit of d as 0 or ~0, against
// which both halves of the lanes that have it take one exclusive or each (selecting the lanes or their complement, the
// compiler needs twice as many instructions).
__device__ __forceinline__ uint64_t lanes_with(int d, uint64_t among) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int b = 0; b < kRadixBits; ++b) {
    const uint32_t bit = static_cast<uint32_t>(__builtin_amdgcn_sbfe(d, b, 1));
    const uint64_t vote = __ballot(bit != 0);
    lo |= static_cast<uint32_t>(vote) ^ bit;
    hi |= static_cast<uint32_t>(vote >> 32) ^ bit;
  }
  return among & ~(static_cast<uint64_t>(hi) << 32 | lo);
}

// One more key with digit d in each of the wave's 64 lanes (all active, lane order =
// key order up to a fixed stride). Sorted input (a long row, a long fibre) gives
// neighbouring lanes the same digit, and separate LDS atomics on one counter are
// serialised: the first lane of every run of equal digits adds the run's length.
__device__ __forceinline__ void count_digit_runs(int* cnt, int d) {
  const int lane = lane_id();
  // lane l receives lane l-1's digit through the data-parallel-primitive path
  // (wave_shr:1; lane 0 keeps its own), not through the LDS crossbar
  const int prev = __builtin_amdgcn_update_dpp(d, d, 0x138, 0xf, 0xf, false);
  const bool head = lane == 0 || d != prev;
  const uint64_t heads = __ballot(head);
  if (head) {
    const uint64_t above = lane == kWave - 1 ? 0 : heads >> (lane + 1);
    const int len = above ? __ffsll(static_cast<long long>(above)) : kWave - lane;
    atomicAdd(&cnt[d], len);
  }
}

// hist[d * ntiles + tile] = number of keys of this tile whose digit is d.
// A workgroup counts `group` (up to kHistGroup) consecutive tiles, each wave a quarter of a tile at
// a time into that tile's LDS counters, and thread d then stores digit d's counts of all
// its tiles side by side: the layout is digit-major for the scan that follows, and
// one count per tile and digit stored on its own would be a scattered 4-byte write.
// VEC: 16-byte key loads (needs a 16-byte aligned key array).
constexpr int kHistGroup = 8;
template <bool VEC>
__global__ __launch_bounds__(kBlock) void radix_hist_kernel(const int32_t* __restrict__ key, int n,
                                                            int shift, int ntiles, int group,
                                                            int32_t* __restrict__ hist) {
  __shared__ int s_cnt[kHistGroup][kRadix];
  for (int q = threadIdx.x; q < group * kRadix; q += kBlock) (&s_cnt[0][0])[q] = 0;
  __syncthreads();
  const int tile0 = xcd_contiguous_block_id() * group;  // neighbours store into the same cache lines
  const int lane = lane_id();
  constexpr int kPart = kSortTile / kWaves;
  for (int t = 0; t < group && tile0 + t < ntiles; ++t) {
    const int base = (tile0 + t) * kSortTile + wave_id() * kPart;
    int* cnt = s_cnt[t];
    if (VEC) {
      typedef int32_t i4 __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int q = 0; q < kPart / (4 * kWave); ++q) {
        const int i = base + (q * kWave + lane) * 4;
        if (base + (q + 1) * kWave * 4 <= n) {  // the whole wave is inside the array
          const i4 k4 = __builtin_nontemporal_load(reinterpret_cast<const i4*>(key + i));
#pragma unroll
          for (int r = 0; r < 4; ++r) count_digit_runs(cnt, digit_of(k4[r], shift));
        } else if (i + 4 <= n) {
          const i4 k4 = __builtin_nontemporal_load(reinterpret_cast<const i4*>(key + i));
#pragma unroll
          for (int r = 0; r < 4; ++r) atomicAdd(&cnt[digit_of(k4[r], shift)], 1);
        } else {
          for (int r = 0; r < 4; ++r)
            if (i + r < n) atomicAdd(&cnt[digit_of(key[i + r], shift)], 1);
        }
      }
    } else {
#pragma unroll 4
      for (int q = 0; q < kPart / kWave; ++q) {
        const int i = base + q * kWave + lane;
        if (i < n) atomicAdd(&cnt[digit_of(key[i], shift)], 1);
      }
    }
  }
  __syncthreads();
  const int nt = min(group, ntiles - tile0);
  int32_t* out = hist + (int64_t)threadIdx.x * ntiles + tile0;
  for (int t = 0; t < nt; ++t) out[t] = s_cnt[t][threadIdx.x];
}


#if defined(__HIPCC__)
// Enqueues the histogram of the digits for every tile of kSortTile keys.
inline spt_status launch_radix_hist(const int32_t* key, int n, int shift, int ntiles, int32_t* hist,
                                    hipStream_t s) {
  // few tiles: more, shorter workgroups (3.2M keys: 26 us with eight tiles each)
  const int group = ntiles >= 8192 ? kHistGroup : ntiles >= 2048 ? 2 : 1;
  if ((reinterpret_cast<uintptr_t>(key) & 15) == 0)
    hipLaunchKernelGGL((radix_hist_kernel<true>), dim3((ntiles + group - 1) / group),
                       dim3(kBlock), 0, s, key, n, shift, ntiles, group, hist);
  else
    hipLaunchKernelGGL((radix_hist_kernel<false>), dim3((ntiles + group - 1) / group),
                       dim3(kBlock), 0, s, key, n, shift, ntiles, group, hist);
  SPT_CHECK_LAUNCH("radix_hist");
  return SPT_OK;
}
#endif

}  // namespace spt
