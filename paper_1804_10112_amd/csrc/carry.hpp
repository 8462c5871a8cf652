// What follows a segmented reduction that was split evenly: adding up the carries.
#pragma once
#include "common.hpp"
#include "wavescan.hpp"

namespace spt {

// A choice between two kernels made on the device: an earlier kernel writes kSelectFlags flags,
// both candidates are launched, and each runs only if "any flag set" equals its `want`.
constexpr int kSelectFlags = 64;  // one per lane of a wave
__device__ __forceinline__ bool selected(const int32_t* __restrict__ select, int want) {
  if (!select) return true;
  const int any = __ballot(select[threadIdx.x & (kSelectFlags - 1)] != 0) != 0;
  return any == want;
}

// Adds the carries to y: carries of one row are consecutive, key -1 means no carry. A wave has 64
// carries; the one that holds the first of a row adds the whole row, reading on, 64 carries at a
// time, as long as they belong to it (a fixed order, so deterministic). The sums are formed in double
// also for float data. Bound by latency: one thread per row, reading the row's carries one after the
// other, took 28 us for rows of 190 carries, and each launch of few carries is 2 us.
template <typename T>
__global__ __launch_bounds__(kBlock) void carry_fixup_kernel(int n,
                                                             const int32_t* __restrict__ carry_key,
                                                             const T* __restrict__ carry_val,
                                                             T* __restrict__ y,
                                                             const int32_t* __restrict__ select = nullptr,
                                                             int want = 0) {
  if (!selected(select, want)) return;
  const int w = blockIdx.x * kBlock + threadIdx.x, lane = lane_id();
  if (w - lane >= n) return;
  const int32_t key = w < n ? carry_key[w] : -1;
  const double v = w < n && key >= 0 ? static_cast<double>(carry_val[w]) : 0.0;
  int32_t prev = dpp_move<0x138, 0xf>(-1, key);  // wave_shr:1
  if (lane == 0) prev = w > 0 ? carry_key[w - 1] : -1;
  const uint64_t heads = __ballot(key != prev);
  const int from = last_lane(heads, false);
  double sum = wave_marked_sum(v, from >= 0 ? lane - from : kWave);
  const bool last = lane == kWave - 1;
  const bool ends = last || (heads >> (lane + 1) & 1);
  const bool mine = from >= 0 && key >= 0 && ends;
  bool more = __shfl(static_cast<int>(mine), kWave - 1);
  const int32_t open = __shfl(key, kWave - 1);
  for (int p = w - lane + kWave; more; p += kWave) {
    const bool match = p + lane < n && carry_key[min(p + lane, n - 1)] == open;
    const double t = wave_total<double>(match ? static_cast<double>(carry_val[p + lane]) : 0.0);
    if (last) sum += t;
    more = __ballot(match) == ~uint64_t{0};
  }
  if (mine) y[key] = static_cast<T>(static_cast<double>(y[key]) + sum);
}

}  // namespace spt
