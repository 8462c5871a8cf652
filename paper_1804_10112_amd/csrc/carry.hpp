// What follows a segmented reduction that was split evenly: adding up the carries.
#pragma once
#include "common.hpp"
#include "wavescan.hpp"

namespace spt {

// A choice between kernels made on the device: the workgroups of an earlier kernel write kChoiceFlags flags, the
// candidates are launched, and each looks whether it is the one. By rows unless a block of rows is heavy or the
// columns lie scattered; scattered if more than half of the flags that tell about columns say so.
constexpr int kChoiceFlags = 256;  // bytes, four per lane of a wave
constexpr int kChoiceHeavy = 1, kChoiceScattered = 2, kChoiceTells = 4;
enum { kByRows, kByEntries, kBySlices };
__device__ __forceinline__ int read_choice(const uint8_t* __restrict__ flags) {
  const uint32_t f = reinterpret_cast<const uint32_t*>(flags)[lane_id()];
  int scattered = 0, tells = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    scattered += __popcll(__ballot(f >> (8 * q) & kChoiceScattered));
    tells += __popcll(__ballot(f >> (8 * q) & kChoiceTells));
  }
  return 2 * scattered > tells ? kBySlices : __ballot(f & 0x01010101u * kChoiceHeavy) ? kByEntries : kByRows;
}
__device__ __forceinline__ bool selected(const uint8_t* __restrict__ select, int want) {
  return !select || (read_choice(select) != kByRows) == want;
}

// Adds the carries to y: carries of one row are consecutive, key -1 means no carry. A wave has 64
// carries; the one that holds the first of a row adds the whole row, reading on, 64 carries and then 64 U at a
// time, as long as they belong to it (a fixed order, so deterministic). The sums are formed in double
// also for float data. Bound by latency: one thread per row, reading the row's carries one after the
// other, took 28 us for rows of 190 carries, and each launch of few carries is 2 us. U = 16 where a row may have
// thousands of carries (one of 4700, 60M entries, fp32, local columns: 197 -> 162 us).
template <typename T, int U = 1>
__global__ __launch_bounds__(kBlock) void carry_fixup_kernel(int n,
                                                             const int32_t* __restrict__ carry_key,
                                                             const T* __restrict__ carry_val,
                                                             T* __restrict__ y,
                                                             const uint8_t* __restrict__ select = nullptr,
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
  // the next 64 carries, then 1024 a round
  int64_t p = static_cast<int64_t>(w) + kWave;
  if (more) {
    const bool match = p < n && carry_key[p < n ? p : n - 1] == open;
    const double t = wave_total<double>(match ? static_cast<double>(carry_val[p]) : 0.0);
    if (last) sum += t;
    more = __ballot(match) == ~uint64_t{0};
    p += kWave;
  }
  while (more) {
    int32_t k[U];
    T c[U];
    double t = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t at = p + u * kWave < n ? p + u * kWave : n - 1;
      k[u] = carry_key[at];
      c[u] = carry_val[at];
    }
    uint64_t all = ~uint64_t{0};
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool match = all == ~uint64_t{0} && p + u * kWave < n && k[u] == open;
      all = __ballot(match);
      t += match ? static_cast<double>(c[u]) : 0.0;
    }
    more = all == ~uint64_t{0};
    t = wave_total<double>(t);
    if (last) sum += t;
    p += U * kWave;
  }
  if (mine) y[key] = static_cast<T>(static_cast<double>(y[key]) + sum);
}

}  // namespace spt
