// Searches by several lanes of a wave at once.
#pragma once
#include "common.hpp"

namespace spt {
#if defined(__HIPCC__)

// Largest r in [lo, hi) for which p(r) holds; p(lo) does, and p turns false at most once. Groups of
// W lanes search together, W probes a step.
template <int W, typename P>
__device__ __forceinline__ int group_last_true(int64_t lo, int64_t hi, P p) {
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + W - 1) / W;
    const int64_t at = lo + lane_id() % W * step;
    const uint64_t holds = __ballot(at < hi && p(static_cast<int>(at))) >> (lane_id() / W * W);
    lo += max(__popcll(W < kWave ? holds & ((uint64_t{1} << (W % kWave)) - 1) : holds) - 1, 0) * step;
    hi = min(hi, lo + step);
  }
  return static_cast<int>(lo);
}

#endif
}  // namespace spt
