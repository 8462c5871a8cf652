// Sorting of 32-bit words by one workgroup, in registers.
#pragma once
#include "common.hpp"

namespace spt {

// Lane exchange with lane ^ MASK, through the vector ALU where a lane movement of it exists.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v) {
  if constexpr (MASK == 0) return v;
  else if constexpr (MASK == 1) return dpp_u32<0xB1>(v);        // quad_perm 1,0,3,2
  else if constexpr (MASK == 2) return dpp_u32<0x4E>(v);        // quad_perm 2,3,0,1
  else if constexpr (MASK == 3) return dpp_u32<0x1B>(v);        // quad_perm 3,2,1,0
  else if constexpr (MASK == 7) return dpp_u32<0x141>(v);       // row_half_mirror
  else if constexpr (MASK == 4) return dpp_u32<0x1B>(dpp_u32<0x141>(v));
  else if constexpr (MASK == 8) return dpp_u32<0x128>(v);       // row_ror:8
  else if constexpr (MASK == 15) return dpp_u32<0x140>(v);      // row_mirror
  else if constexpr (MASK < 32)
    return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(static_cast<int>(v), (MASK << 10) | 0x1f));
  else return static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), MASK));
}

// The smaller of a and b where `bound` is 0, the larger where it is ~0.
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t bound) {
  uint32_t r;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(bound));
  return r;
}

// One comparison step of the network below: partner of key i = tid * E + e is i ^ MASK, MASK being
// either one bit (a stride) or all bits below a power of two (the mirror step that opens a phase).
template <int NT, int E, int MASK>
__device__ __forceinline__ void bitonic_step(uint32_t (&v)[E], uint32_t* buf) {
  constexpr int TOP = MASK & (MASK + 1) ? MASK : (MASK + 1) / 2;  // the bit that tells the pair apart
  if constexpr (MASK < E) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (!(e & TOP)) {
        const uint32_t a = v[e], b = v[e ^ MASK];
        v[e] = min(a, b);
        v[e ^ MASK] = max(a, b);
      }
    }
  } else {
    const int tid = threadIdx.x;
    constexpr int LM = MASK / E;       // partner thread: tid ^ LM
    constexpr int EM = MASK & (E - 1); // its key: e ^ EM
    const uint32_t bound = (tid & (TOP / E)) ? ~0u : 0u;
    uint32_t o[E];
    if constexpr (LM < kWave) {
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = lane_xor_u32<LM>(v[e ^ EM]);
    } else {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < E; ++e) buf[e * NT + tid] = v[e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = buf[(e ^ EM) * NT + (tid ^ LM)];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = med3_u32(v[e], o[e], bound);
  }
}
template <int NT, int E, int J>
__device__ __forceinline__ void bitonic_strides(uint32_t (&v)[E], uint32_t* buf) {
  if constexpr (J >= 1) {
    bitonic_step<NT, E, J>(v, buf);
    bitonic_strides<NT, E, J / 2>(v, buf);
  }
}
template <int NT, int E, int K>
__device__ __forceinline__ void bitonic_phases(uint32_t (&v)[E], uint32_t* buf) {
  if constexpr (K <= NT * E) {
    bitonic_step<NT, E, K - 1>(v, buf);
    bitonic_strides<NT, E, K / 4>(v, buf);
    bitonic_phases<NT, E, K * 2>(v, buf);
  }
}

// Ascending sort of the NT * E 32-bit words of the workgroup (powers of two): a bitonic network in
// registers whose steps cost a lane movement and one v_med3 per word; only the few steps between
// waves go through LDS. (A merge sort of 64-bit keys in LDS took three times as long, a bitonic
// network on 64-bit keys five times: compare-and-select of two registers.) On return buf[0 .. NT * E) holds the words in order, visible to all
// threads. buf must be 16-byte aligned.
// In two steps: the network, after which thread t holds words t * E .. t * E + E - 1, and the store.
template <int NT, int E>
__device__ __forceinline__ void block_sort_regs(uint32_t (&v)[E], uint32_t* buf) {
  bitonic_phases<NT, E, 2>(v, buf);
  __syncthreads();
}
template <int NT, int E>
__device__ __forceinline__ void block_sort_store(const uint32_t (&v)[E], uint32_t* buf) {
#pragma unroll
  for (int e = 0; e < E; ++e) buf[threadIdx.x * E + e] = v[e];
  __syncthreads();
}
template <int NT, int E>
__device__ __forceinline__ void block_sort_u32(uint32_t (&v)[E], uint32_t* buf) {
  block_sort_regs<NT, E>(v, buf);
  block_sort_store<NT, E>(v, buf);
}

}  // namespace spt
