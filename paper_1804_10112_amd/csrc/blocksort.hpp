// Sorting of 32-bit words by one workgroup, in registers.
#pragma once
#include <utility>

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

// Two words of a thread in order.
template <int A, int B, int E>
__device__ __forceinline__ void order_pair(uint32_t (&v)[E]) {
  const uint32_t a = v[A], b = v[B];
  v[A] = min(a, b);
  v[B] = max(a, b);
}

// The comparators of a merge exchange (Batcher's, as in Knuth 5.2.2 M), which orders any number of words.
template <int N>
struct MergeExchange {
  int a[N * 6] = {}, b[N * 6] = {}, count = 0;
  constexpr MergeExchange() {
    static_assert(N <= 16, "");
    int top = 1;
    while (top < N) top *= 2;
    for (int p = top / 2; p > 0; p /= 2) {
      int q = top / 2, r = 0, d = p;
      for (;;) {
        for (int i = 0; i + d < N; ++i) {
          if ((i & p) == r) {
            a[count] = i;
            b[count++] = i + d;
          }
        }
        if (q == p) break;
        d = q - p;
        q /= 2;
        r = p;
      }
    }
  }
};
template <int OFF, int N, int E, int... K>
__device__ __forceinline__ void merge_exchange(uint32_t (&v)[E], std::integer_sequence<int, K...>) {
  constexpr MergeExchange<N> list;
  (order_pair<OFF + list.a[K], OFF + list.b[K]>(v), ...);
}

// Orders words OFF .. OFF + N - 1 of a thread: in any order, or (BITONIC) a bitonic sequence, which takes fewer
// comparators while its length is even.
template <bool BITONIC, int OFF, int N, int E, int I = 0>
__device__ __forceinline__ void order_words(uint32_t (&v)[E]) {
  if constexpr (N > 1 && BITONIC && N % 2 == 0) {
    if constexpr (I < N / 2) {
      order_pair<OFF + I, OFF + I + N / 2>(v);
      order_words<true, OFF, N, E, I + 1>(v);
    } else {
      order_words<true, OFF, N / 2>(v);
      order_words<true, OFF + N / 2, N / 2>(v);
    }
  } else if constexpr (N > 1) {
    merge_exchange<OFF, N>(v, std::make_integer_sequence<int, MergeExchange<N>().count>());
  }
}

// One comparison step of the network below: a thread's words meet those of thread tid ^ LM, LM being one bit (a stride)
// or, in the MIRROR step that opens a phase, all bits below a power of two; they meet in reverse there.
template <int NT, int E, int LM, bool MIRROR>
__device__ __forceinline__ void bitonic_step(uint32_t (&v)[E], uint32_t* buf) {
  constexpr int TOP = MIRROR ? (LM + 1) / 2 : LM;  // the bit that tells the pair apart
  const int tid = threadIdx.x;
  const uint32_t bound = (tid & TOP) ? ~0u : 0u;
  uint32_t o[E];
  if constexpr (LM < kWave) {
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = lane_xor_u32<LM>(v[MIRROR ? E - 1 - e : e]);
  } else {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) buf[e * NT + tid] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = buf[(MIRROR ? E - 1 - e : e) * NT + (tid ^ LM)];
  }
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = med3_u32(v[e], o[e], bound);
}
template <int NT, int E, int LM>
__device__ __forceinline__ void bitonic_strides(uint32_t (&v)[E], uint32_t* buf) {
  if constexpr (LM >= 1) {
    bitonic_step<NT, E, LM, false>(v, buf);
    bitonic_strides<NT, E, LM / 2>(v, buf);
  }
}
template <int NT, int E, int T>
__device__ __forceinline__ void bitonic_phases(uint32_t (&v)[E], uint32_t* buf) {
  if constexpr (T <= NT) {
    bitonic_step<NT, E, T - 1, true>(v, buf);
    bitonic_strides<NT, E, T / 4>(v, buf);
    order_words<true, 0, E>(v);
    bitonic_phases<NT, E, T * 2>(v, buf);
  }
}

// Ascending sort of the NT * E 32-bit words of the workgroup (NT a power of two, E up to 16): a bitonic network in
// registers whose steps between threads cost a lane movement and one v_med3 per word; only the few steps between
// waves go through LDS. (A merge sort of 64-bit keys in LDS took three times as long, a bitonic
// network on 64-bit keys five times: compare-and-select of two registers.) Halving works for a bitonic sequence
// of any even length, so E need be no power of two: an even E costs as much per word as the next power of two, an odd
// one a little more (instructions per word, NT = 256: E = 4 97, 5 108, 6 104, 7 117, 8 104).
// In two steps: the network, after which thread t holds words t * E .. t * E + E - 1, and the store, after which
// buf[0 .. NT * E) holds the words in order, visible to all threads.
template <int NT, int E>
__device__ __forceinline__ void block_sort_regs(uint32_t (&v)[E], uint32_t* buf) {
  order_words<false, 0, E>(v);
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
