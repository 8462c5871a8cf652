// Ordering a few thousand (row, column) records in one workgroup, and the store of their columns and pos: what the
// sample sort and the sort by reserved regions share.
#pragma once
#include "blocksort.hpp"
#include "common.hpp"
#include "rows.hpp"

namespace spt {

constexpr int kLiBits = 12;         // bits of a record's number inside its bucket; the rest of a word: its key, coarsely
constexpr int kMaxSamples = 4096;   // of the sample sort's; numbered by kLiBits bits, too

// Bits of a record's number among n.
constexpr int number_bits(int n) { return n <= 1024 ? 10 : 1 + number_bits((n + 1) / 2); }

// p[i] at an offset of 32 bits (fewer instructions than a 64-bit address): for fewer than 2^29 elements.
template <typename E>
__device__ __forceinline__ const E& at32(const E* p, int i) {
  return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(p) + static_cast<uint32_t>(i) * static_cast<uint32_t>(sizeof(E)));
}
template <typename E>
__device__ __forceinline__ E& at32(E* p, int i) {
  return *reinterpret_cast<E*>(reinterpret_cast<char*>(p) + static_cast<uint32_t>(i) * static_cast<uint32_t>(sizeof(E)));
}

// Position of sample t of S out of m records: one in every m / S, at a place of the stretch that
// differs from stretch to stretch.
template <int S, uint32_t MIX = 2654435769u>
__device__ __forceinline__ int sample_pos(int t, int m) {
  const uint32_t jitter = (static_cast<uint32_t>(t) * MIX) >> 16;
  return static_cast<int>((((static_cast<uint64_t>(t) << 16) | jitter) * static_cast<uint64_t>(m) / S) >> 16);
}

// ---- sorting a few thousand records in one workgroup ------------------------------------------
// After the network: do kCrowd neighbours share their coarse bits? (Of a thread's own words, or of lanes of one
// row of 16: a stretch of twice that many is seen wherever it lies.)
constexpr int kCrowd = 16;
template <int NT, int LI, int E>
__device__ __forceinline__ bool crowded(const uint32_t (&v)[E], int n) {
  const int tid = threadIdx.x;
  if constexpr (E >= kCrowd) {
    bool c = false;
#pragma unroll
    for (int e = 0; e < E; e += kCrowd)
      c = c || (tid * E + e + kCrowd <= n && v[e] >> LI == v[e + kCrowd - 1] >> LI);
    return c;
  } else {
    constexpr int D = (kCrowd + E - 1) / E - 1;  // lanes further on
    const uint32_t last = dpp_u32<0x100 | D>(v[E - 1]);  // row_shl:D
    return (tid & 15) + D < 16 && (tid + D + 1) * E <= n && v[0] >> LI == last >> LI;
  }
}

// Orders n records (numbered as in the input) by key. rel_at gives a record's key less a lower bound of all, below 2^(32 - LI + shift).
// A record travels through the sort as one 32-bit word: the upper 32 - LI bits of that and LI bits of its number in input
// order. Where that many bits do not tell two neighbours apart, a record counts the keys of its stretch that come before
// it. Stretches are two or three records long where columns are
// anywhere, but as long as a row where they are neighbours in a wide matrix: once one of them has kCrowd
// records, all are sorted again, by 32 - LI bits at a time from the lowest on. (30M records, counted / sorted
// again: rows of 20 neighbours in 2M columns 1374 / 1098 us, of 30 1603 / 1099, of 1000 in 2^31 columns
// 16 900 / 1151. From eight records on, rows of 10 neighbours would gain 4 %, but power-law rows, whose long ones
// crowd a few buckets, lose up to 2 %: 6M records 271 us counted, 272 and 276 sorted again from 16 and from 8 on.
// Looking for such stretches costs 0.5 of 21 us for 50 000 records.)
// Bound by vector instructions (half of them in the finishing kernel are the network).
// Left out after measuring: dealing the words to 1024 equal bins of the key range and ranking
// inside the bins (631 instead of 503 us for 60M records with power-law rows: long and short rows
// in one bucket crowd the bins).
// words: NT * E words of LDS; ord: n half-words, the records in order.
template <int NT, int E, int LI = kLiBits, class KA>
__device__ __forceinline__ void sort_records(uint32_t* words, uint16_t* ord, int n, int shift, const KA& rel_at) {
  __shared__ int s_crowded;
  static_assert(NT * E <= 1 << LI, "a record's number takes LI bits");
  constexpr uint32_t kLi = (1 << LI) - 1;
  constexpr int kKeyBits = 32 - LI;
  const int tid = threadIdx.x;
  uint32_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int li = e * NT + tid;
    v[e] = ~0u;
    if (li < n) v[e] = (static_cast<uint32_t>(rel_at(li) >> shift) << LI) | li;
  }
  if (tid == 0) s_crowded = 0;
  block_sort_regs<NT, E>(v, words);
  if (shift > 0 && crowded<NT, LI>(v, n)) s_crowded = 1;
  block_sort_store<NT, E>(v, words);
  if (s_crowded) {  // uniform
    for (int low = 0; low < shift + kKeyBits; low += kKeyBits) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e * NT + tid;
        v[e] = ~0u;
        if (i < n) v[e] = static_cast<uint32_t>(rel_at(low ? ord[i] : i) >> low) << LI | i;
      }
      block_sort_regs<NT, E>(v, words);
      block_sort_store<NT, E>(v, words);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e * NT + tid;
        if (i < n) v[e] = low ? ord[words[i] & kLi] : words[i] & kLi;
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e * NT + tid;
        if (i < n) ord[i] = static_cast<uint16_t>(v[e]);
      }
      __syncthreads();
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * NT + tid;
    if (i < n) {
      const uint32_t w = words[i], q = w >> LI;
      const int li = w & kLi;
      int at = i;
      if (shift > 0 && ((i > 0 && words[i - 1] >> LI == q) || (i + 1 < n && words[i + 1] >> LI == q))) {
        const auto key = rel_at(li);
        int g = i;
        while (g > 0 && words[g - 1] >> LI == q) --g;
        at = g;
        for (; g < n && words[g] >> LI == q; ++g) {
          const int other = words[g] & kLi;
          const auto k = rel_at(other);
          at += (k < key || (k == key && other < li)) ? 1 : 0;
        }
      }
      ord[at] = static_cast<uint16_t>(li);
    }
  }
  __syncthreads();
}

// The number of low key bits that 32 - LI bits cannot hold between two bounds.
template <int LI = kLiBits>
__device__ __forceinline__ int coarse_shift(uint64_t lo, uint64_t hi) {
  const int bits = 64 - __clzll(static_cast<long long>((hi - lo) | 1));
  return max(0, bits - (32 - LI));
}

// Key and value side by side, as the last partition leaves them: KT = uint64_t, the key K; or uint32_t, K - base, where
// 32 bits hold that for every bucket of a segment (a third of the record and the wide arithmetic of the last sort less).
template <typename KT, typename VT>
struct Record {
  static constexpr int kWords = (sizeof(KT) + sizeof(VT)) / 4;
  uint32_t w[kWords];
  __device__ __forceinline__ static Record of(KT k, VT v) {
    Record r;
    __builtin_memcpy(r.w, &k, sizeof(KT));
    __builtin_memcpy(r.w + sizeof(KT) / 4, &v, sizeof(VT));
    return r;
  }
  __device__ __forceinline__ KT key() const {
    KT k;
    __builtin_memcpy(&k, w, sizeof(KT));
    return k;
  }
  __device__ __forceinline__ VT val() const {
    VT v;
    __builtin_memcpy(&v, w + sizeof(KT) / 4, sizeof(VT));
    return v;
  }
};
// A bucket's records before the last sort, from its first one on: `rel` is what the sort compares, K - base of the record
// or its row alone.
template <typename KT_, typename VT_>
struct RecordBucket {
  typedef VT_ VT;
  typedef KT_ KT;
  const Record<KT, VT>* __restrict__ r;
  uint64_t base;  // of the order's keys
  int kshift;
  __device__ __forceinline__ void load(int p, KT& key, VT& val) const {
    const Record<KT, VT> x = at32(r, p);
    key = x.key();
    val = x.val();
  }
  __device__ __forceinline__ KT key(int p) const { return at32(r, p).key(); }
  __device__ __forceinline__ VT val(int p) const { return at32(r, p).val(); }
  __device__ __forceinline__ KT rel(KT key) const {
    return sizeof(KT) == 4 ? key >> kshift : static_cast<KT>((key >> kshift) - base);
  }
  __device__ __forceinline__ uint64_t whole(KT key) const { return sizeof(KT) == 4 ? (base << kshift) + key : key; }
};

// Columns and pos of the bucket's entries in order; the record's value is left to the caller.
template <int NT, int E, class F, class KA, class PUT>
__device__ __forceinline__ void store_entries(const uint16_t* ord, int n, int first, int lo_row, int hi_row,
                                              const F& f, const KA& key_at, int32_t* __restrict__ pos,
                                              int32_t* __restrict__ crd_out, const PUT& put) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = e * NT + tid;
    const bool live = j < n;
    if (!__any(live)) break;
    int row = 0, prev = 0;
    if (live) {
      const int li = ord[j];
      const uint64_t K = key_at(li);
      row = f.row_in(K);
      crd_out[first + j] = f.col_of(K);
      put(j, li);
    }
    prev = __shfl_up(row, 1);
    if (lane_id() == 0 && live) prev = j > 0 ? f.row_in(key_at(ord[j - 1])) : lo_row;
    store_pos_range(pos, live ? prev : 0, row, first + j);
    const bool last = j == n - 1;
    if (__any(last)) store_pos_range(pos, last ? row : 0, last ? hi_row : 0, first + n);
  }
}

// Up to NT * E records, whose keys and values pass through LDS.
template <int NT, int E, int LI = kLiBits, class SRC, class F>
__device__ __forceinline__ void finish_staged(char* mem, const SRC& src, int n, int first, int shift, int lo_row, int hi_row,
                                              const F& f, int32_t* __restrict__ pos, int32_t* __restrict__ crd_out,
                                              typename SRC::VT* __restrict__ val_out) {
  typedef typename SRC::VT VT;
  typedef typename SRC::KT KT;
  KT* s_key = reinterpret_cast<KT*>(mem);
  VT* s_val = reinterpret_cast<VT*>(mem);
  uint32_t* words = reinterpret_cast<uint32_t*>(s_key + NT * E);
  uint16_t* ord = reinterpret_cast<uint16_t*>(words + NT * E);
  static_assert(sizeof(VT) <= sizeof(KT) + 4, "");
  const int tid = threadIdx.x;
  KT k[E];
  VT v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) src.load(min(e * NT + tid, n - 1), k[e], v[e]);
#pragma unroll
  for (int e = 0; e < E; ++e) s_key[e * NT + tid] = k[e];
  __syncthreads();
  sort_records<NT, E, LI>(words, ord, n, shift, [&](int li) { return src.rel(s_key[li]); });
  store_entries<NT, E>(ord, n, first, lo_row, hi_row, f, [&](int li) { return src.whole(s_key[li]); }, pos, crd_out,
                         [](int, int) {});
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) s_val[e * NT + tid] = v[e];
  __syncthreads();
  val_out += first;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = e * NT + tid;
    if (j < n) at32(val_out, j) = s_val[ord[j]];
  }
}

// Up to NT * E records, whose keys and values are fetched where they are used.
template <int NT, int E, int LI = kLiBits, class SRC, class F>
__device__ __forceinline__ void finish_direct(char* mem, const SRC& src, int n, int first, int shift, int lo_row, int hi_row,
                                              const F& f, int32_t* __restrict__ pos, int32_t* __restrict__ crd_out,
                                              typename SRC::VT* __restrict__ val_out) {
  uint32_t* words = reinterpret_cast<uint32_t*>(mem);
  uint16_t* ord = reinterpret_cast<uint16_t*>(words + E * NT);
  sort_records<NT, E, LI>(words, ord, n, shift, [&](int li) { return src.rel(src.key(li)); });
  store_entries<NT, E>(ord, n, first, lo_row, hi_row, f, [&](int li) { return src.whole(src.key(li)); }, pos, crd_out,
                         [&](int j, int li) { val_out[first + j] = src.val(li); });
}

}  // namespace spt
