// COO -> CSR of a middling number of records in one partition, gfx950.
//
// The sample sort (sample_sort.hip) partitions stably: count, scan, scatter, five launches for one level and nine or ten for
// two, and conversions of less than three million records spend most of their time between dependent loads and launches. Here
// a record carries its position among the bits of its key, (row, column, position) or (row, position, column): no two
// keys are alike, so records may move in any order. One launch places them: a workgroup counts its tile's records of
// each bucket in LDS, takes as much of each bucket's region with an atomic add, and stores them there. One workgroup per
// bucket then sorts it in LDS. What its workgroup does not hold is picked out of its region, a part of the key range at
// a time; what a bucket's region does not hold is picked out of the input by all workgroups, a part each. The result is that of a stable sort whatever order the adds come in.
// Keys of more than 64 bits and workspaces of less than the query are for the sample sort.
//
// Measured (fp64, 107 000 records, 34.1 us before: samples' ranks 5, partition 7, finish 7 us; 500 000 63 -> 33;
// 1M 73 -> 46, of which the finish takes 25; 2.2M 115 -> 90; 50 000 19.8 -> 15.3). Up to 100 000 records the launches and the chain of loads in
// each bound it, beyond the network of the finish (vector instructions and barriers) and the adds (counters
// each in a line of their own: within 2 %).
#include <algorithm>

#include "common.hpp"
#include "radix.hpp"
#include "sortrecords.hpp"
#include "wavescan.hpp"

namespace spt {

// K = row, column and position side by side (by row alone: row, position, column).
struct UniqueForm {
  int row_shift, col_shift, pos_shift;
  uint32_t col_mask, pos_mask;
  __device__ __forceinline__ uint64_t key(int row, int col, int p) const {
    return static_cast<uint64_t>(static_cast<uint32_t>(row)) << row_shift | static_cast<uint64_t>(static_cast<uint32_t>(col)) << col_shift |
           static_cast<uint64_t>(static_cast<uint32_t>(p)) << pos_shift;
  }
  __device__ __forceinline__ int row_in(uint64_t K) const { return static_cast<int>(K >> row_shift); }
  __device__ __forceinline__ int col_of(uint64_t K) const { return static_cast<int>(static_cast<uint32_t>(K >> col_shift) & col_mask); }
  __device__ __forceinline__ int pos_of(uint64_t K) const { return static_cast<int>(static_cast<uint32_t>(K >> pos_shift) & pos_mask); }
};
struct UniqueSource {
  const int32_t* __restrict__ row;
  const int32_t* __restrict__ col;
  UniqueForm f;
  __device__ __forceinline__ uint64_t key(int p) const { return f.key(row[p], col[p], p); }
};

// ---- splitters ------------------------------------------------------------------------------
// Every (S / nb)th of S samples in order; the first bucket has none. The counts are cleared beside.
template <int S>
__device__ __forceinline__ void store_splitter(int rank, uint64_t key, int nb, uint64_t* __restrict__ skey) {
  const int step = S / nb;
  if (rank % step == 0) skey[rank / step] = rank ? key : ~uint64_t{0};
}
template <int S>
__global__ __launch_bounds__(kWave) void reserve_pick_kernel(const UniqueSource src, int n, uint64_t* __restrict__ picked) {
  const int t = blockIdx.x * kWave + threadIdx.x;
  picked[t] = src.key(sample_pos<S>(t, n));
}
// S up to 4096: a workgroup counts how many samples come before each of 16 of them. Each has all samples; from 4096 on they are
// put side by side first, which saves every compute unit the lines of rows and columns that hold them.
constexpr int kRankThreads = 512, kRankLanes = 32;
template <int S>
__global__ __launch_bounds__(kRankThreads) void reserve_rank_kernel(const UniqueSource src, int n, int nb,
                                                                    const uint64_t* __restrict__ picked, uint64_t* __restrict__ skey,
                                                                    int32_t* __restrict__ count) {
  constexpr int kOwn = S / kRankThreads;
  __shared__ uint64_t s_key[S];
  const int tid = threadIdx.x;
  uint64_t own[kOwn];
#pragma unroll
  for (int e = 0; e < kOwn; ++e) {
    const int t = e * kRankThreads + tid;
    own[e] = S >= 4096 ? picked[t] : src.key(sample_pos<S>(t, n));
  }
#pragma unroll
  for (int e = 0; e < kOwn; ++e) s_key[e * kRankThreads + tid] = own[e];
  if (blockIdx.x == 0 && tid < nb) count[tid] = 0;
  __syncthreads();
  const int t = (blockIdx.x * kRankThreads + tid) / kRankLanes;
  const uint64_t key = s_key[t];
  int rank = 0;
#pragma unroll 8
  for (int q = tid % kRankLanes; q < S; q += kRankLanes) rank += s_key[q] < key + (q < t ? 1 : 0) ? 1 : 0;  // (the same position may be drawn twice)
#pragma unroll
  for (int d = 1; d < kRankLanes; d <<= 1) rank += __shfl_xor(rank, d);
  if (tid % kRankLanes == 0) store_splitter<S>(rank, key, nb, skey);
}
// S = 16384 (the square of which would take 40 us): lists of 1024 in order, then each sample is looked up in the others.
constexpr int kList = 1024, kListThreads = 256;
template <int S>
__global__ __launch_bounds__(kListThreads) void reserve_lists_kernel(const UniqueSource src, int n, int bits, uint64_t* __restrict__ list) {
  constexpr int E = kList / kListThreads, L = S / kList;
  __shared__ uint64_t s_key[kList];
  __shared__ __attribute__((aligned(16))) uint32_t words[kList];
  __shared__ uint16_t ord[kList];
  const int tid = threadIdx.x;
  uint64_t own[E];
#pragma unroll
  for (int e = 0; e < E; ++e) own[e] = src.key(sample_pos<S>((e * kListThreads + tid) * L + blockIdx.x, n));
#pragma unroll
  for (int e = 0; e < E; ++e) s_key[e * kListThreads + tid] = own[e];
  __syncthreads();
  sort_records<kListThreads, E>(words, ord, kList, max(0, bits - (32 - kLiBits)), [&](int li) { return s_key[li]; });
#pragma unroll
  for (int e = 0; e < E; ++e) list[blockIdx.x * kList + e * kListThreads + tid] = s_key[ord[e * kListThreads + tid]];
}
// (Four lanes to a sample, each with a quarter of the lists, and three keys of a list at a time: five loads in a row. Bisections by one
// lane, eleven: 16384 samples 8.4 and 11.3 us.)
constexpr int kMergeLanes = 4;
template <int S>
__global__ __launch_bounds__(kListThreads) void reserve_merge_kernel(const uint64_t* __restrict__ list, int nb,
                                                                     uint64_t* __restrict__ skey, int32_t* __restrict__ count) {
  constexpr int L = S / kList, kOwn = L / kMergeLanes;
  static_assert(kList == 1024 && L % kMergeLanes == 0, "");
  const int at = blockIdx.x * kListThreads + threadIdx.x, t = at / kMergeLanes, part = at % kMergeLanes;
  if (at < nb) count[at] = 0;
  const int own = t / kList;
  const uint64_t key = list[t];
  int lo[kOwn];
#pragma unroll
  for (int i = 0; i < kOwn; ++i) lo[i] = 0;
#pragma unroll
  for (int step = kList / 4; step > 0; step >>= 2) {
    uint64_t q[kOwn][3];
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
#pragma unroll
      for (int r = 0; r < 3; ++r) q[i][r] = list[(i * kMergeLanes + part) * kList + lo[i] + (r + 1) * step - 1];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const uint64_t k = key + (i * kMergeLanes + part < own ? 1 : 0);
      lo[i] += ((q[i][0] < k ? 1 : 0) + (q[i][1] < k ? 1 : 0) + (q[i][2] < k ? 1 : 0)) * step;
    }
  }
  int rank = part == 0 ? t % kList : 0;
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const int l = i * kMergeLanes + part;
    if (l != own) rank += lo[i] + (list[l * kList + lo[i]] < key + (l < own ? 1 : 0) ? 1 : 0);
  }
#pragma unroll
  for (int d = 1; d < kMergeLanes; d <<= 1) rank += __shfl_xor(rank, d);
  if (part == 0) store_splitter<S>(rank, key, nb, skey);
}

// ---- partition ------------------------------------------------------------------------------
// Four records to a thread. The bucket is found as in the sample sort's classification: a bisection on the first 31 bits of the
// key, by the whole keys where those are a splitter's.
template <typename VT, int NB, int NT>
__global__ __launch_bounds__(NT) void reserve_partition_kernel(const UniqueSource src, const VT* __restrict__ val_in, int n,
                                                               int coarse_bits, int room, const uint64_t* __restrict__ skey,
                                                               int32_t* __restrict__ count, Record<uint64_t, VT>* __restrict__ out) {
  constexpr int IPT = 4, kLevels = NB == 128 ? 7 : NB == 256 ? 8 : NB == 512 ? 9 : 10;
  __shared__ uint64_t s_key[NB];
  __shared__ uint32_t s_coarse[NB], s_tree[NB];
  __shared__ int s_cnt[NB];
  const int tid = threadIdx.x;
  const int begin = blockIdx.x * (NT * IPT);
  int row[IPT], col[IPT];
  VT val[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int p = min(begin + k * NT + tid, n - 1);
    row[k] = __builtin_nontemporal_load(src.row + p);
    col[k] = __builtin_nontemporal_load(src.col + p);
    val[k] = __builtin_nontemporal_load(val_in + p);
  }
  const auto coarse = [&](uint64_t k) { return static_cast<uint32_t>(k >> coarse_bits); };
  for (int b = tid; b < NB; b += NT) {
    const int level = 31 - __clz(b | 1);
    const uint64_t own = skey[b], node = skey[b == 0 ? 1 : ((b - (1 << level)) * 2 + 1) << (kLevels - 1 - level)];
    s_key[b] = own;
    s_coarse[b] = b == 0 ? ~0u : coarse(own);  // (~0: no record's)
    s_tree[b] = coarse(node);
    s_cnt[b] = 0;
  }
  __syncthreads();
  uint64_t key[IPT];
  int at[IPT];  // bucket << 16 | number among the tile's of it
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int p = begin + k * NT + tid;
    const bool live = p < n;
    const uint64_t K = src.f.key(row[k], col[k], min(p, n - 1));
    const uint32_t c = static_cast<uint32_t>(K >> coarse_bits);
    uint32_t node = 4;
#pragma unroll
    for (int level = 0; level < kLevels; ++level)
      node = 2 * node + (*reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(s_tree) + node) <= c ? 4 : 0);
    int d = static_cast<int>(node / 4) - NB;
    if (__any(s_coarse[d] == c)) {
      d = 0;
#pragma unroll
      for (int step = NB / 2; step > 0; step >>= 1) d += s_key[d + step] <= K ? step : 0;
    }
    key[k] = K;
    int r = 0;
    // ordered input: a wave's records share a bucket, and adds to one counter are serialised
    const int d0 = __builtin_amdgcn_readfirstlane(d);
    if (__all(live && d == d0)) {
      if (lane_id() == 0) r = atomicAdd(&s_cnt[d], kWave);
      r = __builtin_amdgcn_readfirstlane(r) + lane_id();
    } else if (live) {
      r = atomicAdd(&s_cnt[d], 1);
    }
    at[k] = d << 16 | r;
  }
  __syncthreads();
  for (int b = tid; b < NB; b += NT) {
    const int c = s_cnt[b];
    if (c) s_cnt[b] = atomicAdd(&count[b], c);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int d = at[k] >> 16, slot = s_cnt[d] + (at[k] & 0xFFFF);
    if (begin + k * NT + tid < n && slot < room) out[d * room + slot] = Record<uint64_t, VT>::of(key[k], val[k]);
  }
}

// ---- finish ---------------------------------------------------------------------------------
constexpr int kStagedWords = 5, kMostWords = 9;  // words of a thread: whose records pass through LDS, and at most
// Where records are picked from: a region of n records, or the whole input.
template <typename VT>
struct PickSource {
  const Record<uint64_t, VT>* __restrict__ region;  // null: the input
  UniqueSource input;
  int n;
};
// f(key) for all keys of a source, by a workgroup. Of the input, a thread has eight rows and columns in flight.
template <int NT, typename VT, class F>
__device__ __forceinline__ void each_key(const PickSource<VT>& s, const F& f) {
  if (s.region) {
    for (int p = threadIdx.x; p < s.n; p += NT) f(at32(s.region, p).key());
    return;
  }
  typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int U = 2;
  for (int p0 = 4 * threadIdx.x; p0 < s.n; p0 += 4 * U * NT) {
    I4 row[U], col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int from = min(p0 + 4 * u * NT, s.n - 4);
      row[u] = *reinterpret_cast<const I4*>(s.input.row + from);
      col[u] = *reinterpret_cast<const I4*>(s.input.col + from);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + 4 * u * NT, from = min(p, s.n - 4);  // (the last four once)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (from + q >= p) f(s.input.f.key(row[u][q], col[u][q], from + q));
    }
  }
}

// What all threads of a workgroup have, added up.
__device__ __forceinline__ int block_total(int x) {
  __shared__ int s_total;
  if (threadIdx.x == 0) s_total = 0;
  __syncthreads();
  const int sum = wave_inclusive_sum(x);
  if (lane_id() == kWave - 1 && sum) atomicAdd(&s_total, sum);
  __syncthreads();
  const int total = s_total;
  __syncthreads();
  return total;
}

// The (rank + 1)th smallest of n keys of LDS, all of them in [lo, last].
template <int NT>
__device__ __forceinline__ uint64_t ranked_key(const uint64_t* keys, int n, int rank, uint64_t lo, uint64_t last) {
  while (lo < last) {
    const uint64_t mid = lo + (last - lo) / 2;
    int upto = 0;
    for (int i = threadIdx.x; i < n; i += NT) upto += keys[i] <= mid ? 1 : 0;
    if (block_total(upto) > rank) last = mid;
    else lo = mid + 1;
  }
  return lo;
}

// [from, to] has more than `most` records: it becomes a range of at most that many and of one at least, before which [from, to] has none.
// Each look counts them in NT parts of the range, so that a range of one part is 2^9 times narrower: eight looks at most, as keys differ.
template <int NT, typename VT>
__device__ __forceinline__ void narrow(uint32_t* hist, const PickSource<VT>& source, int most, uint64_t* from_at, uint64_t* to_at) {
  __shared__ int s_wave[NT / kWave], s_part, s_before;
  const int tid = threadIdx.x;
  uint64_t from = *from_at, to = *to_at;
  for (;;) {
    const int shift = max(0, 64 - __clzll(static_cast<long long>((to - from) | 1)) - (31 - __clz(NT)));
    hist[tid] = 0;
    __syncthreads();
    each_key<NT>(source, [&](uint64_t key) {
      if (key >= from && key <= to) atomicAdd(&hist[(key - from) >> shift], 1u);
    });
    __syncthreads();
    const int own = static_cast<int>(hist[tid]), sum = wave_inclusive_sum(own);
    if (lane_id() == kWave - 1) s_wave[wave_id()] = sum;
    __syncthreads();
    int before = sum - own;
    for (int w = 0; w < wave_id(); ++w) before += s_wave[w];
    if (before <= most && before + own > most) {  // one thread's
      s_part = tid;
      s_before = before;
    }
    __syncthreads();
    const uint64_t start = from + (static_cast<uint64_t>(s_part) << shift);
    const bool some = s_before > 0;
    __syncthreads();
    if (some) {
      to = start - 1;
    } else {
      const uint64_t width = (uint64_t{1} << shift) - 1;
      from = start;
      to = to - start < width ? to : start + width;
    }
    if (some || shift == 0) break;
  }
  *from_at = from;
  *to_at = to;
}

template <int NT>
constexpr int kPickKeys = 8 * NT;  // of LDS, at most
// n keys of LDS in order, padded to a power of two: a bitonic sort that takes few registers, for what is rarely sorted.
template <int NT>
__device__ __forceinline__ void sort_keys(uint64_t* key, int n) {
  int size = 2 * NT;
  while (size < n) size *= 2;
  for (int i = n + threadIdx.x; i < size; i += NT) key[i] = ~uint64_t{0};
  __syncthreads();
  for (int k = 2; k <= size; k *= 2)
    for (int d = k / 2; d > 0; d /= 2) {
#pragma unroll 1
      for (int t = threadIdx.x; t < size / 2; t += NT) {
        const int i = 2 * t - (t & (d - 1)), j = i + d;
        const uint64_t a = key[i], b = key[j];
        if ((a > b) == ((i & k) == 0)) {
          key[i] = b;
          key[j] = a;
        }
      }
      __syncthreads();
    }
}

// The records of a source with keys in [lo, last], stored in order from entry `first` on, which counts from key `below` on: as many at a time as LDS
// holds keys of. A key tells the position and so the value.
template <int NT, typename VT>
__device__ __forceinline__ void pick_and_store(uint64_t* mem, const PickSource<VT>& source, const VT* __restrict__ val_in, int first,
                                               uint64_t below, uint64_t lo, uint64_t last, int lo_row, int hi_row, int32_t* __restrict__ pos,
                                               int32_t* __restrict__ crd_out, VT* __restrict__ val_out) {
  constexpr int kMost = kPickKeys<NT>;
  const UniqueForm& f = source.input.f;
  __shared__ int s_found;
  const int tid = threadIdx.x;
  uint64_t from = lo, to = last;
  int a_row = lo_row, left = -1;  // left: how many lie in [from, last], once that is known
  for (;;) {
    if (tid == 0) s_found = 0;
    __syncthreads();
    int before = 0;
    each_key<NT>(source, [&](uint64_t key) {
      if (key >= from && key <= to) {
        const int i = atomicAdd(&s_found, 1);
        if (i < kMost) mem[i] = key;
      }
      before += key >= below && key < lo ? 1 : 0;
    });
    __syncthreads();
    int cnt = s_found;
    if (left < 0) {
      left = cnt;
      first += block_total(before);
      below = lo;
    }
    __syncthreads();
    if (cnt > kMost && from < to) {
      narrow<NT>(reinterpret_cast<uint32_t*>(mem), source, kMost, &from, &to);
      continue;
    }
    cnt = min(cnt, kMost);
    sort_keys<NT>(mem, cnt);
    const int b_row = to == last ? hi_row : f.row_in(to + 1);
    for (int j0 = 0; j0 == 0 || j0 < cnt; j0 += NT) {
      const int j = j0 + tid;
      int row = 0, prev = 0;
      if (j < cnt) {
        const uint64_t K = mem[j];
        row = f.row_in(K);
        prev = j > 0 ? f.row_in(mem[j - 1]) : a_row;
        crd_out[first + j] = f.col_of(K);
        val_out[first + j] = val_in[f.pos_of(K)];
      }
      store_pos_range(pos, prev, row, first + j);
      const bool end = j == max(cnt - 1, 0);
      store_pos_range(pos, end ? (cnt ? row : a_row) : 0, end ? b_row : 0, first + cnt);
    }
    if (to == last) break;
    first += cnt;
    left -= cnt;
    a_row = b_row;
    from = to + 1;
    to = last;
    __syncthreads();
    if (left > kMost) narrow<NT>(reinterpret_cast<uint32_t*>(mem), source, kMost, &from, &to);
  }
  __syncthreads();
}

// What the last sort does not hold: the workgroup's own bucket, if it is in its region, m records; and its share of the buckets whose regions
// are full. Of these, a part of the key range, cut at samples of a second draw (the first had few of it or none), is picked out of the
// input. So an order that the first draw misses costs a scan of the input for a part, a part or two to a workgroup; one that both
// miss, one for each 4096 or 8192 records by one workgroup, and as many to narrow the range. All records but the samples in one bucket, us, by its
// workgroup alone, which halved the range until 2048 or 4096 were left / so / in even order:
//   20 011 records 309 / 137 / 17; 100 003 4452 / 222 / 22; 1M 128 000 / 532 / 55; 1.5M - / 2267 / 70; 3M - / 3460 / 115
// (rows and columns fetched four at a time: 1.5M 6900 without.) A call without such buckets takes as long as before (50 000 records 15.2 / 15.2,
// 900 000 44.6 / 43.7): few registers are left for what is rare, hence the plain sort of keys.
template <int NT, typename VT>
__device__ __forceinline__ void sort_the_rest(uint64_t* mem, const Record<uint64_t, VT>* __restrict__ own_region, int m, int own_first,
                                              bool overflow, const UniqueSource& src, const VT* __restrict__ val_in, int n, int nrows, int room,
                                              const uint64_t* __restrict__ skey, const int32_t* __restrict__ count,
                                              int32_t* __restrict__ pos, int32_t* __restrict__ crd_out, VT* __restrict__ val_out) {
  constexpr int kSamples = kPickKeys<NT>, kTarget = kPickKeys<NT> / 2;  // kTarget: records of a part
  __shared__ int s_samples;
  const int nb = gridDim.x, tid = threadIdx.x;
  bool mine = m <= room && m > kMostWords * NT;
  for (int part_of_all = blockIdx.x;;) {
    int b = blockIdx.x, part = 0, parts = 1, first = own_first;
    const Record<uint64_t, VT>* region = nullptr;
    if (mine) {
      region = own_region;
    } else if (overflow) {
      part = part_of_all;
      part_of_all += nb;
      first = 0;
      for (b = 0; b < nb; ++b) {
        const int c = count[b];
        if (c > room) {
          parts = (c + kTarget - 1) / kTarget;
          if (part < parts) break;
          part -= parts;
        }
        first += c;
      }
      if (b == nb) return;
    } else {
      return;
    }
    mine = false;
    const uint64_t lo = b > 0 ? skey[b] : 0;
    const uint64_t last = (b + 1 < nb ? skey[b + 1] : static_cast<uint64_t>(nrows) << src.f.row_shift) - 1;
    uint64_t from = lo, to = last;
    if (parts > 1) {
      if (tid == 0) s_samples = 0;
      __syncthreads();
#pragma unroll 1
      for (int t = tid; t < kSamples; t += NT) {
        const uint64_t key = src.key(sample_pos<kSamples, 3266489917u>(t, n));
        if (key >= lo && key <= last) mem[atomicAdd(&s_samples, 1)] = key;
      }
      __syncthreads();
      const int samples = s_samples;
      __syncthreads();
      parts = min(parts, max(samples, 1));
      if (part >= parts) continue;  // fewer samples than parts
      // (a part begins at a sample after the first of them, and the samples' keys differ)
#pragma unroll 1
      for (int q = part; q <= part + 1; ++q) {
        if (q == 0 || q == parts) continue;
        const uint64_t cut = ranked_key<NT>(mem, samples, static_cast<int>(static_cast<int64_t>(q) * samples / parts), lo, last);
        if (q == part) from = cut;
        else to = cut - 1;
      }
    }
    pick_and_store<NT, VT>(mem, PickSource<VT>{region, src, region ? m : n}, val_in, first, lo, from,
                           to, b == 0 && part == 0 ? -1 : src.f.row_in(from), b + 1 == nb && part + 1 == parts ? nrows : src.f.row_in(to + 1),
                           pos, crd_out, val_out);
  }
}

// Bound by the network, whose steps wait for each other: as many workgroups to a compute unit as registers and LDS allow (1024 threads, eight
// waves a SIMD, keep four to fourteen registers in scratch memory). What is rare comes last: before the own bucket it kept 16 scalars in vector
// registers, and ranges of 48 000 empty rows took 10 % longer. A
// bucket's keys are compared in 32 - LI bits first, LI being no more than its records need (14 for all of them: 1M records with
// power-law rows 58 us, 49 so).
template <int NT, int WAVES, typename VT>
__global__ __launch_bounds__(NT, WAVES) void reserve_finish_kernel(const Record<uint64_t, VT>* __restrict__ in, const UniqueSource src,
                                                            const VT* __restrict__ val_in, int n, int nrows, int room,
                                                            const uint64_t* __restrict__ skey, const int32_t* __restrict__ count,
                                                            int32_t* __restrict__ pos, int32_t* __restrict__ crd_out,
                                                            VT* __restrict__ val_out) {
  __shared__ __attribute__((aligned(16))) char s_mem[NT * 14 * kStagedWords];
  static_assert(kPickKeys<NT> * 8 <= sizeof(s_mem), "");
  __shared__ int s_before, s_overflow;
  const int g = blockIdx.x, nb = gridDim.x, tid = threadIdx.x;
  if (tid == 0) s_before = s_overflow = 0;
  __syncthreads();
  for (int b0 = 0; b0 < nb; b0 += NT) {
    const int c = b0 + tid < nb ? count[b0 + tid] : 0;
    const int sum = wave_inclusive_sum(b0 + tid < g ? c : 0);
    if (lane_id() == kWave - 1 && sum) atomicAdd(&s_before, sum);
    if (c > room) s_overflow = 1;
  }
  const int m = count[g];
  const uint64_t lo = g > 0 ? skey[g] : 0;
  const uint64_t last = (g + 1 < nb ? skey[g + 1] : static_cast<uint64_t>(nrows) << src.f.row_shift) - 1;
  const int lo_row = g > 0 ? src.f.row_in(lo) : -1, hi_row = g + 1 < nb ? src.f.row_in(last + 1) : nrows;
  __syncthreads();
  const int first = s_before;
  const bool fits = m <= room && m <= kMostWords * NT;
  const RecordBucket<uint64_t, VT> bucket{in + static_cast<int64_t>(g) * room, lo, 0};
#define SPT_FINISH(HOW_, E_)                                                                                             \
  do {                                                                                                                   \
    constexpr int kWords = E_, kLi = number_bits(NT * kWords);                                                           \
    HOW_<NT, kWords, kLi>(s_mem, bucket, m, first, coarse_shift<kLi>(lo, last), lo_row, hi_row, src.f, pos, crd_out, val_out); \
  } while (0)
  if (!fits) {
  } else if (m == 0) {
    if (tid < kWave) store_pos_range(pos, tid == 0 ? lo_row : 0, tid == 0 ? hi_row : 0, first);
  } else if (m <= NT) {
    SPT_FINISH(finish_staged, 1);
  } else if (m <= 2 * NT) {
    SPT_FINISH(finish_staged, 2);
  } else if (m <= 3 * NT) {
    SPT_FINISH(finish_staged, 3);
  } else if (m <= 4 * NT) {
    SPT_FINISH(finish_staged, 4);
  } else if (m <= kStagedWords * NT) {
    SPT_FINISH(finish_staged, kStagedWords);
  } else if (m <= 6 * NT) {
    SPT_FINISH(finish_direct, 6);
  } else {
    SPT_FINISH(finish_direct, kMostWords);
  }
#undef SPT_FINISH
  if (s_overflow || !fits) {  // uniform
    __syncthreads();
    sort_the_rest<NT, VT>(reinterpret_cast<uint64_t*>(s_mem), in + static_cast<int64_t>(g) * room, m, s_before, s_overflow, src, val_in, n, nrows,
                          room, skey, count, pos, crd_out, val_out);
  }
}

// ---- host -----------------------------------------------------------------------------------
// How many buckets, samples, records to a tile and threads of a workgroup that finishes a bucket (in us, fp64 uniform, before:
// by the sample sort). More buckets are sorted faster, but take more room by atomic adds and better splitters:
//   records    before   128 / 1024   256 / 2048   512 / 4096   1024 / 16384 buckets / samples
//    12 000     12.5       13.1         14.8
//    20 000     14.7       13.9         14.8
//    64 000     20.4       15.6         17.5
//   150 000     37.3                    21.3         22.8
//   300 000     44.8                    26.5         26.7
//   600 000     66.5                                 36.0          46.3
//   1.0M        73.4                                 45.9          56.2
//   1.5M        90.2                                 69.5          71.6 (power-law rows: 108.6 and 72.6)
//   1.7M        96.0                                               73.9 (from here on with the samples' ranks as they are found now)
//   2.2M       114.8                                               90.3 (in 2048 buckets 101.6)
//   3.0M       133.1                                              119.9 (117.2)
// Threads: 512 while buckets are small (512 buckets of 500 000 records 32.8, with 1024 threads 35.1), 1024 beyond (850 000 42.1, with 512
// five samples of a hundred calls split a bucket; 1.7M in 1024 buckets 76.1). Tiles: 300 000 records in tiles of 2048 / 4096 26.5 / 26.6,
// 1M 65 / 61.
struct ReservePlan {
  int nb, samples, tile, threads, room;
};
constexpr int64_t kReserveMin = 1 << 14, kReserveMax = 3 << 20;
static ReservePlan reserve_plan(int64_t n) {
  ReservePlan P = n <= 5 << 14   ? ReservePlan{128, 1024, 1024, 512, 0}
                  : n <= 9 << 15 ? ReservePlan{256, 2048, 2048, 512, 0}
                  : n <= 5 << 17 ? ReservePlan{512, 4096, 4096, 512, 0}
                  : n <= 5 << 18 ? ReservePlan{512, 4096, 4096, 1024, 0}
                  : n <= 3 << 19 ? ReservePlan{1024, 16384, 4096, 512, 0}
                                 : ReservePlan{1024, 16384, 4096, 1024, 0};
  // In random order, a bucket of eight samples has more than five times the mean with a chance of 2e-10, one of sixteen more
  // than 3.2 times with 3e-9; what it costs, stands at sort_the_rest. (What nine words of a thread hold, 3.6 and 2.9 times the mean at least: 1e-6 and 5e-8.)
  const int64_t mean = (n + P.nb - 1) / P.nb;
  P.room = static_cast<int>(P.samples == 8 * P.nb ? 5 * mean : (16 * mean + 4) / 5);
  return P;
}
bool reserve_sort_applies(int64_t n, int64_t nrows, int64_t ncols) {
  const int low = bits_for(ncols) + bits_for(n);
  return n > kReserveMin && n <= kReserveMax && low + bits_for(nrows) <= 64;
}
size_t reserve_sort_workspace(int dtype, int64_t n) {
  const ReservePlan P = reserve_plan(n);
  const size_t record = dtype == SPT_F64 ? sizeof(Record<uint64_t, uint64_t>) : sizeof(Record<uint64_t, uint32_t>);
  return align_up(static_cast<size_t>(P.nb) * P.room * record, 256) + align_up(P.samples * 8, 256) + align_up(P.nb * 8, 256) +
         align_up(P.nb * 4, 256);
}

// The splitters, and counts of nothing.
static spt_status launch_splitters(const UniqueSource& src, int n, int bits, const ReservePlan& P, uint64_t* picked, uint64_t* skey,
                                   int32_t* count, hipStream_t s) {
#define SPT_RANK(S_)                                                                                                          \
  hipLaunchKernelGGL((reserve_rank_kernel<S_>), dim3(S_ * kRankLanes / kRankThreads), dim3(kRankThreads), 0, s, src, n, P.nb, \
                     picked, skey, count)
  if (P.samples == 1024) {
    SPT_RANK(1024);
  } else if (P.samples == 2048) {
    SPT_RANK(2048);
  } else if (P.samples == 4096) {
    hipLaunchKernelGGL(reserve_pick_kernel<4096>, dim3(4096 / kWave), dim3(kWave), 0, s, src, n, picked);
    SPT_CHECK_LAUNCH("samples");
    SPT_RANK(4096);
  } else {
    hipLaunchKernelGGL(reserve_lists_kernel<16384>, dim3(16384 / kList), dim3(kListThreads), 0, s, src, n, bits, picked);
    SPT_CHECK_LAUNCH("samples");
    hipLaunchKernelGGL(reserve_merge_kernel<16384>, dim3(16384 * kMergeLanes / kListThreads), dim3(kListThreads), 0, s, picked, P.nb, skey, count);
  }
#undef SPT_RANK
  SPT_CHECK_LAUNCH("splitters");
  return SPT_OK;
}

template <typename VT>
spt_status reserve_sort_convert(int64_t n64, int64_t nrows, int64_t ncols, bool by_col, const int32_t* row, const int32_t* col,
                                const VT* vals, int32_t* pos_out, int32_t* crd_out, VT* vals_out, void* ws, size_t ws_bytes,
                                hipStream_t s) {
  const int n = static_cast<int>(n64);
  const ReservePlan P = reserve_plan(n64);
  const int cb = bits_for(ncols), pb = bits_for(n64), bits = bits_for(nrows) + cb + pb;
  const UniqueForm f{cb + pb, by_col ? pb : 0, by_col ? 0 : cb, static_cast<uint32_t>((uint64_t{1} << cb) - 1), static_cast<uint32_t>((uint64_t{1} << pb) - 1)};
  const UniqueSource src{row, col, f};
  Workspace W(ws, ws_bytes);
  typedef Record<uint64_t, VT> R;
  R* records = W.take<R>(static_cast<size_t>(P.nb) * P.room);
  uint64_t* picked = W.take<uint64_t>(P.samples);
  uint64_t* skey = W.take<uint64_t>(P.nb);
  int32_t* count = W.take<int32_t>(P.nb);
  const spt_status st = launch_splitters(src, n, bits, P, picked, skey, count, s);
  if (st != SPT_OK) return st;
#define SPT_PART(NB_, NT_)                                                                                                \
  hipLaunchKernelGGL((reserve_partition_kernel<VT, NB_, NT_>), dim3((n + P.tile - 1) / P.tile), dim3(NT_), 0, s, src, vals, n, \
                     std::max(0, bits - 31), P.room, skey, count, records)
  if (P.nb == 128) SPT_PART(128, 256);
  else if (P.nb == 256) SPT_PART(256, 512);
  else if (P.nb == 512) SPT_PART(512, 1024);
  else SPT_PART(1024, 1024);
#undef SPT_PART
  SPT_CHECK_LAUNCH("partition");
#define SPT_FINISH(NT_, WAVES_)                                                                                              \
  hipLaunchKernelGGL((reserve_finish_kernel<NT_, WAVES_, VT>), dim3(P.nb), dim3(NT_), 0, s, records, src, vals, n,                 \
                     static_cast<int>(nrows), P.room, skey, count, pos_out, crd_out, vals_out)
  if (P.threads == 512) SPT_FINISH(512, 4);
  else SPT_FINISH(1024, 8);
#undef SPT_FINISH
  SPT_CHECK_LAUNCH("finish");
  return SPT_OK;
}

template spt_status reserve_sort_convert<uint64_t>(int64_t, int64_t, int64_t, bool, const int32_t*, const int32_t*, const uint64_t*,
                                                   int32_t*, int32_t*, uint64_t*, void*, size_t, hipStream_t);
template spt_status reserve_sort_convert<uint32_t>(int64_t, int64_t, int64_t, bool, const int32_t*, const int32_t*, const uint32_t*,
                                                   int32_t*, int32_t*, uint32_t*, void*, size_t, hipStream_t);

}  // namespace spt
