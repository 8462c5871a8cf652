// COO -> CSR by sample sort (paper Section 4.3 reordering + Section 5.4), gfx950.
//
// A radix sort of (row, column) keys moves every record once per 8 bits of key, six times for
// 22-bit rows and columns, and starts four kernels each time. Here the key range is cut at
// splitters drawn from the input itself, so that every piece holds about the same number of
// records however skewed the rows are, and pieces that fit the LDS of one workgroup are finished
// there:
//   up to kSelectMax records          one launch: workgroup j sorts a sample of the keys, picks
//                                     the records between its two splitters out of the whole
//                                     input (which stays in L2) and sorts them;
//   up to kOneLevelMax                one stable partition into up to 256 buckets, one workgroup
//                                     per bucket;
//   beyond                            two stable partitions, then one workgroup per bucket.
// A partition is count -> exclusive scan -> stable scatter, as a radix pass, with the digit found
// by bisection among the splitters instead of taken from the key bits. The count kernel notes
// each record's digit in one byte for the scatter. The second partition leaves records, key and value
// side by side, whose keys count from their bucket's lower bound: 32 bits, except in segments with a bucket
// that spans more (the segment's splitters tell; its records then keep 64).
// Equal keys: splitters are (key, position) pairs, so that even a million copies of one
// coordinate spread over the buckets, and inside a bucket records carry their number in input
// order: the result is that of a stable sort.
// pos (Table 3: running sum of the row counts) falls out of the last step: the workgroup of the
// keys between splitters of rows a and b stores pos[a+1 .. b].
// A bucket that the sample got wrong (more records than fit LDS) is split once more by its workgroup,
// at splitters of a sample of its own. In random order that happens in none of 100 calls up to 30M
// records, in 2 or 3 at 50M, some 20 at 60M and 50 at 2^26, where 256 buckets of a segment are
// not enough for the larger segments; such a call takes 2 to 3 % longer (60M records 1478 -> 1515 to 1529 us; with
// the ranks of the bucket's records counted, 10.4 ms).
//
// (From 16 385 records to 3M most calls are reserve_sort.hip's; here come those with wider keys, or less workspace than the query's.)
// Measured against the six radix passes it replaces (fp64): 60M records with power-law rows
// 3.09 -> 1.52 ms (splitters 10 + 70 us, classify 2 x 133, offsets 8 + 9, partitions 405 + 352, finish 400; with whole
// keys and separate arrays the second partition took 418); 20M 0.52 ms, 5M 0.19 ms, 250 000 48 us,
// 50 000 171 -> 19 us. The partitions write 256 interleaved streams for each array
// and are bound by how the memory system takes them: it is the bytes in flight that count. Two workgroups of 512 threads
// on a compute unit: 60M records fp64 1.70 ms in all (before splitters, offsets and records were made as now), three 1.83, three
// of 256 threads 1.87, two 1.68; 20M 0.62, 0.63, 0.64 and 0.65; fp32, 40M 1.01, 1.04, 1.03 and 1.06. Tiles of 6144 and
// 8192: up to 4 and 8 % longer for fp64, 3 % shorter for fp32 of 40M. Fewer vector instructions for the ranks do not change
// large partitions (+-1 %) and take 1 to 2 % off all below 6M records. The
// classification has vector ALU, LDS and memory busy half of the time each (four records to a lane in loads of 16 bytes,
// two or four bisections side by side: within 1 %; a table of equal cells in place of the upper steps: 14 % longer where
// long rows crowd the cells), the finishing kernel is bound by vector instructions (70 % of the time).
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "radix.hpp"
#include "scan.hpp"
#include "sortrecords.hpp"
#include "wavescan.hpp"

namespace spt {

constexpr int kFin = 256;           // threads of a workgroup that finishes a bucket of its own
constexpr int kSel = 1024;          // threads of a workgroup that selects its records first
constexpr int kCap = 4096;          // records either can sort in LDS
constexpr int kStaged = 2048;       // records whose keys and values also pass through LDS (own bucket)
constexpr int kTile = 4096;         // records per tile of a partition of many,
constexpr int kSmallTile = 1024;    // and of few records (see tile_of)
// Threads that scatter a tile (few records: more, smaller workgroups).
constexpr int part_threads(int tile) { return tile >= kTile ? 512 : 256; }
constexpr int kGroup = 4;           // consecutive tiles that one workgroup classifies
constexpr int kSelTarget = 384;     // records per workgroup: selected out of the whole (small) input,
constexpr int kDirTarget = 1408;    // of a bucket of its own
constexpr int64_t kSelectMax = 64 * 1024;                   // every workgroup reads all rows: 256 KB from L2
constexpr int64_t kOneLevelMax = int64_t(256) * kDirTarget;  // 256 buckets that fit LDS
constexpr int64_t kSampleSortMax = int64_t(1) << 26;  // 256 x 256 buckets of kDirTarget and the sample's spread
constexpr int kSegMax = 256;        // buckets of a partition

// How a record's key is put together: K = row << cb | col; what the order compares is K
// (row, then column) or the row alone (kshift = cb: rows stable).
struct KeyForm {
  int cb;      // bits of a column
  int kshift;  // 0: order by (row, col); cb: by row
  __device__ __forceinline__ int row_of(uint64_t ckey) const {
    return static_cast<int>(kshift ? ckey : ckey >> cb);
  }
  __device__ __forceinline__ int row_in(uint64_t K) const { return static_cast<int>(K >> cb); }
  __device__ __forceinline__ int col_of(uint64_t K) const { return static_cast<int>(K & ((uint64_t{1} << cb) - 1)); }
};

// The records of one level: the caller's row and column arrays, or packed keys of a partition.
struct RcSource {
  const int32_t* __restrict__ row;
  const int32_t* __restrict__ col;
  __device__ __forceinline__ uint64_t key(int p, const KeyForm& f) const {
    return (static_cast<uint64_t>(static_cast<uint32_t>(row[p])) << f.cb) | static_cast<uint32_t>(col[p]);
  }
  __device__ __forceinline__ uint64_t key_stream(int p, const KeyForm& f) const {
    return (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_nontemporal_load(row + p))) << f.cb) |
           static_cast<uint32_t>(__builtin_nontemporal_load(col + p));
  }
  __device__ __forceinline__ RcSource from(int p) const { return {row + p, col + p}; }
  __device__ __forceinline__ uint64_t key_near(int p, const KeyForm& f) const {
    return (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_nontemporal_load(&at32(row, p)))) << f.cb) |
           static_cast<uint32_t>(__builtin_nontemporal_load(&at32(col, p)));
  }
};
struct KSource {
  const uint64_t* __restrict__ k;
  __device__ __forceinline__ uint64_t key(int p, const KeyForm&) const { return k[p]; }
  __device__ __forceinline__ uint64_t key_stream(int p, const KeyForm&) const { return __builtin_nontemporal_load(k + p); }
  __device__ __forceinline__ KSource from(int p) const { return {k + p}; }
  __device__ __forceinline__ uint64_t key_near(int p, const KeyForm&) const { return __builtin_nontemporal_load(&at32(k, p)); }
};

// A bucket's records before the last sort, from its first one on: `rel` is what the sort compares, K - base of the record
// or its row alone.
template <typename VT_>
struct ArraysBucket {
  typedef VT_ VT;
  typedef uint64_t KT;
  const uint64_t* __restrict__ k;
  const VT* __restrict__ v;
  uint64_t base;  // of the order's keys
  int kshift;
  __device__ __forceinline__ void load(int p, KT& key, VT& val) const {
    key = at32(k, p);
    val = at32(v, p);
  }
  __device__ __forceinline__ KT key(int p) const { return at32(k, p); }
  __device__ __forceinline__ VT val(int p) const { return at32(v, p); }
  __device__ __forceinline__ KT rel(KT key) const { return (key >> kshift) - base; }
  __device__ __forceinline__ uint64_t whole(KT key) const { return key; }
};
// The records of the segment that begins at record `begin`, in the room of as many of the wide form.
template <typename VT, typename P>
__device__ __forceinline__ auto segment_records(P* records, int begin) {
  typedef std::conditional_t<std::is_const_v<P>, const char, char> C;
  return static_cast<C*>(records) + static_cast<int64_t>(begin) * (sizeof(uint64_t) + sizeof(VT));
}
// Do 32 bits hold K - (lo << kshift) of every record between two cuts?
__device__ __forceinline__ bool narrow_keys(uint64_t lo, uint64_t hi, const KeyForm& f) {
  return hi - lo < (uint64_t{1} << 32 >> f.kshift);
}

// A cut of the order: everything from (key, pos) on.
struct Cut {
  uint64_t key;
  int pos;
  __device__ __forceinline__ bool at_or_before(uint64_t k, int p) const {
    return key < k || (key == k && pos <= p);
  }
};

// ---- segments of the second level -----------------------------------------------------------
struct Tables {
  int32_t* seg_start;  // [nseg + 1] first record of each bucket of level 1
  int32_t* seg_tile;   // [nseg + 1] tiles before the segment
  int32_t* seg_group;  // [nseg + 1] groups of tiles before the segment
  int32_t* seg_bucket; // [nseg + 1] final buckets before the segment
  int32_t* group_seg;  // segment of each group
  int32_t* tile_seg;   // segment of each tile
  int32_t* bucket_seg; // segment of each final bucket
};

__device__ __forceinline__ int tiles_in(int m, int tile) { return (m + tile - 1) / tile; }
__device__ __forceinline__ int final_buckets(int m, int target) {
  return max(1, min(kSegMax, (m + target - 1) / target));
}

// ---- splitters ------------------------------------------------------------------------------
// Level 1: S = 1024 * E sampled keys; every (S / nb)th in order is a splitter. A workgroup counts how many of the
// samples come before each of kRankSamples of them (4096 samples: 10 us, 35 sorted by one workgroup; 1024 samples 5 and 6).
// Every workgroup has all samples, each a line of rows and one of columns that its L2 is asked for by every compute unit;
// 4096 of them are put side by side first (250 000 records 15.4 -> 9.4 us with the launch, 60M 19.3 -> 9.8; 2048 as before).
constexpr int kRankSamples = 16, kRankBlock = 512;
__global__ __launch_bounds__(kWave) void pick_samples_kernel(const RcSource src, const KeyForm f, int n, uint64_t* __restrict__ picked) {
  const int t = blockIdx.x * kWave + threadIdx.x;
  picked[t] = src.key(sample_pos<kMaxSamples>(t, n), f) >> f.kshift;
}
template <int E>
__global__ __launch_bounds__(kRankBlock) void rank_splitters_kernel(const RcSource src, const KeyForm f, int n, int nb,
                                                                const uint64_t* __restrict__ picked,
                                                                uint64_t* __restrict__ skey, int32_t* __restrict__ spos) {
  constexpr int S = 1024 * E, kLanes = kRankBlock / kRankSamples, kOwn = S / kRankBlock;
  __shared__ uint64_t s_key[S];
  const int tid = threadIdx.x;
  uint64_t own[kOwn];
#pragma unroll
  for (int e = 0; e < kOwn; ++e) {
    const int t = e * kRankBlock + tid;
    own[e] = S == kMaxSamples ? picked[t] : src.key(sample_pos<S>(t, n), f) >> f.kshift;
  }
#pragma unroll
  for (int e = 0; e < kOwn; ++e) s_key[e * kRankBlock + tid] = own[e];
  if (blockIdx.x == 0 && (tid == 0 || tid >= nb) && tid < kSegMax) {  // unused splitters lie beyond every key
    skey[tid] = ~uint64_t{0};
    spos[tid] = INT32_MAX;
  }
  __syncthreads();
  const int t = blockIdx.x * kRankSamples + tid / kLanes;
  const uint64_t key = s_key[t];
  int rank = 0;
#pragma unroll 8
  for (int q = tid % kLanes; q < S; q += kLanes) rank += s_key[q] < key + (q < t ? 1 : 0) ? 1 : 0;
#pragma unroll
  for (int d = 1; d < kLanes; d <<= 1) rank += __shfl_xor(rank, d);
  const int b = static_cast<int>((static_cast<int64_t>(rank) * nb + S - 1) / S);
  if (tid % kLanes == 0 && b > 0 && b < nb && static_cast<int>(static_cast<int64_t>(b) * S / nb) == rank) {
    skey[b] = key;
    spos[b] = sample_pos<S>(t, n);
  }
}

// Records before each bucket of level 1, in the first four waves of the workgroup. Every thread calls.
__device__ __forceinline__ int bucket_start(int count, int* s_sum) {
  const int w = wave_id(), lane = lane_id();
  const int incl = wave_inclusive_sum(count);
  if (w < 4 && lane == kWave - 1) s_sum[w] = incl;
  __syncthreads();
  int start = incl - count;
  for (int u = 0; u < (w & 3); ++u) start += s_sum[u];
  return start;
}

// Level 2: sorts S = 1024 * E sampled keys of segment blockIdx.x, a bucket of level 1 (of total1[] records each), and
// takes every (S / nb)th as a splitter; nb follows from the segment's size. The workgroup also fills in its rows of the
// segment tables, and says in place of a position of splitter 0, which there is none of, whether the segment's records are narrow.
template <int E>
__global__ __launch_bounds__(1024) void splitters_kernel(const KSource src, const KeyForm f, int nrows, int group, int tile,
                                                         const int32_t* __restrict__ total1, int nseg,
                                                         const Tables T, const uint64_t* __restrict__ skey1,
                                                         uint64_t* __restrict__ skey,
                                                         int32_t* __restrict__ spos) {
  constexpr int S = 1024 * E;
  __shared__ uint64_t s_key[S];
  __shared__ __attribute__((aligned(16))) uint32_t words[S];
  __shared__ uint16_t ord[S];
  __shared__ int s_sum[4], s_begin, s_wide;
  const int tid = threadIdx.x;
  const int seg = blockIdx.x;
  if (tid == 0) s_wide = 0;
  if (tid < 3) s_sum[tid] = 0;
  if (tid == 0) s_begin = 0;
  __syncthreads();
  const int m = total1[seg], nb = final_buckets(m, kDirTarget);
  if (tid < seg) {  // what the segments before this one take of each table
    const int before = total1[tid];
    const int nt = tiles_in(before, tile);
    atomicAdd(&s_sum[0], nt);
    atomicAdd(&s_sum[1], (nt + group - 1) / group);
    atomicAdd(&s_sum[2], final_buckets(before, kDirTarget));
    atomicAdd(&s_begin, before);
  }
  __syncthreads();
  const int begin = s_begin;
  const int nt = tiles_in(m, tile), ng = (nt + group - 1) / group;
  const int t0 = s_sum[0], g0 = s_sum[1], b0 = s_sum[2];
  if (tid == 0) {
    T.seg_start[seg] = begin;
    T.seg_tile[seg] = t0;
    T.seg_group[seg] = g0;
    T.seg_bucket[seg] = b0;
    if (seg == nseg - 1) {
      T.seg_start[nseg] = begin + m;
      T.seg_tile[nseg] = t0 + nt;
      T.seg_group[nseg] = g0 + ng;
      T.seg_bucket[nseg] = b0 + nb;
    }
  }
  for (int q = tid; q < nt; q += 1024) T.tile_seg[t0 + q] = seg;
  for (int q = tid; q < ng; q += 1024) T.group_seg[g0 + q] = seg;
  for (int q = tid; q < nb; q += 1024) T.bucket_seg[b0 + q] = seg;
  if (m == 0) return;  // uniform; one empty bucket, no splitter
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * 1024 + tid;
    s_key[t] = src.key(begin + sample_pos<S>(t, m), f) >> f.kshift;
  }
  __syncthreads();
  const uint64_t lo = seg > 0 ? skey1[seg] : 0;
  const uint64_t hi = seg + 1 < nseg ? skey1[seg + 1] : static_cast<uint64_t>(nrows) << (f.cb - f.kshift);
  sort_records<1024, E>(words, ord, S, coarse_shift(lo, hi), [&](int t) { return s_key[t] - lo; });
  if (tid < kSegMax) {
    uint64_t key = ~uint64_t{0};  // unused splitters lie beyond every key
    int pos = INT32_MAX;
    if (tid > 0 && tid < nb) {
      const int t = ord[static_cast<int>((static_cast<int64_t>(tid) * S) / nb)];
      key = s_key[t];
      pos = begin + sample_pos<S>(t, m);
    }
    skey[seg * kSegMax + tid] = key;
    spos[seg * kSegMax + tid] = pos;  // (of tid 0: written below)
    const auto bound = [&](int d) {
      return d == 0 ? lo : d >= nb ? hi : s_key[ord[static_cast<int>((static_cast<int64_t>(d) * S) / nb)]];
    };
    if (tid < nb && !narrow_keys(bound(tid), bound(tid + 1), f)) s_wide = 1;
  }
  __syncthreads();
  if (tid == 0) spos[seg * kSegMax] = !s_wide;
}

// ---- partition ------------------------------------------------------------------------------
// Splitters 1 .. 255 of a segment in LDS: whole, and as the first 31 bits of the segment's key
// range, on which the bisection runs (half the LDS traffic, 32-bit compares). A record whose
// bits equal a splitter's is placed by the whole keys. The bisection's tree is stored level by
// level (children of node i: 2i and 2i + 1): the nodes of one level lie side by side, so that the
// lanes of a wave, scattered over a level, meet few bank conflicts. Stored in key order, the
// nodes of a level share a bank: 190 us for 60M records, two thirds of it conflicts.
struct SplitterTable {
  uint64_t key[kSegMax];
  int32_t pos[kSegMax];
  uint32_t coarse[kSegMax];
  uint32_t tree[kSegMax];
};
// Bucket of a record: the number of splitters at or before it. c: its key's place in the segment's range, coarsely.
__device__ __forceinline__ int bucket_of(const SplitterTable& t, uint64_t k, int p, uint32_t c) {
  uint32_t at = 4;  // four times the node
#pragma unroll
  for (int level = 0; level < kRadixBits; ++level) at = 2 * at + (*reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(t.tree) + at) <= c ? 4 : 0);
  int d = static_cast<int>(at / 4) - kSegMax;
  if (__any(t.coarse[d] == c)) {
    d = 0;
#pragma unroll
    for (int step = kSegMax / 2; step > 0; step >>= 1) {
      const uint64_t q = t.key[d + step];
      bool le = q < k;
      if (q == k) le = t.pos[d + step] <= p;
      d += le ? step : 0;
    }
  }
  return d;
}

// hist[base + d * nt + i] = records of tile i of the segment whose bucket is d, and each record's
// bucket as one byte in dig. A workgroup takes up to `group` consecutive tiles of one segment
// and stores each bucket's counts of them side by side (digit-major for the scan).
template <class SRC, bool LEVEL2, int TILE, int NT = kBlock>
__global__ __launch_bounds__(NT) void classify_kernel(const SRC src, const KeyForm f, int n, int nrows, int group,
                                                          int nseg, const Tables T,
                                                          const uint64_t* __restrict__ skey1,
                                                          const uint64_t* __restrict__ skey,
                                                          const int32_t* __restrict__ spos,
                                                          uint8_t* __restrict__ dig, int32_t* __restrict__ hist) {
  __shared__ SplitterTable t;
  __shared__ int s_cnt[kGroup][kRadix];
  constexpr int kSide = NT / kBlock;  // tiles side by side, a workgroup's part of kBlock threads to each
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(kSide == 1 ? wave_id() : wave_id() % (kBlock / kWave));
  const int side = kSide == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave_id() / (kBlock / kWave));
  int seg = 0, begin = 0, end = n, tile0, ntiles;
  int64_t base = 0;
  // a contiguous part for each XCD of the groups there are, not of the grid's bound on them, which would leave the last
  // XCD the idle ones (1M records 74 us instead of 72, 5.7M 192 and 186)
  if (LEVEL2 && static_cast<int>(blockIdx.x) >= T.seg_group[nseg]) return;
  const int g = xcd_contiguous_block_id(blockIdx.x, LEVEL2 ? T.seg_group[nseg] : static_cast<int>(gridDim.x));
  if (LEVEL2) {
    seg = T.group_seg[g];
    begin = T.seg_start[seg];
    end = T.seg_start[seg + 1];
    ntiles = T.seg_tile[seg + 1] - T.seg_tile[seg];
    tile0 = (g - T.seg_group[seg]) * group;
    base = static_cast<int64_t>(T.seg_tile[seg]) * kRadix;
  } else {
    ntiles = tiles_in(n, TILE);
    tile0 = g * group;
  }
  if (kSide == 1 || tid < kSegMax) {
    t.key[tid] = skey[seg * kSegMax + tid];
    t.pos[tid] = spos[seg * kSegMax + tid];
  }
  for (int q = tid; q < group * kRadix; q += NT) (&s_cnt[0][0])[q] = 0;
  __syncthreads();
  // the segment's keys lie in [lo, hi]
  const uint64_t lo = LEVEL2 && seg > 0 ? skey1[seg] : 0;
  const uint64_t hi = LEVEL2 && seg + 1 < nseg ? skey1[seg + 1] : static_cast<uint64_t>(nrows) << (f.cb - f.kshift);
  const int shift = max(0, 33 - __clzll(static_cast<long long>((hi - lo) | 1)));
  const auto coarse_key = [&](uint64_t k) { return static_cast<uint32_t>((k - lo) >> shift); };
  if (kSide == 1 || tid < kSegMax) t.coarse[tid] = tid == 0 || t.key[tid] == ~uint64_t{0} ? ~0u : coarse_key(t.key[tid]);  // ~0: no record's
  __syncthreads();
  if (tid > 0 && (kSide == 1 || tid < kSegMax)) {  // node tid of the tree: which splitter
    const int level = 31 - __clz(tid);
    t.tree[tid] = t.coarse[((tid - (1 << level)) * 2 + 1) << (kRadixBits - 1 - level)];
  }
  __syncthreads();
  const int nt = min(group, ntiles - tile0);
  // a wave's 64 records from p on: the address is the same for all lanes but for the lane
  const auto load = [&](int p) {
    const int from = min(p, end - 1);  // (beyond the end: the last record, not used)
    return src.from(from).key_near(min(lane, end - 1 - from), f) >> f.kshift;
  };
  const int first = begin + (tile0 + side) * TILE + w * kWave;
  constexpr int kAhead = TILE / kBlock < 8 ? TILE / kBlock : 8;  // keys in flight per thread, across tiles
  uint64_t ahead[kAhead];
#pragma unroll
  for (int k = 0; k < kAhead; ++k) ahead[k] = load(first + k * kBlock);
  for (int q = side; q < nt; q += kSide) {
    int* cnt = s_cnt[q];
#pragma unroll
    for (int k = 0; k < (TILE / kBlock); ++k) {
      const int p = first + (q - side) * TILE + k * kBlock;  // uniform
      const uint64_t key = ahead[k % kAhead];
      ahead[k % kAhead] = load(p + (k + kAhead < TILE / kBlock ? 0 : (kSide - 1) * TILE) + kAhead * kBlock);
      const int d = bucket_of(t, key, p + lane, coarse_key(key));
      if (p + kWave <= end) {  // the whole wave
        // ordered input: a wave's records share a bucket, and adds to one counter are serialised
        if (__all(d == __builtin_amdgcn_readfirstlane(d))) {
          if (lane == 0) atomicAdd(&cnt[d], kWave);
        } else {
          atomicAdd(&cnt[d], 1);
        }
        (dig + p)[lane] = static_cast<uint8_t>(d);
      } else if (p + lane < end) {
        atomicAdd(&cnt[d], 1);
        dig[p + lane] = static_cast<uint8_t>(d);
      }
    }
  }
  __syncthreads();
  const int d = kSide == 1 ? tid : tid % kRadix;
  int32_t* out = hist + base + static_cast<int64_t>(d) * ntiles + tile0;
  for (int q = kSide == 1 ? 0 : tid / kRadix; q < nt; q += kSide) out[q] = s_cnt[q][d];
}

// The counts become offsets, in place. Level 1: a workgroup has the counts of one bucket, which become the records of the
// bucket in the tiles before; total: of all tiles. Level 2: it has a segment's, which become positions in the array.
// (A scan of all counts at once takes two launches and three passes over them: 60M records 2 x 18 us instead of 8 and 10, 3.2M 2 x 11.)
constexpr int kOffBlock = 1024;
template <bool LEVEL2>
__global__ __launch_bounds__(kOffBlock) void offsets_kernel(int ntiles1, const Tables T, int32_t* __restrict__ hist,
                                                            int32_t* __restrict__ total) {
  const int g = blockIdx.x;
  int run = 0;
  int64_t len = ntiles1;
  if (LEVEL2) {
    len = static_cast<int64_t>(T.seg_tile[g + 1] - T.seg_tile[g]) * kRadix;
    hist += static_cast<int64_t>(T.seg_tile[g]) * kRadix;
    run = T.seg_start[g];
  } else {
    hist += static_cast<int64_t>(g) * ntiles1;
  }
  run = block_exclusive_scan<kOffBlock>(hist, len, run);
  if (!LEVEL2 && threadIdx.x == 0) total[g] = run;
}

// Stable scatter of one tile by the noted buckets; ranks as in the radix scatter: a ballot match
// inside the wave plus per-wave counters, then the tile is put in bucket order in LDS so that
// consecutive lanes store to consecutive addresses.
// Level 1: `off` holds the records of a bucket in the tiles before, total1 those of the buckets.
// SELF (few tiles): `off` holds the plain counts, and every workgroup adds up those before its own
// tile itself; the first leaves the start of every bucket in `starts` (one more than buckets).
// Level 2 leaves records in `out` (level 1 keys in it and values in val_out).
template <typename VT, class SRC, bool LEVEL2, int TILE, bool SELF = false>
__global__ __launch_bounds__(part_threads(TILE)) void partition_kernel(const SRC src, const VT* __restrict__ val_in,
                                                           const KeyForm f, int n, int nseg, const Tables T,
                                                           const uint8_t* __restrict__ dig,
                                                           const int32_t* __restrict__ off,
                                                           void* __restrict__ out,
                                                           VT* __restrict__ val_out,
                                                           int32_t* __restrict__ starts,
                                                           const int32_t* __restrict__ total1,
                                                           const uint64_t* __restrict__ skey1,
                                                           const uint64_t* __restrict__ skey2,
                                                           const int32_t* __restrict__ spos2) {
  constexpr int kPart = part_threads(TILE), kPartWaves = kPart / kWave, IPT = TILE / kPart;
  __shared__ int s_cnt[kPartWaves][kRadix];
  __shared__ int s_gdelta[kRadix];
  __shared__ int s_sum[4];
  __shared__ uint64_t s_buf[TILE];
  __shared__ uint8_t s_dig[TILE];
  __shared__ VT s_values[LEVEL2 ? TILE : 1];
  __shared__ uint32_t s_lo[LEVEL2 ? kRadix : 1];  // lower bounds of the buckets' keys, as far as a narrow record needs them
  VT* s_val = LEVEL2 ? s_values : reinterpret_cast<VT*>(s_buf);
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  // (as in the classification)
  if (LEVEL2 && static_cast<int>(blockIdx.x) >= T.seg_tile[nseg]) return;
  const int tile = xcd_contiguous_block_id(blockIdx.x, LEVEL2 ? T.seg_tile[nseg] : static_cast<int>(gridDim.x));
  int begin, end, ntiles, i0, seg = 0;
  int64_t base = 0;
  if (LEVEL2) {
    seg = T.tile_seg[tile];
    const int t0 = T.seg_tile[seg];
    ntiles = T.seg_tile[seg + 1] - t0;
    i0 = tile - t0;
    begin = T.seg_start[seg] + i0 * TILE;
    end = T.seg_start[seg + 1];
    base = static_cast<int64_t>(t0) * kRadix;
  } else {
    ntiles = tiles_in(n, TILE);
    i0 = tile;
    begin = tile * TILE;
    end = n;
  }
  for (int q = tid; q < kPartWaves * kRadix; q += kPart) (&s_cnt[0][0])[q] = 0;
  __syncthreads();
  const int tile_n = min(TILE, end - begin);
  const int wave_base = begin + w * (kWave * IPT);
  int* cnt = s_cnt[w];

  uint64_t key[IPT];
  VT val[IPT];
  int lpos[IPT];  // digit << 16 | rank inside (wave, digit), later the slot in the sorted tile
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int p = min(wave_base + k * kWave + lane, end - 1);
    lpos[k] = dig[p];
    key[k] = src.key_stream(p, f);
    val[k] = __builtin_nontemporal_load(val_in + p);
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const bool valid = wave_base + k * kWave + lane < end;
    const int d = lpos[k];
    const uint64_t same = lanes_with(d, __ballot(valid));
    const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(same >> 32),
                                                 __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(same), 0));
    int basecnt = 0;
    if (valid) basecnt = cnt[d];
    wave_lds_order();
    if (valid && before == 0) cnt[d] = basecnt + __popcll(same);
    wave_lds_order();
    lpos[k] = (d << 16) | (basecnt + before);
  }
  __syncthreads();
  {  // thread d: where digit d starts inside the sorted tile and in global memory
    const int d = tid & (kRadix - 1);
    int c[kPartWaves], tot = 0;
#pragma unroll
    for (int u = 0; u < kPartWaves; ++u) {
      c[u] = s_cnt[u][d];
      tot += c[u];
    }
    int start = wave_inclusive_sum(tot);
    if (lane == kWave - 1) s_sum[w & 3] = start;
    __syncthreads();
    for (int u = 0; u < (w & 3); ++u) start += s_sum[u];
    start -= tot;
    int global = 0;
    if (!SELF) global = off[base + static_cast<int64_t>(d) * ntiles + i0];
    if (!SELF && !LEVEL2) {
      __syncthreads();
      global += bucket_start(total1[d], s_sum);
    }
    if (SELF) {
      int total = 0;  // of this digit over all tiles; `global`: over the tiles before this one
      typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
      const int32_t* counts = off + static_cast<int64_t>(d) * ntiles;
      int q = 0;
#pragma unroll 8
      for (; q + 4 <= ntiles; q += 4) {
        const I4 x = *reinterpret_cast<const I4*>(counts + q);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          total += x[r];
          global += q + r < i0 ? x[r] : 0;
        }
      }
      for (; q < ntiles; ++q) {
        total += counts[q];
        global += q < i0 ? counts[q] : 0;
      }
      int incl = wave_inclusive_sum(total);
      __syncthreads();
      if (lane == kWave - 1) s_sum[w & 3] = incl;
      __syncthreads();
      for (int u = 0; u < (w & 3); ++u) incl += s_sum[u];
      global += incl - total;
      if (i0 == 0 && tid < kRadix) {
        starts[d] = incl - total;
        if (d == kRadix - 1) starts[kRadix] = incl;
      }
    }
    if (tid < kRadix) {
      s_gdelta[d] = global - start;
      if (LEVEL2) {
        s_gdelta[d] -= T.seg_start[seg];
        s_lo[d] = static_cast<uint32_t>((d > 0 ? skey2[seg * kSegMax + d] : seg > 0 ? skey1[seg] : 0) << f.kshift);
      }
#pragma unroll
      for (int u = 0; u < kPartWaves; ++u) {
        s_cnt[u][d] = start;
        start += c[u];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (wave_base + k * kWave + lane < end) {
      const int d = lpos[k] >> 16;
      lpos[k] = (lpos[k] & 0xFFFF) + s_cnt[w][d];
      s_buf[lpos[k]] = key[k];
      s_dig[lpos[k]] = static_cast<uint8_t>(d);
      if (LEVEL2) s_val[lpos[k]] = val[k];
    }
  }
  __syncthreads();
  if constexpr (LEVEL2) {
    char* at = segment_records<VT>(out, T.seg_start[seg]);
    const bool narrow = spos2[seg * kSegMax] != 0;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const int j = k * kPart + tid;
      if (j < tile_n) {
        const int d = s_dig[j], to = j + s_gdelta[d];
        if (narrow) {
          typedef Record<uint32_t, VT> R;
          at32(reinterpret_cast<R*>(at), to) = R::of(static_cast<uint32_t>(s_buf[j]) - s_lo[d], s_val[j]);
        } else {
          typedef Record<uint64_t, VT> R;
          at32(reinterpret_cast<R*>(at), to) = R::of(s_buf[j], s_val[j]);
        }
      }
    }
    return;
  }
  uint64_t* key_out = static_cast<uint64_t*>(out);
  int dst[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int j = k * kPart + tid;
    if (j < tile_n) {
      dst[k] = j + s_gdelta[s_dig[j]];
      key_out[dst[k]] = s_buf[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k)
    if (wave_base + k * kWave + lane < end) s_val[lpos[k]] = val[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int j = k * kPart + tid;
    if (j < tile_n) val_out[dst[k]] = s_val[j];
  }
}

// ---- finish ---------------------------------------------------------------------------------
// The last resort for more records than fit: every record's rank is counted. `in` tells whether the
// record at a position belongs to the bucket.
template <int NT, typename VT, class KA, class VA, class IN>
__device__ void rank_and_store(const KA& key_at, const VA& val_at, int end, const IN& in, int n, int first, int lo_row, int hi_row,
                               const KeyForm& f, int32_t* __restrict__ pos, int32_t* __restrict__ crd_out,
                               VT* __restrict__ val_out) {
  for (int p0 = 0; p0 < end; p0 += NT) {
    const int p = p0 + threadIdx.x;
    bool live = p < end;
    uint64_t K = 0, key = 0;
    if (live) {
      K = key_at(p);
      key = K >> f.kshift;
      live = in(key, p);
    }
    if (!__any(live)) continue;
    int rank = 0, prev = lo_row;
    for (int q = 0; q < end; ++q) {
      const uint64_t k = key_at(q) >> f.kshift;
      if (in(k, q) && (k < key || (k == key && q < p))) {
        ++rank;
        prev = max(prev, f.row_of(k));
      }
    }
    const int row = static_cast<int>(K >> f.cb);
    if (live) {
      crd_out[first + rank] = static_cast<int>(K & ((uint64_t{1} << f.cb) - 1));
      val_out[first + rank] = val_at(p);
    }
    store_pos_range(pos, live ? prev : 0, live ? row : 0, first + rank);
    const bool last = live && rank == n - 1;
    if (__any(last)) store_pos_range(pos, last ? row : 0, last ? hi_row : 0, first + n);
  }
}

// Puts n positions in order.
template <int NT, int E>
__device__ __forceinline__ void sort_positions(uint32_t* at, int n) {
  uint32_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * NT + static_cast<int>(threadIdx.x);
    v[e] = i < n ? at[i] : ~0u;
  }
  __syncthreads();
  block_sort_u32<NT, E>(v, at);
}

// A bucket with more records than fit is split once more: at splitters of a sample of its own, as in the
// selection from a small input, one part after the other. (A part that is too large again has its records'
// ranks counted.)
constexpr int kSplitSamples = 512, kSplitPart = 1536;
constexpr int kSplitBytes = kSplitSamples * 10 + kSplitPart * 10 + 16;
template <int NT, class SRC>
__device__ __forceinline__ void split_and_store(char* mem, const SRC& src, int n, int first, uint64_t lo_key, uint64_t hi_key,
                                                int lo_row, int hi_row, const KeyForm& f, int32_t* __restrict__ pos,
                                                int32_t* __restrict__ crd_out, typename SRC::VT* __restrict__ val_out) {
  typedef typename SRC::VT VT;
  constexpr int S = kSplitSamples, E = kSplitPart / NT;
  uint64_t* s_key = reinterpret_cast<uint64_t*>(mem);
  uint32_t* words = reinterpret_cast<uint32_t*>(mem + S * 8);
  uint32_t* at = words + kSplitPart;
  uint16_t* ord = reinterpret_cast<uint16_t*>(at + kSplitPart);
  uint16_t* s_ord = ord + kSplitPart;
  int* s_cnt = reinterpret_cast<int*>(s_ord + S);
  const int tid = threadIdx.x, lane = lane_id();
  const auto whole_at = [&](int p) { return src.whole(src.key(p)); };
  for (int t = tid; t < S; t += NT) s_key[t] = whole_at(sample_pos<S>(t, n)) >> f.kshift;
  __syncthreads();
  sort_records<NT, S / NT>(words, s_ord, S, coarse_shift(lo_key, hi_key), [&](int t) { return s_key[t] - lo_key; });
  // A part that does not fit has a chance below 1e-6 in a bucket of up to 18 000 records (16 samples to a part), 3e-4 at 37 000
  // and 1e-3 at 60 000; ranks are then counted, in the square of the bucket's records.
  constexpr int kTarget = kSplitPart * 3 / 8;
  const int nb = min(S, (n + kTarget - 1) / kTarget);
  const auto cut_at = [&](int d) {
    const int t = s_ord[d * S / nb];
    return Cut{s_key[t], sample_pos<S>(t, n)};
  };
  for (int d = 0; d < nb; ++d) {
    const Cut lo = d > 0 ? cut_at(d) : Cut{lo_key, -1}, hi = d + 1 < nb ? cut_at(d + 1) : Cut{hi_key, INT32_MAX};
    const int a_row = d > 0 ? f.row_of(lo.key) : lo_row, b_row = d + 1 < nb ? f.row_of(hi.key) : hi_row;
    const auto in = [&](uint64_t key, int p) {
      return (d == 0 || lo.at_or_before(key, p)) && (d + 1 == nb || !hi.at_or_before(key, p));
    };
    if (tid == 0) *s_cnt = 0;
    __syncthreads();
    constexpr int U = 8;
    for (int p0 = tid; p0 < n; p0 += U * NT) {
      uint64_t key[U];
#pragma unroll
      for (int u = 0; u < U; ++u) key[u] = whole_at(min(p0 + u * NT, n - 1)) >> f.kshift;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * NT;
        if (p < n && in(key[u], p)) {
          const int i = atomicAdd(s_cnt, 1);
          if (i < kSplitPart) at[i] = p;
        }
      }
    }
    __syncthreads();
    const int cnt = *s_cnt;
    if (cnt > kSplitPart) {
      rank_and_store<NT, VT>(whole_at, [&](int p) { return src.val(p); }, n, in, cnt, first, a_row, b_row, f, pos, crd_out, val_out);
    } else if (cnt == 0) {
      if (tid < kWave) store_pos_range(pos, lane == 0 ? a_row : 0, lane == 0 ? b_row : 0, first);
    } else {
      sort_positions<NT, E>(at, cnt);  // records are numbered in input order
      sort_records<NT, E>(words, ord, cnt, coarse_shift(lo.key, hi.key),
                          [&](int li) { return (whole_at(at[li]) >> f.kshift) - lo.key; });
      store_entries<NT, E>(ord, cnt, first, a_row, b_row, f, [&](int li) { return whole_at(at[li]); }, pos, crd_out,
                           [&](int j, int li) { val_out[first + j] = src.val(at[li]); });
    }
    first += cnt;
    __syncthreads();
  }
}

// A bucket of n records whose keys lie in [lo, hi], its rows of pos in (lo_row, hi_row]. mem: ROOM bytes of LDS. MOST: words of a
// thread, beyond which the bucket is split.
template <int ROOM, int MOST, class SRC>
__device__ __forceinline__ void finish_bucket(char* mem, const SRC& src, int n, int first, uint64_t lo, uint64_t hi, int lo_row,
                                              int hi_row, const KeyForm& f, int32_t* __restrict__ pos,
                                              int32_t* __restrict__ crd_out, typename SRC::VT* __restrict__ val_out) {
  // as many words of a thread as the records need (six for most; with eight for all of them: 30 us longer for 60M)
#define SPT_FINISH(HOW_, E_)                                                                                              \
  do {                                                                                                                    \
    constexpr int kWords = E_, kLi = number_bits(kFin * kWords);                                                          \
    HOW_<kFin, kWords, kLi>(mem, src, n, first, coarse_shift<kLi>(lo, hi), lo_row, hi_row, f, pos, crd_out, val_out);     \
  } while (0)
  constexpr int kStagedMost = ROOM / (sizeof(typename SRC::KT) + 6) / kFin;
  static_assert(kStagedMost >= 6 && MOST * kFin * 6 <= ROOM && MOST * kFin <= kCap && kSplitBytes <= ROOM, "");
  if (n > MOST * kFin) {
    split_and_store<kFin>(mem, src, n, first, lo, hi, lo_row, hi_row, f, pos, crd_out, val_out);
  } else if (n <= 4 * kFin) {
    SPT_FINISH(finish_staged, 4);
  } else if (n <= 6 * kFin) {
    SPT_FINISH(finish_staged, 6);
  } else if (n <= 8 * kFin) {
    if constexpr (kStagedMost >= 8) SPT_FINISH(finish_staged, 8);
    else SPT_FINISH(finish_direct, 8);
  } else {
    SPT_FINISH(finish_direct, MOST);
  }
#undef SPT_FINISH
}

// One workgroup per bucket of the last partition. LEVELS == 1: of the only one, whose scanned
// counts are off2 and whose splitters are skey2, with nseg buckets, keys and values in arrays (in, val_in).
// LEVELS == 2: records in `in`, those of a segment narrow if spos2 says so.
// Seven workgroups to a compute unit after two levels: the steps of the network wait for each other, and the time goes
// with the number of workgroups that take turns (60M records, fp64: 650 us with three, 534 with four, 468 with five, 419
// with six, 400 with seven). Hence the room in LDS and the registers of a lane. After one level there are no more than 256.
template <typename VT, int LEVELS>
__global__ __launch_bounds__(kFin, LEVELS == 1 ? 5 : 7) void finish_kernel(const void* __restrict__ in, const VT* __restrict__ val_in,
                                                      const KeyForm f, int nseg, int nrows, const Tables T,
                                                      const int32_t* __restrict__ off2,
                                                      const uint64_t* __restrict__ skey1,
                                                      const uint64_t* __restrict__ skey2,
                                                      const int32_t* __restrict__ spos2,
                                                      int32_t* __restrict__ pos, int32_t* __restrict__ crd_out,
                                                      VT* __restrict__ val_out) {
  constexpr int kRoom = LEVELS == 1 ? kStaged * 14 : 14 * kFin * 6;
  __shared__ __attribute__((aligned(16))) char s_mem[kRoom];  // keys, later values, words and order; many records: words and order
  const int g = blockIdx.x;
  int first, end, begin = 0;
  bool narrow = false;
  // the bucket's keys lie in [lo, hi], its rows of pos are (row of lo, row of hi]
  const uint64_t top = static_cast<uint64_t>(nrows) << (f.cb - f.kshift);
  uint64_t lo, hi;
  if (LEVELS == 1) {
    first = off2[g];
    end = off2[g + 1];
    lo = g > 0 ? skey2[g] : 0;
    hi = g + 1 < nseg ? skey2[g + 1] : top;
  } else {
    if (g >= T.seg_bucket[nseg]) return;
    const int seg = T.bucket_seg[g];
    const int d = g - T.seg_bucket[seg], nb = T.seg_bucket[seg + 1] - T.seg_bucket[seg];
    const int nt = T.seg_tile[seg + 1] - T.seg_tile[seg];
    const int64_t base = static_cast<int64_t>(T.seg_tile[seg]) * kRadix;
    first = begin = T.seg_start[seg];
    end = T.seg_start[seg + 1];
    narrow = spos2[seg * kSegMax] != 0;
    if (nt > 0) {
      first = off2[base + static_cast<int64_t>(d) * nt];
      if (d + 1 < nb) end = off2[base + static_cast<int64_t>(d + 1) * nt];
    }
    lo = d > 0 ? skey2[seg * kSegMax + d] : seg > 0 ? skey1[seg] : 0;
    hi = d + 1 < nb ? skey2[seg * kSegMax + d + 1] : seg + 1 < nseg ? skey1[seg + 1] : top;
  }
  const int n = end - first;
  const int lo_row = g > 0 ? f.row_of(lo) : -1, hi_row = f.row_of(hi);
  if (n == 0) {
    if (threadIdx.x < kWave) store_pos_range(pos, threadIdx.x == 0 ? lo_row : 0, threadIdx.x == 0 ? hi_row : 0, first);
    return;
  }
  if constexpr (LEVELS == 1) {
    const ArraysBucket<VT> src{static_cast<const uint64_t*>(in) + first, val_in + first, lo, f.kshift};
    finish_bucket<kRoom, kCap / kFin>(s_mem, src, n, first, lo, hi, lo_row, hi_row, f, pos, crd_out, val_out);
  } else {
    const char* at = segment_records<VT>(in, begin);
    if (narrow) {
      const RecordBucket<uint32_t, VT> src{reinterpret_cast<const Record<uint32_t, VT>*>(at) + (first - begin), lo, f.kshift};
      finish_bucket<kRoom, 14>(s_mem, src, n, first, lo, hi, lo_row, hi_row, f, pos, crd_out, val_out);
    } else {
      const RecordBucket<uint64_t, VT> src{reinterpret_cast<const Record<uint64_t, VT>*>(at) + (first - begin), lo, f.kshift};
      finish_bucket<kRoom, 12>(s_mem, src, n, first, lo, hi, lo_row, hi_row, f, pos, crd_out, val_out);
    }
  }
}

// Small inputs: one workgroup per kSelTarget records. It samples the input, keeps the two
// splitters around its share, and picks its records out of the input.
// Bound by latency: four round trips to memory and two networks (50 000 records: 20 us; 22 with the picked positions
// put in order by a third, and keys and values fetched where they are used; all rows loaded ahead of the sample's sort
// 22, rows between the splitters picked without a look at their keys 20.5).
template <int E, typename VT>
__global__ __launch_bounds__(kSel) void select_finish_kernel(const RcSource src, const VT* __restrict__ val_in,
                                                             const KeyForm f, int n, int nrows,
                                                             int32_t* __restrict__ pos,
                                                             int32_t* __restrict__ crd_out,
                                                             VT* __restrict__ val_out) {
  constexpr int S = kSel * E;
  __shared__ uint64_t s_key[S];
  __shared__ __attribute__((aligned(16))) uint32_t words[kCap];
  __shared__ __attribute__((aligned(16))) int32_t s_at[kCap];  // positions of the bucket's records
  __shared__ uint16_t s_ord[kCap];
  __shared__ uint32_t s_picked[kSelectMax / 32];  // bit per record
  __shared__ int s_sum[kSel / kWave], s_less;
  const int tid = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const int d = blockIdx.x, nb = gridDim.x;
  // ---- splitters
  Cut lo{0, -1}, hi{static_cast<uint64_t>(nrows) << (f.cb - f.kshift), INT32_MAX};
  int lo_row = -1, hi_row = nrows;
  if (nb > 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int t = e * kSel + tid;
      s_key[t] = src.key(sample_pos<S>(t, n), f) >> f.kshift;
    }
    __syncthreads();
    sort_records<kSel, E>(words, s_ord, S, coarse_shift(lo.key, hi.key), [&](int t) { return s_key[t]; });
    if (d > 0) {
      const int t = s_ord[static_cast<int>((static_cast<int64_t>(d) * S) / nb)];
      lo = Cut{s_key[t], sample_pos<S>(t, n)};
      lo_row = f.row_of(lo.key);
    }
    if (d + 1 < nb) {
      const int t = s_ord[static_cast<int>((static_cast<int64_t>(d + 1) * S) / nb)];
      hi = Cut{s_key[t], sample_pos<S>(t, n)};
      hi_row = f.row_of(hi.key);
    }
    __syncthreads();
  }
  const bool cut_below = d > 0, cut_above = d + 1 < nb;
  const auto in = [&](uint64_t key, int p) {
    return (!cut_below || lo.at_or_before(key, p)) && (!cut_above || !hi.at_or_before(key, p));
  };
  // ---- pick: the positions of the bucket's records, and how many records precede it.
  // What decides is the row, except for the rows that the splitters cut; few records qualify.
  constexpr int kWords = kSelectMax / 32 / kSel;  // of a thread
#pragma unroll
  for (int q = 0; q < kWords; ++q) s_picked[q * kSel + tid] = 0;
  if (tid == 0) s_less = 0;
  __syncthreads();
  const int cut_lo = cut_below ? lo_row : -1, cut_hi = cut_above ? hi_row : INT32_MAX;
  int less = 0;
  constexpr int U = 16;
  for (int p0 = tid; p0 < n; p0 += U * kSel) {
    int32_t row[U];
#pragma unroll
    for (int u = 0; u < U; ++u) row[u] = src.row[min(p0 + u * kSel, n - 1)];
    uint32_t maybe = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = p0 + u * kSel < n;
      less += ok && row[u] < cut_lo ? 1 : 0;
      maybe |= ok && row[u] >= cut_lo && row[u] <= cut_hi ? 1u << u : 0u;
    }
    while (maybe) {
      const int u = __ffs(static_cast<int>(maybe)) - 1;
      maybe &= maybe - 1;
      const int p = p0 + u * kSel;
      const uint64_t key = src.key(p, f) >> f.kshift;
      if (cut_below && !lo.at_or_before(key, p)) {
        ++less;
      } else if (!cut_above || !hi.at_or_before(key, p)) {
        atomicOr(&s_picked[p >> 5], 1u << (p & 31));
      }
    }
  }
#pragma unroll
  for (int s = kWave / 2; s > 0; s >>= 1) less += __shfl_xor(less, s);
  if (lane == 0) atomicAdd(&s_less, less);
  __syncthreads();
  // the positions in order, so that records are numbered in input order (sorting them takes another network)
  uint32_t picked[kWords];
  int own = 0;
#pragma unroll
  for (int q = 0; q < kWords; ++q) {
    picked[q] = s_picked[tid * kWords + q];
    own += __popc(picked[q]);
  }
  int at = wave_inclusive_sum(own) - own, cnt = 0;
  if (lane == kWave - 1) s_sum[w] = at + own;
  __syncthreads();
  for (int u = 0; u < kSel / kWave; ++u) {
    if (u < w) at += s_sum[u];
    cnt += s_sum[u];
  }
  // a lane puts those of its words in place; the wave together, where few lanes have many: input in order has them in a
  // few words (20 000 records 13.4 us, 16.6 with a lane for all of its own)
  constexpr int kFewPicked = 10, kFewLanes = 8;
  static_assert(kWords * 32 == kWave, "");
  const uint64_t many = __ballot(own > kFewPicked);
  const bool together = __popcll(many) <= kFewLanes;
  for (uint64_t todo = together ? many : 0; todo; todo &= todo - 1) {
    const int from = __ffsll(static_cast<long long>(todo)) - 1;
    const uint64_t bits = static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(picked[1]), from))) << 32 |
                          static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(picked[0]), from));
    const int place = __builtin_amdgcn_readlane(at, from) + __popcll(bits & ((uint64_t{1} << lane) - 1));
    if ((bits >> lane & 1) && place < kCap) s_at[place] = (w * kWave + from) * kWave + lane;
  }
#pragma unroll
  for (int q = 0; q < kWords; ++q) {
    for (uint32_t m = together && own > kFewPicked ? 0 : picked[q]; m; m &= m - 1, ++at)
      if (at < kCap) s_at[at] = (tid * kWords + q) * 32 + __ffs(static_cast<int>(m)) - 1;
  }
  __syncthreads();
  const int first = s_less;
  if (cnt > kCap) {
    rank_and_store<kSel, VT>([&](int p) { return src.key(p, f); }, [&](int p) { return val_in[p]; }, n, in, cnt, first, lo_row,
                             hi_row, f, pos, crd_out, val_out);
    return;
  }
  if (cnt == 0) {
    if (w == 0) store_pos_range(pos, lane == 0 ? lo_row : 0, lane == 0 ? hi_row : 0, first);
    return;
  }
  const int shift = coarse_shift(lo.key, hi.key);
  const auto key_at = [&](int li) { return src.key(s_at[li], f); };
  const auto rel_at = [&](int li) { return (src.key(s_at[li], f) >> f.kshift) - lo.key; };
  const auto put = [&](int j, int li) { val_out[first + j] = val_in[s_at[li]]; };
#define SPT_FINISH(E_)                                                                                     \
  sort_records<kSel, E_>(words, s_ord, cnt, shift, rel_at);                                              \
  store_entries<kSel, E_>(s_ord, cnt, first, lo_row, hi_row, f, key_at, pos, crd_out, put)
  if (cnt <= kSel) {
    // a record of each thread: keys and values are fetched together, once
    VT* s_val = reinterpret_cast<VT*>(words);
    static_assert(kSel * sizeof(VT) <= sizeof(words), "");
    const int p = s_at[min(tid, cnt - 1)];
    const VT v = val_in[p];
    s_key[tid] = src.key(p, f);
    __syncthreads();
    sort_records<kSel, 1>(words, s_ord, cnt, shift, [&](int li) { return (s_key[li] >> f.kshift) - lo.key; });
    s_val[tid] = v;
    __syncthreads();
    store_entries<kSel, 1>(s_ord, cnt, first, lo_row, hi_row, f, [&](int li) { return s_key[li]; }, pos, crd_out,
                           [&](int j, int li) { val_out[first + j] = s_val[li]; });
  } else if (cnt <= 2 * kSel) {
    SPT_FINISH(2);
  } else {
    SPT_FINISH(4);
  }
#undef SPT_FINISH
}

// ---- host -----------------------------------------------------------------------------------

bool sample_sort_applies(int64_t n) { return n > 0 && n <= kSampleSortMax; }

// Few records: a thread takes eight or 16 of a large tile one after the other (14 us to classify them, whatever n),
// which tiles of 1024 cut (fp64, tiles of 1024 / 4096: 1.2M records 84 / 108 us, 2M 122 / 128, 3M 162 / 160, 4M
// 195 / 185, 6M 259 / 228, whose counts no longer fit the caches). From 2M records on tiles of 2048 (of 1024 / 2048, fp32:
// 1.75M 95 / 96 us, 1.9M 99 / 99, 2.2M 112 / 107, 2.9M 130 / 122; fp64: 101 / 103, 105 / 105, 121 / 114, 137 / 131).
// A single partition's workgroups each add up the counts of all tiles, so it has at most 176 of them.
constexpr int64_t kLeastTileMax = int64_t(15) << 17, kSmallTileMax = int64_t(11) << 18;
static int tile_of(int64_t n) {
  if (n <= kOneLevelMax) return n <= 128 * kSmallTile ? kSmallTile : 2 * kSmallTile;
  return n <= kLeastTileMax ? kSmallTile : n <= kSmallTileMax ? 2 * kSmallTile : kTile;
}
// LDS that the first scatter of large tiles asks for beyond what it uses (46 KB), so that two of its workgroups share a compute
// unit, not three (see above; the second one, which has keys and values in LDS at a time, uses 62 or 78 KB).
constexpr size_t kPartPad = 10 * 1024;
static int64_t tiles_bound(int64_t n) { return (n + tile_of(n) - 1) / tile_of(n) + kSegMax; }

size_t sample_sort_workspace(int dtype, int64_t n) {
  const size_t vsz = dtype == SPT_F64 ? 8 : 4;
  if (n <= kSelectMax) return 256;
  const int levels = n > kOneLevelMax ? 2 : 1;
  const size_t hist = align_up(static_cast<size_t>(tiles_bound(n)) * kRadix * 4, 256);
  size_t b = levels * (align_up(n * 8, 256) + align_up(n * vsz, 256)) + align_up(n, 256);
  b += levels * hist;
  b += align_up(kSegMax * 8, 256) + align_up(kSegMax * 4, 256);
  b += 5 * align_up((kSegMax + 1) * 4, 256);
  if (levels == 2) {
    b += align_up(kSegMax * kSegMax * 8, 256) + align_up(kSegMax * kSegMax * 4, 256);
    b += 2 * align_up(tiles_bound(n) * 4, 256) + align_up((n / kDirTarget + kSegMax + 1) * 4, 256);
  }
  return b + 256;
}

template <typename VT>
spt_status sample_sort_convert(int64_t n64, int64_t nrows, int64_t ncols, bool by_col, const int32_t* row,
                               const int32_t* col, const VT* vals, int32_t* pos_out, int32_t* crd_out,
                               VT* vals_out, void* ws, size_t ws_bytes, hipStream_t s) {
  const int n = static_cast<int>(n64);
  KeyForm f;
  f.cb = bits_for(ncols);
  f.kshift = by_col ? 0 : f.cb;
  const RcSource rc{row, col};
  if (n64 <= kSelectMax) {
    const int nb = (n + kSelTarget - 1) / kSelTarget;
    // six or more samples per share: that a share holds ten times its target has a chance below 1e-17
    hipLaunchKernelGGL((select_finish_kernel<1, VT>), dim3(nb), dim3(kSel), 0, s, rc, vals, f, n,
                       static_cast<int>(nrows), pos_out, crd_out, vals_out);
    SPT_CHECK_LAUNCH("select finish");
    return SPT_OK;
  }
  const bool two = n64 > kOneLevelMax;
  if (!ws || ws_bytes < sample_sort_workspace(sizeof(VT) == 8 ? SPT_F64 : SPT_F32, n64))
    return fail(SPT_ERR_WORKSPACE, "coo_to_csr: workspace of %zu bytes needed, %zu given",
                sample_sort_workspace(sizeof(VT) == 8 ? SPT_F64 : SPT_F32, n64), ws_bytes);
  Workspace W(ws, ws_bytes);
  uint64_t* k1 = W.take<uint64_t>(n);
  VT* v1 = W.take<VT>(n);
  uint8_t* dig = W.take<uint8_t>(n);
  int32_t* hist1 = W.take<int32_t>(tiles_bound(n) * kRadix);
  uint64_t* skey1 = W.take<uint64_t>(kSegMax);
  int32_t* spos1 = W.take<int32_t>(kSegMax);
  Tables T{};

  // level 1
  const int tile = tile_of(n), nt1 = (n + tile - 1) / tile;
  // one level: final buckets; two: up to 256 buckets of sixteen final ones or more
  const int per = two ? 16 * kDirTarget : kDirTarget;
  const int nb1 = std::min(kSegMax, (n + per - 1) / per);
  const int samples = (two ? 16 : 14) * nb1;
#define SPT_RANK(E_)                                                                                                    \
  hipLaunchKernelGGL((rank_splitters_kernel<E_>), dim3(1024 * E_ / kRankSamples), dim3(kRankBlock), 0, s, rc, f, n, nb1, \
                     k1, skey1, spos1)
  if (samples <= 1024) SPT_RANK(1);
  else if (samples <= 2048) SPT_RANK(2);
  else {
    // (in the place of the keys that the first partition writes)
    hipLaunchKernelGGL(pick_samples_kernel, dim3(kMaxSamples / kWave), dim3(kWave), 0, s, rc, f, n, k1);
    SPT_CHECK_LAUNCH("samples");
    SPT_RANK(4);
  }
#undef SPT_RANK
  SPT_CHECK_LAUNCH("splitters");
  // Few tiles: a workgroup for each. From 2048 on, one for four, which shares its table; up to 4096 of twice the threads, as there are hardly
  // enough workgroups (fp64, in us, four tiles by 256 / four by 512 / one by 256: 8.6M 298 / 282 / 284, 12M 354 / 337 / 342, 14.5M
  // 413 / 399 / 408, 16.5M 462 / 458 / 467; 18M 474 / 484 / 481, 30M 761 / 768 / 780, 60M 1503 / 1514 / 1551; 5.4M 192 / 202 / 191).
  const int group = nt1 >= 2048 && tile == kTile ? kGroup : 1;
  const bool wide = group == kGroup && nt1 < 4096;
#define SPT_CLASSIFY(TILE_, ...)                                                                                          \
  hipLaunchKernelGGL((classify_kernel<RcSource, false, TILE_, ##__VA_ARGS__>), dim3((nt1 + group - 1) / group), dim3(wide ? 2 * kBlock : kBlock), 0, s, \
                     rc, f, n, static_cast<int>(nrows), group, 1, T, nullptr, skey1, spos1, dig, hist1)
  if (tile == kSmallTile) SPT_CLASSIFY(kSmallTile);
  else if (tile == 2 * kSmallTile) SPT_CLASSIFY(2 * kSmallTile);
  else if (wide) SPT_CLASSIFY(kTile, 2 * kBlock);
  else SPT_CLASSIFY(kTile);
#undef SPT_CLASSIFY
  SPT_CHECK_LAUNCH("classify");
  const KSource s1{k1};
  if (!two) {
    int32_t* starts = W.take<int32_t>(kSegMax + 1);
    if (tile == kSmallTile)
      hipLaunchKernelGGL((partition_kernel<VT, RcSource, false, kSmallTile, true>), dim3(nt1), dim3(part_threads(kSmallTile)), 0, s, rc,
                         vals, f, n, 1, T, dig, hist1, k1, v1, starts, nullptr, nullptr, nullptr, nullptr);
    else
      hipLaunchKernelGGL((partition_kernel<VT, RcSource, false, 2 * kSmallTile, true>), dim3(nt1), dim3(part_threads(kSmallTile)), 0, s, rc,
                         vals, f, n, 1, T, dig, hist1, k1, v1, starts, nullptr, nullptr, nullptr, nullptr);
    SPT_CHECK_LAUNCH("partition");
    hipLaunchKernelGGL((finish_kernel<VT, 1>), dim3(nb1), dim3(kFin), 0, s, k1, v1, f, nb1, static_cast<int>(nrows), T,
                       starts, nullptr, skey1, nullptr, pos_out, crd_out, vals_out);
    SPT_CHECK_LAUNCH("finish");
    return SPT_OK;
  }
  // level 2's counts are made later: until then their place holds the sizes of level 1's buckets
  int32_t* hist2 = W.take<int32_t>(tiles_bound(n) * kRadix);
  int32_t* total1 = hist2;
  hipLaunchKernelGGL(offsets_kernel<false>, dim3(kRadix), dim3(kOffBlock), 0, s, nt1, T, hist1, total1);
  SPT_CHECK_LAUNCH("offsets");
  if (tile == kSmallTile)
    hipLaunchKernelGGL((partition_kernel<VT, RcSource, false, kSmallTile>), dim3(nt1), dim3(part_threads(kSmallTile)), 0, s, rc, vals, f, n,
                       1, T, dig, hist1, k1, v1, nullptr, total1, nullptr, nullptr, nullptr);
  else if (tile == 2 * kSmallTile)
    hipLaunchKernelGGL((partition_kernel<VT, RcSource, false, 2 * kSmallTile>), dim3(nt1), dim3(part_threads(2 * kSmallTile)), 0, s, rc, vals, f, n,
                       1, T, dig, hist1, k1, v1, nullptr, total1, nullptr, nullptr, nullptr);
  else
    hipLaunchKernelGGL((partition_kernel<VT, RcSource, false, kTile>), dim3(nt1), dim3(part_threads(kTile)), kPartPad, s, rc, vals, f, n, 1, T,
                       dig, hist1, k1, v1, nullptr, total1, nullptr, nullptr, nullptr);
  SPT_CHECK_LAUNCH("partition");

  // level 2
  char* records = W.take<char>(n64 * (sizeof(uint64_t) + sizeof(VT)));
  uint64_t* skey2 = W.take<uint64_t>(kSegMax * kSegMax);
  int32_t* spos2 = W.take<int32_t>(kSegMax * kSegMax);
  T.seg_start = W.take<int32_t>(kSegMax + 1);
  T.seg_tile = W.take<int32_t>(kSegMax + 1);
  T.seg_group = W.take<int32_t>(kSegMax + 1);
  T.seg_bucket = W.take<int32_t>(kSegMax + 1);
  T.group_seg = W.take<int32_t>(tiles_bound(n));
  T.tile_seg = W.take<int32_t>(tiles_bound(n));
  T.bucket_seg = W.take<int32_t>(n / kDirTarget + kSegMax + 1);
  const int samples2 = 32 * static_cast<int>(std::min<int64_t>(kSegMax, n64 / nb1 * 3 / 2 / kDirTarget + 1));
#define SPT_SPLIT(E_)                                                                                                  \
  hipLaunchKernelGGL((splitters_kernel<E_>), dim3(nb1), dim3(1024), 0, s, s1, f, static_cast<int>(nrows), group, tile, \
                     total1, nb1, T, skey1, skey2, spos2)
  if (samples2 <= 1024) SPT_SPLIT(1);
  else if (samples2 <= 2048) SPT_SPLIT(2);
  else SPT_SPLIT(4);
#undef SPT_SPLIT
  SPT_CHECK_LAUNCH("splitters 2");
  const unsigned tiles2 = static_cast<unsigned>(tiles_bound(n));
  if (tile == kSmallTile)
    hipLaunchKernelGGL((classify_kernel<KSource, true, kSmallTile>), dim3(tiles2 / group + kSegMax), dim3(kBlock), 0, s, s1,
                       f, n, static_cast<int>(nrows), group, nb1, T, skey1, skey2, spos2, dig, hist2);
  else if (tile == 2 * kSmallTile)
    hipLaunchKernelGGL((classify_kernel<KSource, true, 2 * kSmallTile>), dim3(tiles2 / group + kSegMax), dim3(kBlock), 0, s, s1,
                       f, n, static_cast<int>(nrows), group, nb1, T, skey1, skey2, spos2, dig, hist2);
  else if (wide)
    hipLaunchKernelGGL((classify_kernel<KSource, true, kTile, 2 * kBlock>), dim3(tiles2 / group + kSegMax), dim3(2 * kBlock), 0, s, s1, f,
                       n, static_cast<int>(nrows), group, nb1, T, skey1, skey2, spos2, dig, hist2);
  else
    hipLaunchKernelGGL((classify_kernel<KSource, true, kTile>), dim3(tiles2 / group + kSegMax), dim3(kBlock), 0, s, s1, f,
                       n, static_cast<int>(nrows), group, nb1, T, skey1, skey2, spos2, dig, hist2);
  SPT_CHECK_LAUNCH("classify 2");
  hipLaunchKernelGGL(offsets_kernel<true>, dim3(nb1), dim3(kOffBlock), 0, s, 0, T, hist2, nullptr);
  SPT_CHECK_LAUNCH("offsets 2");
  if (tile == kSmallTile)
    hipLaunchKernelGGL((partition_kernel<VT, KSource, true, kSmallTile>), dim3(tiles2), dim3(part_threads(kSmallTile)), 0, s, s1, v1, f, n,
                       nb1, T, dig, hist2, records, nullptr, nullptr, nullptr, skey1, skey2, spos2);
  else if (tile == 2 * kSmallTile)
    hipLaunchKernelGGL((partition_kernel<VT, KSource, true, 2 * kSmallTile>), dim3(tiles2), dim3(part_threads(2 * kSmallTile)), 0, s, s1, v1, f, n,
                       nb1, T, dig, hist2, records, nullptr, nullptr, nullptr, skey1, skey2, spos2);
  else
    hipLaunchKernelGGL((partition_kernel<VT, KSource, true, kTile>), dim3(tiles2), dim3(part_threads(kTile)), 0, s, s1, v1, f, n, nb1, T,
                       dig, hist2, records, nullptr, nullptr, nullptr, skey1, skey2, spos2);
  SPT_CHECK_LAUNCH("partition 2");
  hipLaunchKernelGGL((finish_kernel<VT, 2>), dim3(static_cast<unsigned>(n64 / kDirTarget + nb1)), dim3(kFin), 0, s,
                     records, nullptr, f, nb1, static_cast<int>(nrows), T, hist2, skey1, skey2, spos2, pos_out, crd_out,
                     vals_out);
  SPT_CHECK_LAUNCH("finish");
  return SPT_OK;
}

template spt_status sample_sort_convert<uint64_t>(int64_t, int64_t, int64_t, bool, const int32_t*, const int32_t*,
                                                  const uint64_t*, int32_t*, int32_t*, uint64_t*, void*, size_t,
                                                  hipStream_t);
template spt_status sample_sort_convert<uint32_t>(int64_t, int64_t, int64_t, bool, const int32_t*, const int32_t*,
                                                  const uint32_t*, int32_t*, int32_t*, uint32_t*, void*, size_t,
                                                  hipStream_t);

}  // namespace spt
