// Sparse addition with a sparse result, A = B + C: COO + COO and CSR + CSR matrices
// (Section 5.2) and 3rd-order PLUS on COO (Section 5.3), gfx950.
//
// The result's coordinates are the union of the operands' coordinates, enumerated
// in order by the two-way merge of Section 4.4, and the result is assembled by
// appending (Section 3.4 / Table 3: coordinates are produced in order, pos of a CSR
// result is counts + running sum). The merged sequence holds the entries of both operands and,
// for CSR, the start of every row; of two entries with equal coordinates (twins) C's comes first.
// The serial merge becomes:
//   1. add_merge_kernel: a workgroup has a tile of 2048 places of the sequence. B's coordinates
//      go to LDS, every C entry looks up its place among them (inside its row, for CSR), and the
//      tile is noted as three bits per place: C entry, C entry with a twin, row start;
//   2. add_fill_kernel: a lane per place counts bits to find the entry that stands there and where
//      its result goes, copies coordinates and adds values. The running sum of the tiles' results
//      is taken here too. A row start stores its element of pos.
// Many tiles have their ends searched by a kernel of their own (add_cut_kernel) beforehand.
// Everything is deterministic; a value is either copied or the single rounded sum b + c.
// A matrix that is CSR in one operand and COO in the other is brought to the form of B first
// (the result has it): rows expanded, or pos made from the ordered rows.
#include <algorithm>

#include "common.hpp"
#include "merge.hpp"
#include "rows.hpp"
#include "search.hpp"
#include "wavescan.hpp"

namespace spt {

// A tile ends at a multiple of 2047 places, or one later if that keeps twins together.
constexpr int kAddPlaces = 2048;
constexpr int kAddStep = kAddPlaces - 1;
constexpr int kAddWords = kAddPlaces / kWave;  // bits per place, 64 a word
constexpr int kAddIPT = kAddPlaces / kBlock;
// Up to here the workgroups of the merge are all resident at once and search their tiles' ends
// themselves. Beyond, the searches would delay each of a workgroup's tiles.
constexpr int kAddSelfTiles = 2048;
// COO operands are searched over their whole length, by a wave for few tiles (fewest steps), by 16 lanes
// for more (a fourth of the probes, which miss the caches: 1.6M + 800 000 entries, fp64, 38 -> 28 us;
// 20 000 + 10 000 entries 11.0 us by waves, 12.0 by 16 lanes).
constexpr int kAddWaveTiles = 128;
// From here on a search fetches the last coordinate only where the others are the same: its probes of long operands miss the
// caches. Below, a second fetch is one more to wait for. Whole / only where needed, us: rows of 15, fp64, 300 000 + 150 000
// entries 13.3 / 13.4, 500 000 + 250 000 15.9 / 15.8, 800 000 + 400 000 18.8 / 18.3, 2.7M + 1.3M 42.2 / 37.8; three long rows 13.3 /
// 13.7, 15.8 / 16.5, 18.7 / 19.4, 41.8 / 41.6; (since the searches have a launch of their own) 3.8M + 2M 71 / 68, 18M + 14M 317 / 294.
constexpr int kAddWholeTiles = 400;
// Workgroups on a compute unit, as registers allow without scratch memory (and LDS: 160 KB). Merge, of CSR and COO matrices, with six /
// seven / eight, 20M + 10M entries, fp64: call 208 / 203 / 212 us. Fill, of CSR, fp32, with five / six / seven (by registers seven): 20M + 4.7M
// 145 / 142 / 145 us, 2.4M + 2.4M 38.6 / 38.1 / 40.9; COO, fp32, with five / six: 12M + 7.2M 150.8 / 153.3; fp64 has scratch memory with six: 208 / 220.
template <class KL>
constexpr int kAddResident = 6;
template <typename T, int NCRD>
constexpr int kFillResident = sizeof(T) == 4 && NCRD == 1 ? 6 : 5;
constexpr int kCus = 256;

// Keys of the entries of a level list in two parts, so that nothing waits for raw() until key() is
// made of it. from(): this loader, or the other operand's where `other` holds.
struct ColLoader {  // column coordinates of a CSR operand; rows are handled apart
  typedef int32_t Key;
  typedef int32_t Raw;
  const int32_t* a1;
  __device__ __forceinline__ Raw raw(int p) const { return a1[p]; }
  __device__ __forceinline__ static Key key(Raw k) { return k; }
  __device__ __forceinline__ static bool le(const ColLoader& a, int p, const ColLoader& b, int q, bool) { return a.a1[p] <= b.a1[q]; }
  __device__ __forceinline__ ColLoader from(const ColLoader& c, bool other) const { return {other ? c.a1 : a1}; }
};
__device__ __forceinline__ bool key_le(int32_t a, int32_t b) { return a <= b; }
__device__ __forceinline__ bool key_eq(int32_t a, int32_t b) { return a == b; }
template <int ND>
struct CooLoader {  // ND coordinates that fit 63 bits together
  typedef uint64_t Key;
  struct Raw {
    int32_t c[ND];
  };
  const int32_t *a0, *a1, *a2;
  int s0, s1;
  __device__ __forceinline__ Raw raw(int p) const {
    Raw r;
    r.c[0] = a0[p];
    r.c[1] = a1[p];
    if (ND == 3) r.c[ND - 1] = a2[p];
    return r;
  }
  __device__ __forceinline__ Key key(const Raw& r) const {
    Key k = static_cast<Key>(static_cast<uint32_t>(r.c[0])) << s0 | static_cast<Key>(static_cast<uint32_t>(r.c[1])) << s1;
    if (ND == 3) k |= static_cast<uint32_t>(r.c[ND - 1]);
    return k;
  }
  // lazy: the last coordinate is fetched only where the others are the same (see kAddWholeTiles).
  __device__ __forceinline__ static bool le(const CooLoader& a, int p, const CooLoader& b, int q, bool lazy) {
    if (!lazy) return a.key(a.raw(p)) <= b.key(b.raw(q));
    const int32_t i = a.a0[p], k = b.a0[q];
    if (ND == 3) {
      const int32_t j = a.a1[p], l = b.a1[q];
      return i != k ? i < k : j != l ? j < l : a.a2[p] <= b.a2[q];
    }
    return i != k ? i < k : a.a1[p] <= b.a1[q];
  }
  __device__ __forceinline__ CooLoader from(const CooLoader& c, bool o) const {
    return {o ? c.a0 : a0, o ? c.a1 : a1, ND == 3 && o ? c.a2 : a2, s0, s1};
  }
};
struct WideLoader {  // any extents
  typedef Key3 Key;
  typedef Key3 Raw;
  const int32_t *a0, *a1, *a2;
  __device__ __forceinline__ Raw raw(int p) const { return Key3{a0[p], a1[p], a2 ? a2[p] : 0}; }
  __device__ __forceinline__ static Key key(const Raw& r) { return r; }
  __device__ __forceinline__ static bool le(const WideLoader& a, int p, const WideLoader& b, int q, bool) {
    return key_le(a.raw(p), b.raw(q));
  }
  __device__ __forceinline__ WideLoader from(const WideLoader& c, bool o) const {
    return {o ? c.a0 : a0, o ? c.a1 : a1, o ? c.a2 : a2};
  }
};
template <>
constexpr int kAddResident<ColLoader> = 7;
template <>
constexpr int kAddResident<CooLoader<2>> = 7;

template <typename KL>
struct AddOperands {
  KL kb, kc;
  int nb, nc;
  const int32_t *pb, *pc;  // pos, CSR only
  int nrows;               // 0 for COO
  __device__ __forceinline__ int64_t places() const { return static_cast<int64_t>(nb) + nc + nrows; }
};

// the B entries, C entries and row starts before a place
struct AddCut {
  int x, y, r;
};

template <typename KL, bool ROWS, int W>
__device__ __forceinline__ AddCut add_cut(const AddOperands<KL>& o, int64_t d, bool lazy) {
  if (d >= o.places()) return AddCut{o.nb, o.nc, o.nrows};
  AddCut c{0, 0, 0};
  int nb = o.nb, nc = o.nc;
  int64_t e = d;  // entries of the row before the place
  if (ROWS) {
    const int r = group_last_true<W>(0, o.nrows, [&](int q) {
      return static_cast<int64_t>(o.pb[q]) + o.pc[q] + q <= d;
    });
    c = AddCut{o.pb[r], o.pc[r], r};
    e = d - (static_cast<int64_t>(c.x) + c.y + r) - 1;
    if (e < 0) return c;  // the row's start is the place
    c.r = r + 1;
    nb = o.pb[r + 1] - c.x;
    nc = o.pc[r + 1] - c.y;
  }
  // B's entry q is among the first e of the row if it is smaller than C's entry e - 1 - q
  const int64_t lo = max<int64_t>(0, e - nc), hi = min<int64_t>(e, nb);
  const int x = group_last_true<W>(lo, hi + 1, [&](int q) {
    return q == lo || !KL::le(o.kc, c.y + static_cast<int>(e - q), o.kb, c.x + q - 1, lazy);
  });
  const int y = static_cast<int>(e - x);
  const bool twins = y > 0 && x < nb && key_eq(o.kc.key(o.kc.raw(c.y + y - 1)), o.kb.key(o.kb.raw(c.x + x)));
  c.x += x + (twins ? 1 : 0);
  c.y += y;
  return c;
}

// Bound by its probes, which miss the caches: a wave per search, which needs the fewest steps, makes
// four times as many of them as 8 lanes (COO, 10M + 5M entries: 62 us, with 8 lanes 20 us).
constexpr int kCutLanes = 8;
template <typename KL, bool ROWS>
__global__ __launch_bounds__(kBlock) void add_cut_kernel(const AddOperands<KL> o, int ntiles,
                                                         AddCut* __restrict__ cuts) {
  const int t = (blockIdx.x * kBlock + threadIdx.x) / kCutLanes;
  if (t > ntiles) return;
  const AddCut c = add_cut<KL, ROWS, kCutLanes>(o, static_cast<int64_t>(t) * kAddStep, true);
  if (threadIdx.x % kCutLanes == 0) cuts[t] = c;
}

// bits 0 to 7 of the result: the bit m (a value below 128) of bytes 0 to 7, times m
__device__ __forceinline__ int gather_bits(uint64_t bytes, uint32_t m) {
  const uint32_t each = m * 0x01010101u;
  const uint32_t low = __builtin_amdgcn_udot4(static_cast<uint32_t>(bytes) & each, 0x08040201u, 0, false);
  return static_cast<int>(__builtin_amdgcn_udot4(static_cast<uint32_t>(bytes >> 32) & each, 0x80402010u, low, false));
}

// What one thread has of a tile: where it lies and its share of the coordinates, as loaded.
template <typename KL>
struct AddTile {
  AddCut a;
  int nb, nc, nr;
  typename KL::Raw raw[kAddIPT];  // of the tile's C entries and, following them, its B entries
  int p0, q0, q1;  // pos of a row in B, in C and of the next in C

  __device__ __forceinline__ void place(const AddCut& from, const AddCut& to) {
    a = from;
    nb = to.x - a.x;
    nc = to.y - a.y;
    nr = to.r - a.r;
    // a pos that descends would make tiles of any size: nothing is taken from such a tile
    if (nb < 0 || nc < 0 || nr < 0 || nb > kAddPlaces || nc > kAddPlaces || nb + nc + nr > kAddPlaces) nb = nc = nr = 0;
  }
  template <bool ROWS>
  __device__ __forceinline__ void load(const AddOperands<KL>& o) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kAddIPT; ++k)
      if (k * kBlock < nb + nc) {
        const int q = min(k * kBlock + tid, nb + nc - 1);
        raw[k] = o.kc.from(o.kb, q >= nc).raw(q + (q < nc ? a.y : a.x - nc));
      }
    if (ROWS) {
      const int r = min(max(a.r - 1 + tid, 0), o.nrows - 1);
      p0 = o.pb[r];
      q0 = o.pc[r];
      q1 = o.pc[r + 1];
    }
  }
};

// SELF: few tiles, one for each workgroup, whose ends are searched here and stored in cuts.
// Otherwise the workgroups that are resident at once go through the tiles and load the next tile's
// coordinates before they look up this one's. Bound by vector instructions, most of them in the
// lookups (20M + 10M CSR entries, fp64: 49 us; 115 us as a walk of 7 merge steps per thread, which
// also needed the rows expanded to a list, 95 us).
template <typename KL, bool ROWS, bool UNION, bool SELF>
__global__ __launch_bounds__(kBlock, kAddResident<KL>) void add_merge_kernel(const AddOperands<KL> o, int ntiles,
                                                           AddCut* __restrict__ cuts, uint64_t* __restrict__ bits,
                                                           int32_t* __restrict__ counts) {
  typedef typename KL::Key Key;
  constexpr int kBits = ROWS ? 3 : 2;
  __shared__ Key s_b[kAddPlaces];
  __shared__ uint64_t s_kind[kAddPlaces / 8];              // a byte per place: 1 C entry, 2 with a twin, 4 row start
  __shared__ uint16_t s_start[ROWS ? kAddPlaces + 2 : 1];  // first B entry of the tile's rows
  __shared__ uint16_t s_row[ROWS ? kAddPlaces : 1];        // at the first C entry of a row: the row
  __shared__ uint32_t s_first[ROWS ? kAddPlaces / 32 : 1];  // bit per C entry: first of a row
  __shared__ AddCut s_cut[2];
  __shared__ int s_twins[kBlock / kWave];
  const int tid = threadIdx.x, lane = lane_id();
  uint8_t* kind = reinterpret_cast<uint8_t*>(s_kind);
  static_assert(kAddPlaces == 8 * kBlock, "a thread turns eight bytes to bits");
  s_kind[tid] = 0;
  if (ROWS && tid < kAddPlaces / 32) s_first[tid] = 0;

  int tile = blockIdx.x;
  AddTile<KL> t, next;
  if (SELF) {
    if (wave_id() < 2) {
      const int64_t d = (static_cast<int64_t>(tile) + wave_id()) * kAddStep;
      const AddCut c = ROWS || ntiles <= kAddWaveTiles ? add_cut<KL, ROWS, kWave>(o, d, false)
                                                       : add_cut<KL, ROWS, 16>(o, d, ntiles > kAddWholeTiles);
      if (lane == 0) {
        s_cut[wave_id()] = c;
        if (wave_id() == 0 || tile == ntiles - 1) cuts[tile + wave_id()] = c;
      }
    }
    __syncthreads();
    t.place(s_cut[0], s_cut[1]);
  } else {
    t.place(cuts[tile], cuts[tile + 1]);
  }
  t.template load<ROWS>(o);
  for (;;) {
    const int tile2 = tile + gridDim.x;
    const bool more = !SELF && tile2 < ntiles;
    AddCut a2, b2;
    if (more) {
      a2 = cuts[tile2];
      b2 = cuts[tile2 + 1];
    }
#pragma unroll
    for (int k = 0; k < kAddIPT; ++k) {
      const int q = k * kBlock + tid - t.nc;
      if (q >= 0 && q < t.nb) s_b[q] = o.kb.key(t.raw[k]);
    }
    if (!SELF) lds_barrier();  // s_kind and s_first are clear
    if (ROWS) {
      // row 0 is the one that the tile's start cuts (it may be empty here), the others start in the tile
      int p0 = t.p0, q0 = t.q0, q1 = t.q1;
      for (int j = tid; j <= t.nr; j += kBlock) {
        const int r = t.a.r - 1 + j;
        if (j >= kBlock) {
          p0 = o.pb[r];
          q0 = o.pc[r];
          q1 = o.pc[r + 1];
        }
        int bs = 0, cs = 0, ce = 0;
        if (r >= 0) {
          bs = min(max(p0 - t.a.x, 0), t.nb);
          cs = min(max(q0 - t.a.y, 0), t.nc);
          ce = min(max(q1 - t.a.y, 0), t.nc);
        }
        s_start[j] = static_cast<uint16_t>(bs);
        if (j > 0) kind[bs + cs + j - 1] = 4;
        if (cs < ce) {
          s_row[cs] = static_cast<uint16_t>(j);
          atomicOr(&s_first[cs >> 5], 1u << (cs & 31));
        }
      }
      if (tid == 0) s_start[t.nr + 1] = static_cast<uint16_t>(t.nb);
    }
    lds_barrier();
    if (more) {
      next.place(a2, b2);
      next.template load<ROWS>(o);
    }
    // (bound by the number of instructions, not by the latency of the steps: looking up two or four
    // entries of a thread together is 5 to 15 us slower for 20M + 10M entries)
#pragma unroll
    for (int k = 0; k < kAddIPT; ++k) {
      const int y = k * kBlock + tid;
      if (y < t.nc) {
        const Key key = o.kc.key(t.raw[k]);
        int j = 0, lo = 0, hi = t.nb;
        if (ROWS) {
          int w = y >> 5;
          uint32_t m = s_first[w] & ((2u << (y & 31)) - 1);
          while (m == 0 && w > 0) m = s_first[--w];
          j = s_row[max(w * 32 + 31 - __clz(m), 0)];
          lo = s_start[j];
          hi = s_start[j + 1];
        }
        const int end = hi;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (key_le(key, s_b[mid])) hi = mid; else lo = mid + 1;
        }
        const bool twin = lo < end && key_eq(s_b[lo], key);
        kind[y + lo + j] = twin ? 3 : 1;
      }
    }
    lds_barrier();
    if (ROWS && tid < kAddPlaces / 32) s_first[tid] = 0;
    // eight places of a thread: bytes to bits, and clear for the next tile
    const uint64_t kd = s_kind[tid];
    s_kind[tid] = 0;
    uint8_t* out = reinterpret_cast<uint8_t*>(bits + static_cast<int64_t>(tile) * kBits * kAddWords) + tid;
    const int twin_bits = gather_bits(kd, 2) >> 1;
    out[0] = static_cast<uint8_t>(gather_bits(kd, 1));
    out[8 * kAddWords] = static_cast<uint8_t>(twin_bits);
    if (ROWS) out[16 * kAddWords] = static_cast<uint8_t>(gather_bits(kd, 4) >> 2);
    const int twins = wave_inclusive_sum(__popc(twin_bits));
    if (lane == kWave - 1) s_twins[wave_id()] = twins;
    lds_barrier();
    if (tid == 0) {
      int all = 0;
      for (int w = 0; w < kBlock / kWave; ++w) all += s_twins[w];
      counts[tile] = UNION ? t.nb + t.nc - all : all;
    }
    if (!more) break;
    t = next;
    tile = tile2;
  }
}

// n and the bits of m below this lane's
__device__ __forceinline__ int bits_below(uint64_t m, int n) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), n));
}

struct CoordArrays {
  const int32_t *a0, *a1, *a2;  // a0 == nullptr for CSR, a2 == nullptr for matrices
};
struct CoordOut {
  int32_t *a0, *a1, *a2;
};

// x of one lane (the same for the whole wave)
__device__ __forceinline__ int lane_value(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
__device__ __forceinline__ uint64_t lane_value(uint64_t x, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(x), lane);
  return static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(x >> 32), lane))) << 32 | lo;
}

// Bound by memory traffic (20M + 10M CSR entries, fp64: 150 us, 4.4 TB/s). The workgroups that are
// resident at once go through the tiles, so that only the counts of the tiles between one and the
// next have to be added up.
template <typename T, int NCRD, bool UNION>
__global__ __launch_bounds__(kBlock, (kFillResident<T, NCRD>)) void add_fill_kernel(
    int ntiles, const AddCut* __restrict__ cuts, const uint64_t* __restrict__ bits, const int32_t* __restrict__ counts,
    int nb, int nc, int nrows, const CoordArrays B, const T* __restrict__ bv, const CoordArrays C,
    const T* __restrict__ cv, const CoordOut O, T* __restrict__ ov, int32_t* __restrict__ pos,
    int64_t* __restrict__ out_nnz) {
  constexpr bool ROWS = NCRD == 1;
  constexpr int kBits = ROWS ? 3 : 2;
  constexpr int kPart = kAddPlaces / kWave / (kBlock / kWave);  // words of a wave
  __shared__ int s_sum[2][kBlock / kWave];
  const int tid = threadIdx.x, lane = lane_id();
  const int w0 = __builtin_amdgcn_readfirstlane(wave_id() * kPart);

  int off = 0, from = 0, parity = 0;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x, parity ^= 1) {
    const AddCut a = cuts[tile], b = cuts[tile + 1];
    // lane w has word w of the three bit sets
    const uint64_t* in = bits + static_cast<int64_t>(tile) * kBits * kAddWords + lane % kAddWords;
    const uint64_t wc = in[0], wt = in[kAddWords], wr = ROWS ? in[2 * kAddWords] : 0;
    int before = 0;
    for (int t = from + tid; t < tile; t += kBlock) before += counts[t];
    before = wave_inclusive_sum(before);
    if (lane == kWave - 1) s_sum[parity][wave_id()] = before;
    const int nct = __popcll(wc) | __popcll(wt) << 16, pct = wave_inclusive_sum(nct) - nct;
    const int pr = ROWS ? wave_inclusive_sum(__popcll(wr)) - __popcll(wr) : 0;
    lds_barrier();
    for (int w = 0; w < kBlock / kWave; ++w) off += s_sum[parity][w];
    from = tile;
    const int places = (b.x - a.x) + (b.y - a.y) + (b.r - a.r);
    T v[kPart], u[kPart];
    int32_t c0[kPart], c1[kPart], c2[kPart];
    int dst[kPart];  // where the place's result goes; -1: no result
    bool both[kPart];
    uint64_t last = w0 > 0 ? lane_value(wt, max(w0 - 1, 0)) >> 63 : 0;
#pragma unroll
    for (int k = 0; k < kPart; ++k) {
      const int w = w0 + k, place = w * kWave + lane;
      const uint64_t mc = lane_value(wc, w), mt = lane_value(wt, w), mr = ROWS ? lane_value(wr, w) : 0;
      const int p = lane_value(pct, w);
      const int before_c = bits_below(mc, p & 0xFFFF), before_t = bits_below(mt, p >> 16);
      const int before_r = ROWS ? bits_below(mr, lane_value(pr, w)) : 0;
      const bool is_c = mc >> lane & 1, is_t = mt >> lane & 1, is_r = mr >> lane & 1, live = place < places;
      both[k] = (mt << 1 | last) >> lane & 1;
      last = mt >> 63;
      const int at = off + (UNION ? place - before_r - before_t : before_t);
      if (ROWS && is_r && live) pos[a.r + before_r] = at;
      dst[k] = live && !is_r && (UNION ? !is_t : both[k]) ? (UNION ? at : at - 1) : -1;
      // (the bounds matter for operands only whose coordinates are not ordered)
      const unsigned ib = min(static_cast<unsigned>(a.x + place - before_c - before_r), static_cast<unsigned>(nb - 1));
      const unsigned ic = min(static_cast<unsigned>(a.y + before_c - (is_c ? 0 : 1)), static_cast<unsigned>(nc - 1));
      if (dst[k] >= 0) {
        const bool own_c = UNION && is_c;
        const T* pv = own_c ? cv + ic : bv + ib;
        v[k] = *pv;
        if (both[k]) u[k] = cv[ic];  // (for all lanes, the others' own value once more: 20M + 10M CSR entries, fp32, 189 us, so 177)
        c1[k] = *(own_c ? C.a1 + ic : B.a1 + ib);
        if (NCRD >= 2) c0[k] = *(own_c ? C.a0 + ic : B.a0 + ib);
        if (NCRD >= 3) c2[k] = *(own_c ? C.a2 + ic : B.a2 + ib);
      }
    }
#pragma unroll
    for (int k = 0; k < kPart; ++k) {
      if (dst[k] < 0) continue;
      T r = v[k];
      if (both[k]) {
        if (UNION) r += u[k];
        else r *= u[k];
      }
      ov[dst[k]] = r;
      O.a1[dst[k]] = c1[k];
      if (NCRD >= 2) O.a0[dst[k]] = c0[k];
      if (NCRD >= 3) O.a2[dst[k]] = c2[k];
    }
    if (tile == ntiles - 1 && tid == 0) {
      const int all = off + counts[tile];
      *out_nnz = all;
      if (ROWS) pos[nrows] = all;
    }
  }
}

// ---- CSR operands ----------------------------------------------------------

constexpr int kExpIPT = 8;
constexpr int kExpChunk = kExpIPT * kBlock;

// rows[p] = row of entry p of a CSR matrix, for a chunk of 2048 entries per workgroup:
// rows that start inside the chunk mark their first entry in LDS, every entry then takes
// the last mark at or before it (running maximum, rows ascend), entries before the first
// mark belong to the row cut by the chunk's start. Balanced for any row-length skew.
__global__ __launch_bounds__(kBlock) void expand_rows_kernel(int nnz, int nrows,
                                                             const int32_t* __restrict__ pos,
                                                             int32_t* __restrict__ rows) {
  __shared__ int32_t s_mark[kExpChunk];
  __shared__ int s_bounds[2];
  __shared__ int s_wmax[kBlock / kWave];
  const int base = blockIdx.x * kExpChunk;
  const int end = min(base + kExpChunk, nnz);
  // first row with pos > base, minus one = row holding entry `base`; likewise for the last entry
  if (wave_id() == 0) {
    const int r = wave_lower_bound(pos, nrows + 1, base + 1) - 1;
    if (lane_id() == 0) s_bounds[0] = r;
  } else if (wave_id() == 1) {
    const int r = wave_lower_bound(pos, nrows + 1, end) - 1;
    if (lane_id() == 0) s_bounds[1] = r;
  }
  for (int e = threadIdx.x; e < kExpChunk; e += kBlock) s_mark[e] = -1;
  __syncthreads();
  const int r_lo = s_bounds[0], r_hi = s_bounds[1];
  strided(r_lo + 1, r_hi + 1, threadIdx.x, kBlock, [&](int r) {
    const int a = pos[r];
    if (pos[r + 1] > a) s_mark[a - base] = r;  // empty rows own no entry
  });
  __syncthreads();
  int32_t local[kExpIPT];
  int run = -1;
#pragma unroll
  for (int k = 0; k < kExpIPT; ++k) {
    const int m = s_mark[threadIdx.x * kExpIPT + k];
    run = m > run ? m : run;
    local[k] = run;
  }
  // exclusive running maximum over the threads before this one
  int inc = run;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int u = __shfl_up(inc, d);
    if (lane_id() >= d) inc = u > inc ? u : inc;
  }
  if (lane_id() == kWave - 1) s_wmax[wave_id()] = inc;
  __syncthreads();
  int before = __shfl_up(inc, 1);
  if (lane_id() == 0) before = -1;
  for (int w = 0; w < wave_id(); ++w) before = s_wmax[w] > before ? s_wmax[w] : before;
  if (before < r_lo) before = r_lo;
#pragma unroll
  for (int k = 0; k < kExpIPT; ++k) {
    const int p = base + threadIdx.x * kExpIPT + k;
    if (p < end) rows[p] = local[k] > before ? local[k] : before;
  }
}

// the result without entries
__global__ __launch_bounds__(kBlock) void add_empty_kernel(int32_t* __restrict__ pos, int64_t n,
                                                           int64_t* __restrict__ out_nnz) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (i < n) pos[i] = 0;
  if (out_nnz && i == 0) *out_nnz = 0;
}

// ---- host ------------------------------------------------------------------

// parent[p] = index of the pos segment that holds position p (the row of a CSR entry, the
// column of a CSC entry); used by other translation units as well
spt_status launch_expand_parents(int n, int nparents, const int32_t* pos, int32_t* out, hipStream_t s) {
  if (n <= 0) return SPT_OK;
  hipLaunchKernelGGL(expand_rows_kernel, dim3((n + kExpChunk - 1) / kExpChunk), dim3(kBlock), 0, s, n,
                     nparents, pos, out);
  SPT_CHECK_LAUNCH("expand parents");
  return SPT_OK;
}

static int64_t add_tiles(int64_t places) { return (places + kAddStep - 1) / kAddStep; }

// fb / fc: formats of the operands (matrices may mix CSR and COO; the result takes B's format)
size_t add_workspace(Format fb, Format fc, const spt_tensor* B, const spt_tensor* C) {
  const bool rows = fb == Format::CSR;
  const int64_t nt = add_tiles(B->nvals + C->nvals + (rows ? B->level[0].N : 0));
  size_t n = align_up(static_cast<size_t>(nt + 1) * sizeof(AddCut), 256) + align_up(static_cast<size_t>(nt) * 4, 256) +
             align_up(static_cast<size_t>(nt) * (rows ? 3 : 2) * kAddWords * 8, 256) + 256;
  if (fb != fc) n += align_up(static_cast<size_t>(rows ? B->level[0].N + 1 : C->nvals) * 4, 256);
  return n;
}

template <typename KL, bool ROWS, bool UNION>
static spt_status launch_add_merge(const AddOperands<KL>& o, int ntiles, AddCut* cuts, uint64_t* bits,
                                   int32_t* counts, hipStream_t s) {
  if (ntiles > kAddSelfTiles) {
    hipLaunchKernelGGL((add_cut_kernel<KL, ROWS>), dim3((ntiles * kCutLanes + kBlock) / kBlock), dim3(kBlock),
                       0, s, o, ntiles, cuts);
    SPT_CHECK_LAUNCH("add cut");
    hipLaunchKernelGGL((add_merge_kernel<KL, ROWS, UNION, false>), dim3(std::min(ntiles, kAddResident<KL> * kCus)), dim3(kBlock), 0, s,
                       o, ntiles, cuts, bits, counts);
  } else {
    hipLaunchKernelGGL((add_merge_kernel<KL, ROWS, UNION, true>), dim3(ntiles), dim3(kBlock), 0, s, o, ntiles, cuts,
                       bits, counts);
  }
  SPT_CHECK_LAUNCH("add merge");
  return SPT_OK;
}

template <typename T, bool UNION>
static spt_status add_typed(Format fb, Format fc, const spt_tensor* B, const spt_tensor* C,
                            int32_t* out_pos, int32_t* out_crd0, int32_t* out_crd1, int32_t* out_crd2,
                            T* out_vals, int64_t* out_nnz, void* ws, size_t ws_bytes, hipStream_t s) {
  const int64_t nb64 = B->nvals, nc64 = C->nvals, N = B->level[0].N;
  if (nb64 + nc64 + kAddPlaces >= INT32_MAX)
    return fail(SPT_ERR_UNSUPPORTED, "add: more than 2^31 entries in both operands together");
  const bool rows = fb == Format::CSR;
  if (rows && N + 1 >= INT32_MAX) return fail(SPT_ERR_UNSUPPORTED, "add: too many rows");
  const int nb = static_cast<int>(nb64), nc = static_cast<int>(nc64);
  if (UNION ? nb == 0 && nc == 0 : nb == 0 || nc == 0) {
    const int64_t n = rows ? N + 1 : 0;
    hipLaunchKernelGGL(add_empty_kernel, dim3(static_cast<unsigned>(std::max<int64_t>(1, (n + kBlock - 1) / kBlock))),
                       dim3(kBlock), 0, s, out_pos, n, out_nnz);
    SPT_CHECK_LAUNCH("add empty");
    return SPT_OK;
  }
  const size_t need = add_workspace(fb, fc, B, C);
  if (!ws || ws_bytes < need)
    return fail(SPT_ERR_WORKSPACE, "add: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  const int nrows = rows ? static_cast<int>(N) : 0;
  const int ntiles = static_cast<int>(add_tiles(nb64 + nc64 + nrows));
  Workspace W(ws, ws_bytes);
  AddCut* cuts = W.take<AddCut>(static_cast<size_t>(ntiles) + 1);
  int32_t* counts = W.take<int32_t>(ntiles);
  const int grid = std::min(ntiles, (rows ? kFillResident<T, 1> : kFillResident<T, 2>) * kCus);
  uint64_t* bits = W.take<uint64_t>(static_cast<size_t>(ntiles) * (rows ? 3 : 2) * kAddWords);

  const T *bv = static_cast<const T*>(B->vals), *cv = static_cast<const T*>(C->vals);
  spt_status st;
  if (rows) {
    const int32_t* pc = C->level[1].pos;
    if (fc != Format::CSR) {
      int32_t* p = W.take<int32_t>(static_cast<size_t>(N) + 1);
      if (nc > 0) {
        st = launch_pos_from_sorted_rows(C->level[0].crd, nc, nrows, p, s);
        if (st != SPT_OK) return st;
      } else {
        hipLaunchKernelGGL(add_empty_kernel, dim3(static_cast<unsigned>((N + kBlock) / kBlock)), dim3(kBlock), 0, s, p,
                           N + 1, nullptr);
        SPT_CHECK_LAUNCH("add empty rows");
      }
      pc = p;
    }
    const CoordArrays cb{nullptr, B->level[1].crd, nullptr}, cc{nullptr, C->level[1].crd, nullptr};
    const AddOperands<ColLoader> o{{cb.a1}, {cc.a1}, nb, nc, B->level[1].pos, pc, nrows};
    st = launch_add_merge<ColLoader, true, UNION>(o, ntiles, cuts, bits, counts, s);
    if (st != SPT_OK) return st;
    hipLaunchKernelGGL((add_fill_kernel<T, 1, UNION>), dim3(grid), dim3(kBlock), 0, s, ntiles, cuts, bits, counts, nb,
                       nc, nrows, cb, bv, cc, cv, CoordOut{nullptr, out_crd1, nullptr}, out_vals, out_pos, out_nnz);
    SPT_CHECK_LAUNCH("add fill");
    return SPT_OK;
  }
  const bool third = fb == Format::COO3;
  const CoordArrays cb{B->level[0].crd, B->level[1].crd, third ? B->level[2].crd : nullptr};
  CoordArrays cc{C->level[0].crd, C->level[1].crd, third ? C->level[2].crd : nullptr};
  if (fc == Format::CSR) {
    int32_t* r = W.take<int32_t>(nc);
    st = launch_expand_parents(nc, static_cast<int>(N), C->level[1].pos, r, s);
    if (st != SPT_OK) return st;
    cc.a0 = r;
  }
  const int w1 = key_bits_of(B->level[1].N), w2 = third ? key_bits_of(B->level[2].N) : 0;
  if (key_bits_of(N) + w1 + w2 > 63) {
    const AddOperands<WideLoader> o{{cb.a0, cb.a1, cb.a2}, {cc.a0, cc.a1, cc.a2}, nb, nc, nullptr, nullptr, 0};
    st = launch_add_merge<WideLoader, false, UNION>(o, ntiles, cuts, bits, counts, s);
  } else if (third) {
    const AddOperands<CooLoader<3>> o{{cb.a0, cb.a1, cb.a2, w1 + w2, w2}, {cc.a0, cc.a1, cc.a2, w1 + w2, w2},
                                      nb, nc, nullptr, nullptr, 0};
    st = launch_add_merge<CooLoader<3>, false, UNION>(o, ntiles, cuts, bits, counts, s);
  } else {
    const AddOperands<CooLoader<2>> o{{cb.a0, cb.a1, nullptr, w1, 0}, {cc.a0, cc.a1, nullptr, w1, 0},
                                      nb, nc, nullptr, nullptr, 0};
    st = launch_add_merge<CooLoader<2>, false, UNION>(o, ntiles, cuts, bits, counts, s);
  }
  if (st != SPT_OK) return st;
  const CoordOut co{out_crd0, out_crd1, out_crd2};
  if (third)
    hipLaunchKernelGGL((add_fill_kernel<T, 3, UNION>), dim3(grid), dim3(kBlock), 0, s, ntiles, cuts, bits, counts, nb,
                       nc, 0, cb, bv, cc, cv, co, out_vals, nullptr, out_nnz);
  else
    hipLaunchKernelGGL((add_fill_kernel<T, 2, UNION>), dim3(grid), dim3(kBlock), 0, s, ntiles, cuts, bits, counts, nb,
                       nc, 0, cb, bv, cc, cv, co, out_vals, nullptr, out_nnz);
  SPT_CHECK_LAUNCH("add fill");
  return SPT_OK;
}

// op: 0 = addition (union merge), 1 = element-wise multiplication (intersection merge)
spt_status add_dispatch(int op, Format fb, Format fc, const spt_tensor* B, const spt_tensor* C,
                        int32_t* out_pos, int32_t* out_crd0, int32_t* out_crd1, int32_t* out_crd2,
                        void* out_vals, int64_t* out_nnz, void* ws, size_t ws_bytes, hipStream_t s) {
  if (B->dtype == SPT_F64) {
    double* ov = static_cast<double*>(out_vals);
    return op == 0 ? add_typed<double, true>(fb, fc, B, C, out_pos, out_crd0, out_crd1, out_crd2, ov,
                                             out_nnz, ws, ws_bytes, s)
                   : add_typed<double, false>(fb, fc, B, C, out_pos, out_crd0, out_crd1, out_crd2, ov,
                                              out_nnz, ws, ws_bytes, s);
  }
  float* ov = static_cast<float*>(out_vals);
  return op == 0 ? add_typed<float, true>(fb, fc, B, C, out_pos, out_crd0, out_crd1, out_crd2, ov,
                                          out_nnz, ws, ws_bytes, s)
                 : add_typed<float, false>(fb, fc, B, C, out_pos, out_crd0, out_crd1, out_crd2, ov,
                                           out_nnz, ws, ws_bytes, s);
}

}  // namespace spt
