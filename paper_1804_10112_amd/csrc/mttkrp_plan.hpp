// MTTKRP: how the entries are dealt to workgroups and their groups of lanes, and the columns to parts.
#pragma once
#include <algorithm>

#include "common.hpp"

namespace spt {

template <typename T>
constexpr int kVec = 16 / sizeof(T);
constexpr int kLine = 128;
constexpr int kCarryCols = 32, kCarryRows = 8, kCarrySpan = kBlock / kCarryCols * kCarryRows;  // a workgroup of the carries

// Which workgroup takes what: the XCDs are dealt to the parts of the columns in turn, and the chunks to a part's XCDs, in turn
// or, ordered, an equal stretch of the order to each. (Workgroups beyond an XCD's chunks return.)
struct Placing {
  int nchunks, parts, cols;  // cols: of a part
  bool ordered;
};
// The first of the V columns that vector v of a part has, a part being `cols` columns. The last vector of a part ends with the part (it repeats
// columns of the one before if cols is no multiple of V); vectors beyond repeat it, and *keeps says whether this one's sums are anybody's.
__host__ __device__ __forceinline__ int column_of(int cols, int V, int part, int v, bool* keeps) {
  *keeps = v * V < cols;
  return part * cols + (v * V < cols - V ? v * V : cols - V);
}

struct MttkrpPlan {
  int lanes, vec, tiles, epg, chunk, parts;  // tiles: of `lanes` vectors, of a part
  int64_t n1, n2;  // chunks (of each part), workgroups of the first level of carries
  int64_t blocks;  // workgroups that have entries
};

// Lanes: the vectors of a row, up to 32 (longer rows take several passes over the entries, side by
// side). Entries of a group, in the order of the rules:
//   - Small tensors are a chain of loads, four entries after four. 4 entries while that makes no more than two workgroups to a compute
//     unit, 8 up to three (of 16 / 8 / 4, us, skewed slices; CSF's searches for the bounds gain from short chunks, too):
//       COO, 50 000 entries, fp32, J = 32 12.4 / 11.3 / 10.9; 110 000 13.6 / 12.8 / 12.9; 220 000 (3.4 workgroups) 16.1 / 15.6 / 19.5, even
//         15.2 / 16.4 / 20.1; fp64, J = 33, 50 000 15.7 / 15.1 / 19.0; CSF, fp32, J = 8, 110 000 18.7 / 15.1 / 13.6; 400 000 19.6 / 16.8 / 16.7;
//         740 000 23.0 / 19.7 / 24.2; J = 32, 50 000 16.1 / 13.7 / 13.8; 110 000 17.6 / 16.1 / 16.4
//   - COO with two or four lanes: what these hold at a time, since a group that comes back for the rest of its lines finds them gone (four
//     arrays, loaded past the caches: 16 and 32 entries / 8 and 16, us, skewed slices and even ones):
//       J = 8, fp32, 12M entries 124 / 105, 154 / 137; 30M 277 / 225, 351 / 316; 2.5M 34.7 / 30.4, 41 / 40; J = 4, fp64, 30M 319 / 232, 400 / 323
//       J = 16, fp32, 12M 137 / 111, 196 / 167; 30M 291 / 236, 452 / 386; 2.5M 41.2 / 35.8, 49.9 / 46.9; J = 8, fp64, 30M 300 / 266; J = 3,
//       fp32, 20M 196 / 165. (CSF reads two arrays and gains more from long chunks: J = 8, fp32, 12M 113 / 125, J = 16 132 / 147.)
//   - 16, which a group's fixed work (bounds, scan, carry) is worth, while some four (CSF) or five (COO) workgroups go to a compute unit (a line
//     by measurement; by registers five of either fit, of COO in fp64 with two to 16 lanes four). Of COO with eight lanes three, with
//     16 four, then 32 (32 / 16, twelve tensors of each: eight lanes, 410 000 entries, even .97, skewed 1.05, 520 000 .93, .99; 16 lanes,
//     210 000 1.00, 1.11, 255 000 .98, 1.08, 270 000 .92, 1.03, 320 000 .91, 1.03).
//   - Beyond, as many as leave about six workgroups to each, in whole batches of the coordinates that the group's lanes hold (four
//     each), since a part of one costs as much; at most 2048 entries per workgroup
//     (measured with 512 to 4096: more entries keep fewer rows of C in cache, fewer leave more carries;
//     up to 10 % apart) and 128 per group. In multiples of 16 / in batches, J = 32, us:
//       CSF, fp32: 600 000 entries 36.3 / 32.8; 1.3M 56.6 / 47.1; 3M 77.9 / 75.3; fp64: 600 000 58.7 / 51.0; 2M 111 / 107
//       COO, fp32: 900 000 entries 33.2 / 31.3; 1.3M 45.2 / 38.4; 3M 71.3 / 70.6; fp64: 600 000 50.5 / 44.2; 2M 106 / 100
//   - 32 lanes, whose batches of 128 entries are too long (400 000 entries 65.6 in 16, 68.0): multiples of 16, up to 64 of them such that
//     three workgroups go to a compute unit (six / three, J = 33, fp64: COO 150 000 27.4 / 25.6, even 30.2 / 25.6; 300 000
//     40.9 / 38.1, 46.4 / 41.2; 500 000 50.1 / 48.3, 60.6 / 54.8; CSF 300 000 47.2 / 41.9, 55.2 / 46.1). Where four workgroups and more share the
//     columns of a chunk, up to 32 such that three go to a compute unit, or up to 64 such that three chunks do (J = 128 to 1024, 222 calls of
//     any sizes and 396 on a grid: against groups as long as six chunks to a compute unit leave, .96 of the time on average and more than 1.06 of it in 56
//     calls; with up to 64 counting all workgroups .98 and in 130).
//   - 16 lanes, whose batches are of 64 entries: groups of 48 as long as two workgroups on each compute unit hold the tensor.
//     With 64 there are hardly more workgroups than compute units, and a skewed tensor ends on one of them. (COO: even slices
//     lose some of what 64 gain, up to 5 %, skewed ones gain as much; with 32, even slices lose 10 %, fp32.) Groups of
//     16 / 32 / 48 / 64, J = 32, fp64, skewed slices, and even ones:
//       CSF, 265 000 entries  32.5 / 29.7 / 32.2 / 36.9, 35.3 / 31.8 / 29.9 / 31.3; 360 000  35.6 / 32.2 / 33.6 / 37.5, 39.1 / 34.3 / 34.5 / 34.6
//         400 000 37.1 / 35.3 / 36.7 / 37.3, 42.0 / 39.2 / 39.9 / 36.8
//       COO, 330 000 entries  28.3 / 26.7 / 28.4 / 29.5, 30.3 / 28.2 / 28.1 / 27.9; 400 000  32.0 / 31.3 / 32.6 / 31.2, 35.1 / 34.1 / 34.4 / 30.9
//       fp32, J = 64: CSF, 265 000  36.2 / 33.8 / 34.5 / 38.6, 39.8 / 35.2 / 32.7 / 33.3; COO, 330 000  32.4 / 30.7 / 32.1 / 32.8, 36.9 / 32.7 / 31.3 / 31.3
// (A workspace that holds the carries of 16 entries to a group and more, but not of fewer, gets these.)
// Parts of the J columns, each of whole lines, that XCDs of their own go through all entries for (given C and D on lines): an L2
// then holds twice, four or eight times as many rows. A gather takes as long for 64 bytes as for a line, so parts of
// half a line only lose (50M entries, J = 32, fp32: 618 -> 1010 us). The entries are read once per part, which rows that an L2
// holds anyway do not pay for, nor few entries. One part / parts, us (skewed slices, and even ones), C and D in MB:
//   COO, J = 32, fp64, 20.5 and 12.8: 200 000 entries 24.4 / 23.9, 24.2 / 23.6; 1M 68 / 60, 80 / 76; 5M 234 / 204, 335 / 313;
//     20M 692 / 569, 1261 / 1179; 5.1 and 5.1: 1M 45 / 39, 55 / 42; 20M 420 / 419, 859 / 593; 0.5 and 25.6: 2M 88 / 84, 87 / 86
//   CSF: 1M 75 / 69, 87 / 86; 20M 692 / 560, 1281 / 1177; 5.1 and 5.1: 20M 492 / 499, 885 / 642; 0.5 and 25.6: 1M 61 / 56, 58 / 63
//   J = 64, fp64 (four parts), 41 and 25.6: 300 000 62 / 52; 2M 219 / 192; 20M 1491 / 1174
//   2.6 and 0.8: 1M 28.9 / 32.6; 2M 48 / 53; 5.1 and 1.5 (J = 64): 2M 82 / 98; fewer entries than the line: up to 10 % longer
// Factors of which the 256 MB of the Infinity Cache do not hold all rows that the entries may need are not split: no L2 holds a share of their rows worth having, and a row comes from memory in
// pieces. Parts / one part, COO, even slices: J = 64, fp64, C and D 154 and 15 MB, 1.5M entries .90, 6M .91; 154 and 154 1.06, 1.06; 512 and
// 2.6 1.03, 1.05; 512 and 512 1.09, 1.09; 2048 and 2.6 1.15, 1.20; J = 128, fp64, 92 and 31 MB .87, .89; 307 and 31 .98, .98; 1024 and 5.1
// 1.13, 1.15 (skewed 1.16, 1.25; CSF 1.14, 1.42); J = 32, fp64, 77 and 77 1.05, 1.04. Of 300 000 entries, J = 64, fp64, 512 and 2.6 .86, 2048 and 2.6 .83.
// Where a part's vectors leave lanes idle (8 and 16 lanes, and whole groups of 32, have none), every workgroup issues as much for less. An eighth of
// them costs nothing, a quarter is worth it where the factors are that large in the 512 bytes of a row that unsplit workgroups go
// through at a time, or where a row is used by few entries, so that fetching it into every L2 once is what counts. Parts / one part, 1.5M entries, COO,
// skewed slices and even ones; dimensions of C and D 4000 and 4000 (4.1 MB of 512-byte rows), 9000 and 9000, 20 000 and 10 000:
//   24 of 32 lanes: J = 96, fp64 .98 .90, .91 .71, .92 .83; 192 1.15 .90, .87 .72, .85 .83; 384 1.16 .93, .85 .73, .86 .85
//   80 of 96: J = 320 1.14 .96, .91 .89, .93 .93; 640 1.05 .91, .89 .87, .88 .90
//   40 of 64: J = 160 1.20 1.07, 1.06 1.03, 1.06 1.03; 320 1.35 1.11, 1.03 .96, 1.02 .98; 640 1.36 1.15, 1.05 .98, 1.03 .99
//   24 and 80, 20 000 and 10 000, even, one part / parts, us: J = 384 999 / 866, 640 1680 / 1479
//   56 of 64: J = 448 1.02 .85 (1M); 160 of 160: J = 640 .94 .91, .90 .94, .92 .96; 64 of 64: J = 1024 .95 .83, .83 .91, .88 .96
// and of 4000 and 4000, 300 000 entries (37 to a row) and 600 000: 24 of 32, J = 192 1.02 .80, 1.18 .93; 384 .98 .73, 1.13 .84; 80 of 96, J = 320 .89
// .80, 1.05 .94; 640 .85 .75, 1.01 .86.
inline int mttkrp_parts(int64_t nnz, int64_t row_bytes, int64_t rows_c, int64_t rows_d, bool csf) {
  constexpr int64_t kFactors = 9000000, kMostFactors = 250000000;
  const int64_t c = rows_c * row_bytes, d = rows_d * row_bytes;
  if (nnz * row_bytes < 50000000 || c + d < kFactors || (csf && c < 1000000)) return 1;
  if ((std::min(rows_c, nnz) + std::min(rows_d, nnz)) * row_bytes > kMostFactors) return 1;
  const auto worth_it = [&](int parts) {
    if (row_bytes % (parts * int64_t{kLine}) != 0) return false;
    const int64_t vectors = row_bytes / parts / 16, lanes = (vectors + 31) / 32 * 32;
    return vectors == 8 || vectors == 16 || 8 * vectors >= 7 * lanes ||
           (4 * vectors >= 3 * lanes && ((rows_c + rows_d) * 512 >= kFactors || nnz <= 40 * (rows_c + rows_d)));
  };
  int parts = kXcds;
  while (parts > 1 && !worth_it(parts)) parts /= 2;
  return parts;
}
inline MttkrpPlan mttkrp_plan(int64_t nnz, int64_t J, int dtype, bool csf, int parts, bool least_carries = false) {
  MttkrpPlan P;
  P.parts = parts;
  J /= parts;  // (the rest is about one part; its workgroups are as many for each)
  P.vec = dtype == SPT_F64 ? kVec<double> : kVec<float>;
  if (J < P.vec) P.vec = 1;
  const int64_t nv = (J + P.vec - 1) / P.vec;
  P.lanes = P.vec == 1 ? 4 : nv <= 2 ? 2 : nv <= 4 ? 4 : nv <= 8 ? 8 : nv <= 16 ? 16 : 32;
  const int groups = kBlock / P.lanes;
  const int64_t tiles = P.tiles = static_cast<int>((nv + P.lanes - 1) / P.lanes);
  const int batch = P.lanes <= 16 ? std::max(4 * P.lanes, 16) : 16;
  const int64_t at_once = int64_t(256) * groups * 16 / parts;  // with 16 entries to a group, a workgroup to each compute unit
  const int64_t want = nnz * parts / (6 * 256) / groups;
  const auto workgroups = [&](int64_t epg) { return (nnz + groups * epg - 1) / (groups * epg) * tiles * parts; };
  const auto three = [&](int64_t times) { return (nnz * times / (3 * 256) / groups + 8) / 16 * 16; };
  int64_t epg = 16;
  if (P.lanes > 16) epg = std::max<int64_t>(want / 16 * 16, 16);
  else if (P.lanes == 16 && nnz > (csf ? 4 : 5) * at_once && nnz <= int64_t(2) * 256 * groups * 48) epg = 48;
  else if (nnz > (csf ? 4 : 5) * at_once) epg = std::max<int64_t>((want + batch / 2) / batch * batch, batch);
  if (!least_carries) {
    if ((csf || P.lanes > 2) && workgroups(4) <= 2 * 256) epg = 4;
    else if (workgroups(8) <= 3 * 256) epg = 8;
    else if (!csf && P.lanes <= 4) epg = 4 * P.lanes;
    else if (!csf && P.lanes <= 16 && nnz > (P.lanes == 16 ? 4 : 3) * at_once && epg == 16) epg = 32;
    else if (P.lanes > 16) epg = std::max({epg, std::min(three(tiles * parts), int64_t(tiles < 4 ? 64 : 32)), std::min(three(parts), int64_t(64))});
  }
  P.epg = static_cast<int>(std::min<int64_t>(epg, std::min(128, 2048 / groups)));
  P.chunk = P.epg * groups;
  P.n1 = (nnz + P.chunk - 1) / P.chunk;
  P.n2 = (P.n1 + kCarrySpan - 1) / kCarrySpan;
  P.blocks = workgroups(P.epg);
  return P;
}

}  // namespace spt
