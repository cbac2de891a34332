// The planner: turns a tensor list into the tables the kernels walk and lays out the workspace. Plain host C++, no HIP calls.
#pragma once

#include <vector>

#include "lopt_internal.h"

namespace lopt {

constexpr int kThinTiles = 1024;                    // short lists: row/column tiles of fewer than sixteen rows
constexpr uint64_t kShortListFloats = 48u << 20;   // what a short list's statistics pass reads of partial sums, all workgroups together

inline uint32_t pad4(uint64_t x) { return (uint32_t)((x + 3) & ~(uint64_t)3); }
inline uint64_t align64(uint64_t x) { return (x + 63) & ~(uint64_t)63; }
inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }   // a up to 2^31 - 1: a + b - 1 does not fit an int

constexpr uint64_t kFinBatch = 32;                // loads in flight per lane in the sums of the partials

// The apply kernels that take their work from the table of apply tiles (the others walk the statistics tiles).
enum class ApplyTiles { None, Strip, Narrow };   // k_apply_f16s; k_apply_fc4x

// What the planner has to know of a context.
struct PlanOptions {
  int kind = LOPT_SMALL_FC;      // lopt_kind
  int HP = 0, P = 0;             // padded MLP width; VeLO: floats per per-tensor MLP
  int lstm_hidden = 0, n_bank = 0;
  bool head_folded = false;      // VeLO: the hypernetwork head is one folded matrix (WeightsDev::head)
  ApplyTiles apply = ApplyTiles::None;
  int groups_override = 0;       // tensor groups of the two-stream pipeline (0 = choose by size)
  int n_cu = 256;
};

struct Plan {
  std::vector<lopt_tensor_desc> descs;
  std::vector<TensorDev> tensors;   // pointers filled per call
  std::vector<TileDev> tiles;
  std::vector<RcItemDev> rcitems;     // blocks of k_rc_update (none on short lists)
  std::vector<RcItemDev> rcshort;     // short lists: the same blocks, workgroups of the statistics pass (short_rc_block)
  std::vector<TileDev> rctiles;       // short lists: tiles of the row/column sums
  bool short_list = false;
  int groups = 1;                     // tensor groups of the two-stream pipeline
  int keep = 0, keep_off = 0;         // see choose_loads
  bool keep_line = false;
  bool backwards = false;
  bool strip_ordinary = false, off_grid_nt = false;   // see choose_loads
  bool fold_finalize = false;         // k_finalize is not launched: the strip kernel's workgroups form their tensor's scales, the
                                      // LSTM's those of all (few) tensors
  std::vector<ApplyTileDev> atiles;   // apply tiles (none for ApplyTiles::None)
  std::vector<int> atile0;            // first apply tile of every tensor
  uint64_t total_elems = 0;
  int64_t max_rows = 0;               // of any tensor
  std::vector<size_t> state_bytes;
  uint64_t oLstmU = 0, oHNew = 0;   // VeLO scratch (floats)
  uint64_t oHbarPart = 0, oBeff = 0; // VeLO cross-tensor term: slice sums of h, gate bias with the term added
  uint64_t oLstmZ = 0;               // VeLO, lists of few tensors (lstm_ahead): h W_h of the step before, in tile order (0: not used)
  uint64_t oAlpha = 0, oTheta = 0;   // VeLO, long lists: bank coefficients [T][K] and per-tensor MLPs [T][P]
  bool head_batched = false;
  uint64_t oCounters = 0;           // kMaxGroups ints: tile counters of the apply kernel
  uint64_t ws_floats = 0;
  const std::vector<RcItemDev>& rc_blocks() const { return short_list ? rcshort : rcitems; }
};

// Number of tensor groups of the two-stream pipeline for a list of `total` elements (0 override = by size). A group more costs
// two launches, two waits across streams and one more drain of both kernels, about 40 us. Measured, ms a step with
// G = 1 / 2 / 3 / 4 / 5 / 8: 20 M elements 0.370 / 0.389 / 0.410 / 0.439 / 0.458 / 0.583; 40 M 0.752 / 0.766 / 0.807 / 0.851 /
// 0.853 / 1.020; 87 M 1.57 / 1.53 / 1.54 / 1.55 / 1.64 / 1.78; 150 M 2.78 / 2.70 / 2.70 / 2.72 / 2.73 / 2.86; 355 M 6.36 / 6.14 /
// 6.07 / 6.02 / 6.02 / 6.08. With G = 4 / 6 / 8 / 16: 435 M 7.20 / 7.19 / 7.28 / -; 536 M 8.90 / 8.87 / 8.85 / -; 738 M 12.27 / 12.21 /
// 12.20 / 12.49; 1034 M 17.29 / 17.20 / 17.18 / 17.31; 1346 M 22.32 / 22.20 / 22.13 / 22.13.
inline int planned_groups(int override_g, uint64_t total, size_t n) {
  int G = override_g;
  if (!G) G = total >= (512u << 20) ? 8 : total >= (256u << 20) ? 4 : total >= (128u << 20) ? 3 : total >= (64u << 20) ? 2 : 1;
  if ((size_t)G > n) G = (int)n;
  return G < 1 ? 1 : G;
}

// Contiguous tensor ranges [bound[g], bound[g+1]) of about equal element count.
inline void group_bounds(const lopt_tensor_desc* d, size_t n, int G, uint64_t total, int* bound) {
  uint64_t cum = 0;
  int g = 1;
  bound[0] = 0;
  for (size_t i = 0; i < n && g < G; ++i) {
    cum += (uint64_t)d[i].rows * (uint64_t)d[i].cols;
    if (cum * (uint64_t)G >= total * (uint64_t)g && (int)i + 1 > bound[g - 1]) bound[g++] = (int)i + 1;
  }
  while (g <= G) bound[g++] = (int)n;
}

// Short lists: no launch of its own for the means of the rows and columns (k_rc_update: 4.5 to 6 us, a chain of load latencies).
// Every workgroup of the statistics pass forms the ones of its own rows and columns from the partial sums, which the
// row/column pass leaves per 64 or 128 rows for that purpose. us a step with that launch and without: 0.08 M elements (toy list) 29.6 /
// 26.9, 1000x1000 45.7 / 43.8 (VeLO 57.7 / 55.0), 66 tensors of 2.4 M under VeLO 69.1 / 66.7, 2000x2000 107.8 / 104.4, ten layers of
// 1024x1024 at width 16 191.8 / 188.8, nine of 2731x2731 under VeLO 896 / 882; no difference at 14 M elements (width 32), and 495.5 /
// 500 for one 5000x5000 matrix, whose tiles read 63 M words of partial sums again: the line lies between the last two. (One
// 6000x5000, 89 M words, with that launch and without, width 16 546 / 552, VeLO 428 / 428; eight of 6000x500, 69 M, 447 / 452, 342 / 348;
// 2x4096x4096, 34 M, 602 / 598, 427 / 431.) A tile of the row/column sums is a workgroup of sixteen wavefronts, of which most idle
// where it has fewer than sixteen rows; the chip holds 512 of these workgroups, and from a third round on they cost more than the
// launch: vectors of 768 elements, VeLO / width 32, 340 of them (1020 such tiles) 62.7 / 61.7 and 53.7 / 53.6, 400 of them 71.3 / 72.1
// and 59.8 / 61.6, 600 87.9 / 91.1 and 78.6 / 83.1; but 1500 of 64x64 256 / 250. Short lists
// are never cut into tensor groups: the statistics kernel that forms the means does not fit beside the apply kernel, and groups
// cost such lists more than they hide in either form (four tensors of 4096x2560 in two groups, that launch kept / without it / one
// group: 749 / 774 / 738; under VeLO 641 / 579 / 549).
inline bool is_short_list(size_t n, const lopt_tensor_desc* d, uint64_t total, int shrink, bool velo) {
  if (total >= (64u << 20) || n > 4096) return false;   // 4096: the copies of r_k and c_k are no large part of a workspace
  uint64_t floats = 0, thin = 0;
  for (size_t i = 0; i < n; ++i) {
    if (d[i].rows > 96 * kRowUnit || d[i].cols > 96 * kTileCols) return false;
    const uint64_t nrc = (uint64_t)ceil_div(d[i].rows, short_rows((int)d[i].rows, velo)), nct = (uint64_t)ceil_div(d[i].cols, kTileCols);
    const uint64_t tr = kRowUnit / shrink, tiles = (uint64_t)ceil_div(d[i].rows, tr) * nct;
    floats += tiles * (2 * nrc * (uint64_t)(d[i].cols < kTileCols ? d[i].cols : kTileCols) + nct * tr);
    if (d[i].rows < 16) thin += nct;
    if (floats > kShortListFloats || thin > kThinTiles) return false;
  }
  return true;
}

// How the statistics pass reads its tiles. What it reads with ordinary instead of nontemporal loads is still in the 256 MB
// Infinity Cache when the apply pass reads it again, as far as it fits: 10 M elements of 24 bytes. Going from the last tile to
// the first, it ends where the apply pass begins. us a step, two contexts in turn:
//   short lists below 15.5 M elements: everything on the 128-byte grid ordinary (row/column sums too), forwards. VeLO 2.4 M elements
//     62.6 -> 58.3, 4.2 M 84.6 -> 77.1, 8.4 M 132.2 -> 119.5; width 16 9.5 M 189.8 -> 186.7; width 32 12.6 M 247 -> 241
//   short lists from there on: backwards, the first 10 M elements' tiles ordinary, for the narrow widths none, whose apply pass is
//     longer than the cache is of use. Everything ordinary and forwards (backwards from 40 M) / this way, VeLO 17 M of 1024 columns
//     224.7 / 219.3, 34 M 458 / 433, 34 M of 4096 448 / 428, 38 M of 2048 514 / 482; width 32 34 M 601 / 582, 42 M 737 / 721; width 16
//     (598 nontemporal throughout) 619 / 597, 42 M of 4096 749 / 724. At 15 M VeLO 203.7 / 205.5, width 32 302 / 300, width 16 298 / 299.7, at
//     14 M of 3072 columns VeLO 182.6 / 185.5
//   rows off the 16-byte grid: ordinary (8.3 M elements width 32 209 us nontemporal 220; VeLO 8 M 143 / 161), for VeLO from 13 M on
//     nontemporal (13.4 M 229 / 231, 16.4 M 298 / 285, 20 M 360 / 336), again but for the first 10 M. Backwards helps here
//     from 11 M on, which decides for lists with most of their elements off the grid. 1531 columns, forwards / backwards, 9 M VeLO 137.5 /
//     138.3, 12 M 190 / 183, width 32 and 16 the same, 14 M VeLO 221 / 208, width 32 298 / 299.5, width 16 290 / 278, 21 M VeLO 363 / 330, width 32
//     472 / 455, width 16 435 / 417
//   rows on the 16-byte but off the 128-byte grid: in short lists as rows off the 16-byte grid, for the other widths between 1.5 M and 13 M
//     elements. Nontemporal / so, VeLO 1 M elements of 1000 columns 38.5 / 35.3, 4 M of 1000 75.3 / 69.5, 9 M of 1500 150.8 / 147.8, 17 M of
//     2052 270 / 268, 32 M of 2828 500 / 491; width 32 1.1 M of 516 41.2 / 42.6, 1.4 M of 600 43 / 43, 2.2 M of 740 69.8 / 66.5, 4 M 100.4 /
//     96.6, 9 M 194 / 188.5, 17 M 351 / 357, 32 M 637 / 645; width 16 1.4 M 49.1 / 47.8, 4 M 92.6 / 90.1. Long lists: one 8004x8004 932 / 951
//     and 1195 / 1219
//   rows off the 16-byte grid of long lists, ordinary / nontemporal: VeLO 72 M of 6001 columns 1042 / 1006, 84 M of 4099 1197 / 1166; width
//     32 1375 / 1404, 1611 / 1652
//   long lists under VeLO: from the last tile to the first, nontemporal but for the first 10 M elements' tiles: ViT-B/16 shapes
//     1158 -> 1150 (6.5 M 1153, 16 M 1151.5; everything 1181), Llama-1.3B shapes 17310 -> 17283
//   long lists of small_fc_lopt: nontemporal (ViT-B/16 shapes 313 us the pass, 352 with ordinary loads).
inline void choose_loads(const PlanOptions& o, uint64_t total, Plan* pl) {
  constexpr uint64_t kCached = 10u << 20;
  int cached = (int)pl->tiles.size();   // tiles of the first kCached elements
  uint64_t seen = 0, off_grid = 0, off_line = 0;
  for (const TensorDev& T : pl->tensors) {
    off_grid += T.vec == 0 ? (uint64_t)T.m * (uint64_t)T.n : 0;
    off_line += T.vec != 2 ? (uint64_t)T.m * (uint64_t)T.n : 0;
  }
  for (const TensorDev& T : pl->tensors) {
    const uint64_t N = (uint64_t)T.m * (uint64_t)T.n;
    if (seen + N > kCached) {
      cached = T.tile0 + (int)((double)(kCached - seen) / (double)N * (double)((uint64_t)T.nrt * (uint64_t)T.nct));
      break;
    }
    seen += N;
  }
  const int all = 0x7fffffff;
  const bool velo = o.kind == LOPT_VELO;
  const bool small = pl->short_list && total < (2 * off_grid > total ? 11u << 20 : 31u << 19), narrow = o.apply == ApplyTiles::Narrow;
  pl->backwards = pl->short_list ? !small : velo;
  pl->keep = small ? all : velo || (pl->short_list && !narrow) ? cached : 0;
  pl->keep_line = pl->short_list && (velo || (total >= (3u << 19) && total < (13u << 20)));
  pl->keep_off = velo && (!pl->short_list || total >= (13u << 20)) ? cached : all;
  // The apply pass. Width 32 reads 128 bytes of a row at a time; off the 128-byte grid these share their lines with the neighbours, which
  // nontemporal loads fetch again: ordinary ones, except between 7 M and 13 M elements (M: 2^20). There the next step's statistics
  // pass still finds in the 256 MB Infinity Cache what this pass has stored, as long as this pass's loads have not taken the room
  // (nontemporal / ordinary, this pass and the statistics pass: 3701x3701, 13.1 M, 188 / 180 and 54 / 64 us; six of 1500x1500, 12.9 M, 186 /
  // 181 and 57 / 65). Below, both fit; above, neither does (four of 2004x2004, 15.3 M, 258 / 209 and 64 / 65). us a step, nontemporal /
  // ordinary, one to thirteen matrices of so many columns: below, 3.8 M of 1000 101 / 96.5, 4.3 M of 1500 114 / 105.5, 4.8 M of 1301 130.6 /
  // 124.5, 5.7 M of 2001 149.6 / 146.7, 6.4 M of 1501 157 / 157; between, 6.7 M of 1000 162 / 163.5, 7.6 M 170.5 / 173, 8.6 M of 1500 and 1501
  // 193 / 195 and 194.6 / 196, 8.9 M of 1531 200 / 200, 9.5 M of 2001 217.7 / 222, 10.3 M of 1801 238.6 / 245, 10.7 M of 1501 237.5 / 240, 11.4 M
  // of 1000 249 / 259.5, 11.5 M of 2004 and 6001 252 / 262 and 254 / 254, 12.6 M of 2201 287 / 301, 12.9 M of 1301 296 / 295; above, 13.2 M of
  // 2300 294 / 291 (but 13.4 M of 2801 295 / 311), 14.3 M of 1000 311 / 310, 15.3 M of 2001 and 2004 327.5 / 330 and 340 / 320.5, 17.2 M of 1501
  // 376 / 369.5, 24 M of 2451 499 / 486, 44 M of 3301 1004 / 823, 108 M of 6001 2554 / 1989, 128 M of 8004 2842 / 2270. On the grid it is the cache
  // alone that decides: 1.6 M of 640 46.1 / 45.5, 2.4 M of 768 67.8 / 65.5, 5.3 M of 1152 122 / 120, 6.6 M of 1280 143 / 148, 17 M of 2048 306 /
  // 322, ViT-B/16 shapes 1464 / 1482. (All these rules count a list's elements of every kind, and a list is what its larger part is; they were
  // measured on lists of one kind.)
  // Lists that fold the finalize read nontemporally, the shorter of them either way to 5 %: 0.08 M elements in three tensors 17.0 / 16.6,
  // two of 300x300 19.3 / 19.9, 512x512 20.3 / 21.3, 777x1200 32.9 / 34.6, 901x901 33.6 / 34.0, 1000x1000 34.6 / 35.6, 1100x1024 40.1 / 38.4,
  // 1200x1200 43.6 / 44.6.
  pl->strip_ordinary = !pl->fold_finalize && (2 * off_line > total ? total < (7u << 20) || total >= (13u << 20) : total < (11u << 19));
  // VeLO and the narrow widths: rows off the 16-byte grid, ordinary / nontemporal, VeLO 4.8 M elements of 1101 columns 81.5 / 87, 6 M of 1225
  // 101 / 100, 9 M 148.5 / 138, 12 M 189 / 174, 16 M 252 / 238, 20 M 303 / 296, 24 M 357 / 360, 54 M 779 / 821; width 16 4 M 91 / 100, 6 M
  // 136 / 144, 7.3 M 164.5 / 164, 9 M 195 / 192, 16 M 333 / 321, 20 M 396 / 403. (Rows on the 16-byte but off the 128-byte grid: VeLO 9 M
  // 150.6 / 150.3, 17 M 269 / 285.)
  pl->off_grid_nt = total >= (velo ? 6u : 7u) << 20 && total < (velo ? 21u : 18u) << 20;
}

// Lay out tiles, row/column blocks and workspace regions for a tensor list.
// allow_short: see the end.
inline void build_plan(const PlanOptions& o, size_t n, const lopt_tensor_desc* d, Plan* pl, bool allow_short = true) {
  pl->descs.assign(d, d + n);
  pl->tensors.assign(n, TensorDev{});
  pl->tiles.clear();
  pl->rcitems.clear();
  pl->rcshort.clear();
  pl->rctiles.clear();
  pl->atiles.clear();
  pl->atile0.assign(n, 0);
  pl->total_elems = 0;
  pl->max_rows = 0;
  pl->state_bytes.assign(n, 0);
  const bool velo = o.kind == LOPT_VELO;
  const int HP = o.HP;
  const uint64_t prep_floats = (uint64_t)(LOPT_D_VELO + 1) * HP + (uint64_t)HP * HP + HP + 2 * HP + 2;
  uint64_t off = 0;
  auto take = [&](uint64_t nfloats) { uint64_t at = off; off = align64(off + nfloats); return at; };
  pl->oCounters = take(kMaxGroups);
  if (velo) {
    pl->oLstmU = take((uint64_t)n * kLstmInPad);
    pl->oHNew = take((uint64_t)n * o.lstm_hidden);
    pl->oHbarPart = take((uint64_t)kMixSlices * o.lstm_hidden);
    pl->oBeff = take((uint64_t)kMixJSplit * 4ull * o.lstm_hidden);
    pl->head_batched = n >= (size_t)kHeadBatchMin;
    if (pl->head_batched) {
      if (!o.head_folded) pl->oAlpha = take((uint64_t)n * o.n_bank);
      pl->oTheta = take((uint64_t)n * (uint64_t)(o.head_folded ? head_ld(o.P) : o.P));
    }
  }
  uint64_t total = 0;
  for (size_t i = 0; i < n; ++i) total += (uint64_t)d[i].rows * (uint64_t)d[i].cols;
  // Small parameter sets: with the standard 64-row tiles there may be fewer tiles than the chip has workgroup
  // slots (256 CUs x 2..8), so the tile height is halved until the list yields about 2048 tiles or reaches 8 rows.
  uint64_t std_tiles = 0;
  for (size_t i = 0; i < n; ++i)
    std_tiles += (uint64_t)((d[i].rows + kRowUnit - 1) / kRowUnit) * (uint64_t)((d[i].cols + kTileCols - 1) / kTileCols);
  int shrink = 1;
  while (shrink < 8 && std_tiles * shrink < 2048) shrink *= 2;
  pl->short_list = allow_short && is_short_list(n, d, total, shrink, velo);
  // Apply tiles get shorter towards the end of every tensor group of the pipeline (a single group if it is off, as it is for
  // every kernel but the strip one): the apply kernel hands tiles out in table order, so the last tiles of a launch decide how long the chip idles
  // while the final workgroups finish (a 128-row tile is about 90 us of work, a 32-row tile a quarter of that).
  pl->groups = pl->short_list || !(o.apply == ApplyTiles::Strip || (velo && o.groups_override)) ? 1 : planned_groups(o.groups_override, total, n);
  int gbound[kMaxGroups + 1];
  group_bounds(d, n, pl->groups, total, gbound);
  std::vector<uint64_t> gtotal(pl->groups, 0), gbefore(n, 0);
  for (int g = 0; g < pl->groups; ++g)
    for (int i = gbound[g]; i < gbound[g + 1]; ++i) {
      gbefore[i] = gtotal[g];
      gtotal[g] += (uint64_t)d[i].rows * (uint64_t)d[i].cols;
    }
  std::vector<int> group_of(n, 0);
  for (int g = 0; g < pl->groups; ++g)
    for (int i = gbound[g]; i < gbound[g + 1]; ++i) group_of[i] = g;
  // Short lists: the smallest even apply-tile height at which every CU gets at most two tiles, if that is at most 32 rows: the
  // launch is then one round of equal tiles (a 1000x1000 layer: 504 tiles of 16 rows, where the graded heights below gave 650
  // tiles and a second, nearly empty round). The strip kernel has two workgroups per CU. The narrow one has three or four, and
  // as many tiles are its second choice (1700x1400, width 4: 63.6 us a step with graded heights, 59.5 this way; 1000x1000: 39.6
  // with two tiles per CU, 44.2 with four); its wavefronts take narrow_trip_rows at a time, two to a column segment, and
  // a tile is at least that high (toy list of three tensors, width 4: 25.2 us with tiles of two rows, 23.5 with eight).
  const bool narrow = o.apply == ApplyTiles::Narrow;
  int ar_short = 0;
  for (int per_cu : {2, narrow ? narrow_waves_per_simd(HP) : 2})
    for (int ar : {2, 4, 6, 8, 12, 16, 20, 24, 32}) {
      if (ar_short || o.apply == ApplyTiles::None || (narrow && ar < 2 * narrow_trip_rows(HP))) continue;
      const uint64_t most = (uint64_t)per_cu * o.n_cu;
      uint64_t tiles = 0;
      for (size_t i = 0; i < n && tiles <= most; ++i)
        tiles += (uint64_t)((d[i].rows + ar - 1) / ar) * (uint64_t)((d[i].cols + kApplyCols - 1) / kApplyCols);
      if (tiles <= most) ar_short = ar;
    }
  for (size_t i = 0; i < n; ++i) {
    TensorDev& T = pl->tensors[i];
    const int m = (int)d[i].rows, nn = (int)d[i].cols;
    const uint64_t N = (uint64_t)m * nn;
    T.m = m; T.n = nn;
    T.padN = pad4(N); T.padm = pad4(m); T.padn = pad4(nn);
    T.padH = velo ? pad4(o.lstm_hidden) : 0;
    T.ndim = d[i].ndim;
    T.vec = nn % 32 == 0 ? 2 : nn % 4 == 0 ? 1 : 0;
    const int units = ceil_div(m, kRowUnit);
    const int q = ceil_div(units, kMaxRowTiles);
    T.TR = kRowUnit * (q < 1 ? 1 : q) / shrink;   // a multiple of 8: every wavefront of a tile owns whole rows
    // ... but never more than kMaxRowTiles row tiles per tensor (the second-stage reductions loop over them; a small
    // list, whose tiles were made shorter above, may have `shrink` times as many) ...
    const int max_rt = kMaxRowTiles * shrink;
    const int min_tr = (ceil_div(m, max_rt) + 7) & ~7;
    if (T.TR < min_tr) T.TR = min_tr;
    // ... unless that makes a tile taller than kMaxTileRows: a lane sums up to kMaxTileRows values in fp32 (a quarter of the
    // tile's rows at four values each), and such a partial
    // sum must stay at about a thousand terms. Tensors of more than kMaxRowTiles * kMaxTileRows rows get more row tiles instead.
    if (T.TR > kMaxTileRows) T.TR = kMaxTileRows;
    T.nrt = ceil_div(m, T.TR);
    T.nct = ceil_div(nn, kTileCols);
    T.tile0 = (int)pl->tiles.size();
    // Table order: workgroups reach the eight dies in turn, so eight tile rows at a time, column by column, put the tiles of a row
    // on one die, whose L2 then holds the lines that neighbours share (rows off the 128-byte grid) and writes them back whole.
    // VeLO, us a step, before and now: four 4096 x 4100 1026 -> 976, 20 of 1000 x 1000 326 -> 317, 54 M elements of 2731 columns
    // 871 -> 860; rows on the grid: four 4096 x 4096 877 -> 868, ViT-B/16 shapes 1164 -> 1157, Llama-1.3B shapes 17410 -> 17320, 20 of
    // 1024 x 1024 292.3 -> 293.5. Sixteen tile rows the same, four up to 3 % slower.
    constexpr int kDies = 8;
    for (int t0 = 0; t0 < T.nrt; t0 += kDies) {
      const int t1 = t0 + kDies <= T.nrt ? t0 + kDies : T.nrt;
      for (int tj = 0; tj < T.nct; ++tj)
        for (int ti = t0; ti < t1; ++ti) pl->tiles.push_back(TileDev{(int)i, ti, tj, 0});
    }
    const int nrblk = ceil_div(m, kBlock), ncblk = ceil_div(nn, kBlock);
    T.nrpart = pl->short_list ? 2 * nrblk : nrblk;   // short lists: two floats make a double (short_rc_block)
    T.ncpart = pl->short_list ? 2 * ncblk : ncblk;
    T.rc0 = (int)pl->rcitems.size();
    const int nrc = ceil_div(m, short_rows(m, velo));
    if (pl->short_list) {
      for (int ti = 0; ti < nrc; ++ti)
        for (int tj = 0; tj < T.nct; ++tj) pl->rctiles.push_back(TileDev{(int)i, ti, tj, 0});
    }
    std::vector<RcItemDev>& rc = pl->short_list ? pl->rcshort : pl->rcitems;
    for (int b = 0; b < nrblk; ++b) rc.push_back(RcItemDev{(int)i, 0, b, 0});
    for (int b = 0; b < ncblk; ++b) rc.push_back(RcItemDev{(int)i, 1, b, 0});
    // apply tiles, for the kernels that read them: up to kApplyRows x kApplyCols, shorter for small lists like the statistics tiles
    pl->atile0[i] = (int)pl->atiles.size();
    pl->total_elems += N;
    if (m > pl->max_rows) pl->max_rows = m;
    for (int ar0 = 0; o.apply != ApplyTiles::None && ar0 < m;) {
      // position of this row block inside its group: full height for the first 70 %, half to 88 %, a quarter after
      const uint64_t pos = gbefore[i] + (uint64_t)ar0 * (uint64_t)nn, gt = gtotal[group_of[i]];
      int AR = kApplyRows / shrink;
      if (pos * 100 >= gt * 88) AR /= 4;
      else if (pos * 100 >= gt * 70) AR /= 2;
      if (AR < 8) AR = 8;
      if (ar_short) AR = ar_short;
      const int rows = m - ar0 < AR ? m - ar0 : AR;
      for (int64_t ac0 = 0; ac0 < nn; ac0 += kApplyCols) pl->atiles.push_back(ApplyTileDev{(int)i, ar0, (int)ac0, rows});
      ar0 += rows;
    }
    T.oRowPart = take((uint64_t)T.nct * m);
    T.oColPart = take((uint64_t)(pl->short_list ? 2 * nrc : T.nrt) * nn);   // short lists: in double
    T.oRR = take((pl->short_list ? 6ull : 3ull) * T.padm);
    T.oRC = take((pl->short_list ? 6ull : 3ull) * T.padn);
    T.oRcPart = take((uint64_t)(T.nrpart + T.ncpart) * kRcStride);
    T.oStatPart = take((uint64_t)T.nrt * T.nct * kStatStride);
    T.oStats = take(kStatsPerTensor);
    T.oScale = take(kStatsPerTensor);
    T.oPrep = take(prep_floats);
    pl->state_bytes[i] = sizeof(float) * (4ull * T.padN + 3ull * T.padm + 3ull * T.padn + 2ull * T.padH);
  }
  // A launch fewer where every workgroup has one tile and all of them together read at most 64 MB of partials for it. us a step
  // without and with: toy list of three tensors 26.7 / 22.9, 1000x1000 (22 MB) 42.0 / 39.8, 1200x1200 (35 MB) 50.9 / 48.3, 1400x1400 (two rounds of
  // tiles, 70 MB) 61.1 / 60.2, seven layers of 700x700 (several rounds, 46 MB) 86.6 / 93.3, 1700x1700 87.4 / 107.5.
  uint64_t again = 0;
  for (size_t i = 0; i < n && pl->short_list && o.apply == ApplyTiles::Strip; ++i) {
    const TensorDev& T = pl->tensors[i];
    const uint64_t at = (i + 1 < n ? pl->atile0[i + 1] : pl->atiles.size()) - pl->atile0[i];
    again += at * ((uint64_t)T.nrt * T.nct * kStatStride + (uint64_t)(T.nrpart + T.ncpart) * kRcStride);
  }
  pl->fold_finalize = pl->short_list && o.apply == ApplyTiles::Strip && pl->atiles.size() <= 2u * (unsigned)o.n_cu && again <= (16u << 20);
  // h W_h depends on nothing this step computes. Short lists of tensors form it beside the statistics (lstm_ahead); longer ones and
  // workspaces that come near the fixed scratch of lopt_step_static go without the room for it
  pl->oLstmZ = 0;
  if (velo && lstm_ahead(n, o.lstm_hidden) && off <= (48u << 20) / sizeof(float))
    pl->oLstmZ = take((uint64_t)n * 32 * ceil_div(o.lstm_hidden, 8));
  // VeLO: every workgroup of the LSTM launch forms all tensors' scales and inputs, where that is at most two batches of loads for
  // each of its eight half wavefronts, which share the tensors. us a step without and with: four tensors of 0.012 M elements (one batch)
  // 31.2 / 29.2, 1000x1000 (two) 47.5 / 46.1, two of 900x900 (four) 50.7 / 50.7, six of 0.33 M (four) 33.7 / 34.2.
  if (pl->oLstmZ && pl->short_list && n <= (size_t)kFinTensorsMax) {
    const uint64_t share = n <= 1 ? 8 : n <= 2 ? 4 : n <= 4 ? 2 : 1;   // half wavefronts to a tensor
    pl->fold_finalize = true;
    for (const TensorDev& T : pl->tensors) pl->fold_finalize = pl->fold_finalize && (uint64_t)T.nrt * T.nct <= 2 * kFinBatch * share;
  }
  pl->ws_floats = off;
  choose_loads(o, total, pl);
  // A short list's copies of r_k and c_k must not take it over the fixed scratch of lopt_step_static: workspaces that come near it
  // (vectors of millions of elements in all) keep the form without them.
  if (pl->short_list && off > (48u << 20) / sizeof(float)) build_plan(o, n, d, pl, false);
}

inline bool same_descs(const Plan& pl, size_t n, const lopt_tensor_desc* d) {
  if (pl.descs.size() != n) return false;
  for (size_t i = 0; i < n; ++i)
    if (pl.descs[i].ndim != d[i].ndim || pl.descs[i].rows != d[i].rows || pl.descs[i].cols != d[i].cols)
      return false;
  return true;
}

inline size_t table_bytes(const Plan& pl) {
  return align64(pl.tensors.size() * sizeof(TensorDev)) + align64(pl.tiles.size() * sizeof(TileDev)) +
         align64(pl.rc_blocks().size() * sizeof(RcItemDev)) + align64(pl.rctiles.size() * sizeof(TileDev)) +
         align64(pl.atiles.size() * sizeof(ApplyTileDev));
}

}  // namespace lopt
