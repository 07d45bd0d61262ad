// Work decomposition of stage 3 (paper Sec. 3.2 Eq. 3-4) for launches whose query tiles do not fill
// the compute units evenly.
//
// A compute unit runs whole 256-row query tiles, two at a time, and one alone at 0.8 of the rate of two, so
// a launch of T tiles on C units takes ceil(T / C) tile times: 400 tiles on 256 units cost as much as
// 512.  The R = T mod C tiles in excess of a multiple of C (the partial last tiles of the heads first,
// then full tiles from the end) are therefore not run whole.  Their work - R tiles x the key tiles of
// their heads, numbered as one line of "units" of (256 queries x 64 keys) - is cut into S equal
// shares, one per compute unit, whatever R is.  A share is one workgroup - equal work
// is what the hardware's dispatch of workgroups to free slots balances - and where it crosses from one
// query tile into the next it is two (or more) segments that the workgroup runs one after the other.
// A segment sees its key range as the whole key sequence and leaves un-normalised fp32 sums (and
// their softmax shift) in a slot of scratch memory; a second kernel adds the segments of a tile in
// key order.  The shares are dispatched behind the whole tiles (workgroups go to the compute units
// one each before any gets a second one, and then to whichever slot frees up): a launch with less
// than one whole tile per compute unit then has a whole tile and shares side by side on every
// unit, and a long launch ends on the small work items.
//
// The functions below are the single statement of that numbering; the host (plan, scratch size,
// tests) and the kernels (which segment am I, which slots belong to my tile) both call them.
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>

#include "../../include/httm.h"

namespace httm {

constexpr int kAttnTileRows = 256;        // query rows of a tile of the kernel instance that splits
constexpr int kWideRows = 512;            // the same of the kernel with 128 rows a wave
constexpr int kAttnKeyTile = 64;          // keys per unit
constexpr int kAttnSplitGroups = 64;      // runs of tiles of one head the excess set may consist of
constexpr int kAttnMaxShares = 512;
constexpr int kAttnMaxExcess = 255;
constexpr int kAttnMinShareUnits = 8;     // a share is at least 512 keys long (pipeline fill and drain)
constexpr int kAttnLongShareUnits = 240;  // shares of more than 15360 keys are cut in two
constexpr int kAttnMaxPiecesPerTile = 32; // bounds what one workgroup of the second kernel has to add up
constexpr int64_t kAttnSlotWords = (int64_t)kAttnTileRows * (64 + 2);   // 64 sums of weight * v, sum of weights, shift

// Scratch that covers any launch in 256-row tiles: a slot per (share, tile) pair that can occur.  A segment of a 512-row tile
// has two slots, so a plan of those may need 1020; one that needs more than these 767 is dropped (choose_wide_tiles()) for whole
// rounds or 256-row tiles: with 16 equal heads those of 20 800 to 23 300, 29 000 to 30 900 and 37 200 to 38 900 rows run in the
// latter, a quarter of the long launches.  What that leaves, us, so / with room for 1020 slots (17 MB more in every workspace
// and on every GPU): 16 heads of 21000 x 21000 1356 / 1317, 29142 x 29142 2582 / 2497, 30166 x 30166 2737 / 2678, 22000 x 60000 3976 / 3861.
constexpr int64_t kAttnScratchBytes = (int64_t)(kAttnMaxShares + kAttnMaxExcess) * kAttnSlotWords * 4;

// `count` consecutive tiles of one head in the excess set: tile e of the set (tile0 <= e < tile0 +
// count) covers the query rows from q0 + (e - tile0) * tile_rows and the units [cum + (e - tile0) * kt,
// ... + kt), kt = units of one tile of the head: its key tiles, fewer where a unit is more of them (see narrow_tiles).
struct SplitGroup {
  int32_t head, q0, tile0, cum, kt;
};

struct SplitPlan {
  int32_t n_tiles;      // tiles that run in pieces (0: none, every tile runs whole)
  int32_t n_groups;
  int32_t units;        // all units of those tiles
  int32_t share_units;  // units per share (the last share may be shorter)
  int32_t shares;
  int32_t span;         // most tiles a share touches
  int32_t slots;        // 256-row tiles: shares + n_tiles - 1 (a few slots stay unused: a share and a tile that end together)
  int32_t tile_rows;    // 256 or 512
  // 512-row tiles: the first narrow_tiles ones are partial ones of at most 256 rows, whose segments have one slot of scratch
  // instead of two and whose units are 1.6 key tiles: alone on a CU they take 0.62 of the time.  (With units of two the shares
  // that hold them end last: 20 heads of 8942 x 50208 in 1.06 of the time of 256-row tiles.)
  int32_t narrow_tiles;
  int32_t slot_shift;   // what makes the slots of the other ones follow those
  SplitGroup grp[kAttnSplitGroups];
};

struct SplitSegment {
  int32_t head, q0;     // the query tile
  int32_t t0, t1;       // its key tiles [t0, t1) of the head's sequence; t0 >= t1: nothing to do
  int32_t slot;         // where its partial results go
};

// (Device code asks for all groups at once, a lane each: one after the other they are 20 dependent reads of cold
// argument memory.  The plan has at least one group there.)
__host__ __device__ inline int split_group_of_tile(const SplitPlan& p, int e) {
#ifdef __HIP_DEVICE_COMPILE__
  static_assert(kAttnSplitGroups <= 64, "a lane per group");
  const int g = threadIdx.x & 63;
  return __popcll(__builtin_amdgcn_ballot_w64(g < p.n_groups && p.grp[g].tile0 <= e)) - 1;
#else
  int g = 0;
  while (g + 1 < p.n_groups && p.grp[g + 1].tile0 <= e) ++g;
  return g;
#endif
}

// The tile of the excess set that unit `unit` (0 <= unit < p.units) belongs to.
__host__ __device__ inline int split_tile_of_unit(const SplitPlan& p, int unit) {
#ifdef __HIP_DEVICE_COMPILE__
  const int l = threadIdx.x & 63;
  const int g = __popcll(__builtin_amdgcn_ballot_w64(l < p.n_groups && p.grp[l].cum <= unit)) - 1;
#else
  int g = 0;
  while (g + 1 < p.n_groups && p.grp[g + 1].cum <= unit) ++g;
#endif
  return p.grp[g].tile0 + (unit - p.grp[g].cum) / p.grp[g].kt;
}

// Slot of the partial results of share s in tile e: consecutive segments differ in s, in e or in
// both, both never decrease, so s + e is unique; the largest is shares + n_tiles - 2.  512-row tiles (WIDE) have two slots, the
// second one for their rows from 256 on, but for the partial tiles that need one only: those come first.
template <bool WIDE>
__host__ __device__ inline int slots_per_segment(const SplitPlan& p, int tile) { return WIDE && tile >= p.narrow_tiles ? 2 : 1; }
// Key tile at which unit u of a tile begins.
template <bool WIDE>
__host__ __device__ inline int first_key_tile(const SplitPlan& p, int tile, int u) { return WIDE && tile < p.narrow_tiles ? u * 8 / 5 : u; }
template <bool WIDE>
__host__ __device__ inline int split_slot(const SplitPlan& p, int share, int tile) {
  return slots_per_segment<WIDE>(p, tile) == 1 ? share + tile : 2 * (share + tile) - p.slot_shift;
}

// Share s covers the units [s * share_units, (s + 1) * share_units) (the last one up to p.units): the
// tiles first .. first + count - 1 of the excess set.
__host__ __device__ inline void split_share_tiles(const SplitPlan& p, int share, int* first, int* count) {
  const int u0 = share * p.share_units;
  const int u1 = u0 + p.share_units < p.units ? u0 + p.share_units : p.units;
  *first = split_tile_of_unit(p, u0);
  *count = split_tile_of_unit(p, u1 - 1) - *first + 1;
}

// The part of share s that lies in tile e (one of split_share_tiles).
template <bool WIDE>
__host__ __device__ inline SplitSegment split_segment(const SplitPlan& p, int share, int e) {
  const SplitGroup& g = p.grp[split_group_of_tile(p, e)];
  const int tu0 = g.cum + (e - g.tile0) * g.kt;       // first unit of tile e
  const int u0 = share * p.share_units;
  const int u1 = u0 + p.share_units < p.units ? u0 + p.share_units : p.units;
  SplitSegment s;
  s.head = g.head;
  s.q0 = g.q0 + (e - g.tile0) * (WIDE ? kWideRows : kAttnTileRows);
  s.t0 = first_key_tile<WIDE>(p, e, (u0 > tu0 ? u0 : tu0) - tu0);
  s.t1 = first_key_tile<WIDE>(p, e, (u1 < tu0 + g.kt ? u1 : tu0 + g.kt) - tu0);      // (may be one more than there are)
  s.slot = split_slot<WIDE>(p, share, e);
  return s;
}

// Tile e of the excess set for the kernel that adds its segments up: the shares first..last (in key
// order) each left one segment, in slot split_slot(p, share, e).
struct SplitTile {
  int32_t head, q0, first_share, last_share;
};
template <bool WIDE>
__host__ __device__ inline SplitTile split_tile(const SplitPlan& p, int e) {
  const SplitGroup& g = p.grp[split_group_of_tile(p, e)];
  const int tu0 = g.cum + (e - g.tile0) * g.kt;
  return {g.head, g.q0 + (e - g.tile0) * (WIDE ? kWideRows : kAttnTileRows), tu0 / p.share_units, (tu0 + g.kt - 1) / p.share_units};
}

// What the host decides for a launch of 256-row (512-row) tiles on `cus` compute units.  out->n_tiles == 0: no
// split.  *kept_full receives the number of full tiles that stay whole (the first ones, in head
// order), *split_ragged the number of partial tiles (in head order, the first ones) that are split.
// q_off / k_off: H + 1 row offsets each.
inline void plan_attention_split(const int64_t* q_off, const int64_t* k_off, int H, int64_t cus, int tile_rows, SplitPlan* out,
                                 int64_t* kept_full, int* split_ragged) {
  SplitPlan& p = *out;
  p.n_tiles = p.n_groups = p.units = p.share_units = p.shares = p.span = p.slots = p.slot_shift = 0;
  p.tile_rows = tile_rows;
  p.narrow_tiles = 0;
  int64_t full = 0, ragged = 0, min_mk = INT64_MAX;
  for (int h = 0; h < H; ++h) {
    const int64_t mq = q_off[h + 1] - q_off[h], mk = k_off[h + 1] - k_off[h];
    full += mq / tile_rows;
    ragged += (mq % tile_rows) != 0;
    if (mq > 0 && mk < min_mk) min_mk = mk;
  }
  *kept_full = full;
  *split_ragged = 0;
  int n_split_ragged = 0;
  if (cus <= 0 || full + ragged == 0) return;
  const int64_t R = (full + ragged) % cus;
  if (R == 0 || R > kAttnMaxExcess || min_mk < (int64_t)kAttnMinShareUnits * kAttnKeyTile) return;
  // the excess set: partial tiles in head order, then the last full tiles, ascending
  int64_t left = R;
  int64_t units = 0;
  int n_groups = 0, n_tiles = 0;
  const bool wide = tile_rows == kWideRows;
  bool narrow = wide;                                // every partial tile
  for (int h = 0; h < H; ++h) narrow = narrow && (q_off[h + 1] - q_off[h]) % tile_rows <= kAttnTileRows;
  for (int h = 0; h < H && left > 0; ++h) {
    const int64_t mq = q_off[h + 1] - q_off[h], mk = k_off[h + 1] - k_off[h];
    if (mq % tile_rows == 0) continue;
    if (n_groups == kAttnSplitGroups) return;
    const int32_t tiles = (int32_t)((mk + kAttnKeyTile - 1) / kAttnKeyTile), kt = narrow ? (5 * tiles + 7) / 8 : tiles;
    p.grp[n_groups++] = {h, (int32_t)(mq / tile_rows) * tile_rows, n_tiles, (int32_t)units, kt};
    n_tiles += 1;
    units += kt;
    --left;
    ++n_split_ragged;
  }
  const int64_t first_split_full = full - left;     // global index (over heads) of the first full tile that is split
  int64_t tile_start = 0;
  for (int h = 0; h < H && left > 0; ++h) {
    const int64_t mq = q_off[h + 1] - q_off[h], mk = k_off[h + 1] - k_off[h];
    const int64_t nf = mq / tile_rows;
    const int64_t lo = first_split_full > tile_start ? first_split_full : tile_start;   // first split tile of this head
    if (lo < tile_start + nf) {
      if (n_groups == kAttnSplitGroups) return;
      const int32_t cnt = (int32_t)(tile_start + nf - lo);
      const int32_t kt = (int32_t)((mk + kAttnKeyTile - 1) / kAttnKeyTile);
      p.grp[n_groups++] = {h, (int32_t)(lo - tile_start) * tile_rows, n_tiles, (int32_t)units, kt};
      n_tiles += cnt;
      units += (int64_t)cnt * kt;
      left -= cnt;
    }
    tile_start += nf;
  }
  if (left != 0 || units >= ((int64_t)1 << 30)) return;
  // It pays when the tile time it saves - the share (1 - R / cus) of an average tile of the excess
  // set, about 0.75 us per unit - outweighs the second kernel and the traffic of the partial results:
  // (cus - R) * units / R >= 24 * cus.  16 heads, split against whole tiles, by the units saved per CU: 22
  // (7400 rows and keys) 191 : 184 us, 27 (7000) 172 : 172, 33 (6700) 161 : 162, 44 (6376) 146 : 153, 54 (11000)
  // 392 : 406, 78 (10000) 328 : 346.
  // 512-row tiles save twice as much per unit.
  if ((cus - R) * (units / R) < (wide ? 12 : 24) * cus) return;
  // One share per CU.  With any other number some CUs get one more than the others, and twice as many
  // (every CU two) double the partial results: 16 heads of 7000 rows and keys in 330 / 512 / 256 shares 210 /
  // 181 / 172 us, of 10000 in 314 / 512 / 256 364 / 344 / 328, of 15000 in 512 / 256 745 / 708.  Only very long
  // shares are halved, which costs 2 % there (27000 rows and keys 2.27 : 2.21 ms): those launches need more than
  // the library's own array holds, and httm_attention_log2_static refuses them, as it always has.
  // A CU holds one 512-row workgroup.
  int64_t shares = units / kAttnLongShareUnits > cus && !wide ? 2 * cus : cus;
  if (shares > units / kAttnMinShareUnits) shares = units / kAttnMinShareUnits;
  if (shares > kAttnMaxShares) shares = kAttnMaxShares;
  if (shares < 1) return;
  int64_t u = (units + shares - 1) / shares;
  // a tile of kt key tiles is cut into at most kt / u + 2 pieces
  int64_t max_kt = 0;
  for (int g = 0; g < n_groups; ++g) max_kt = p.grp[g].kt > max_kt ? p.grp[g].kt : max_kt;
  const int64_t u_min = (max_kt + kAttnMaxPiecesPerTile - 3) / (kAttnMaxPiecesPerTile - 2);
  if (u < u_min) u = u_min;
  shares = (units + u - 1) / u;
  p.n_groups = n_groups;
  p.units = (int32_t)units;
  p.share_units = (int32_t)u;
  p.shares = (int32_t)shares;
  p.n_tiles = n_tiles;
  int span = 1;
  for (int s = 0; s < p.shares; ++s) {
    const int u0 = s * p.share_units, u1 = u0 + p.share_units < p.units ? u0 + p.share_units : p.units;
    const int d = split_tile_of_unit(p, u1 - 1) - split_tile_of_unit(p, u0) + 1;
    span = d > span ? d : span;
  }
  p.span = span;
  p.slots = p.shares + p.n_tiles - 1;
  if (wide) {
    p.narrow_tiles = narrow ? n_split_ragged : 0;
    if (p.narrow_tiles > 0 && p.narrow_tiles < n_tiles) p.slot_shift = split_tile<true>(p, p.narrow_tiles).first_share + p.narrow_tiles;
    p.slots = split_slot<true>(p, p.shares - 1, n_tiles - 1) + slots_per_segment<true>(p, n_tiles - 1);
  }
  *kept_full = first_split_full;
  *split_ragged = n_split_ragged;
}

// Slots of scratch a plan uses (kAttnSlotWords fp32 words each).
inline int64_t split_slots(const SplitPlan& p) { return p.n_tiles ? p.slots : 0; }

// What the workgroups of a launch are: see choose_attention_route().
enum class AttnTiles {
  kTiles256,    // 256-row tiles; with a split those in excess run in segments
  kTiles128,
  kGroups32,    // tiles of so many rows whose waves share the keys in four / four / two / four / two groups; waves of 32
  kGroups64,    // rows but for the last two, whose 64-row waves read less LDS a product and start and end later
  kGroups128,
  kGroups128Wide,
  kGroups256,
  kRounds,      // whole rounds of 256-row tiles, then the rest in key groups: two launches
  kTiles512,    // log2 keys: 512-row tiles; with a split those in excess run in segments
};

struct AttnRoute {
  AttnTiles tiles;
  SplitPlan split;          // kTiles256 and kTiles512 only; n_tiles == 0: every tile runs whole
  int64_t kept_full;        // full tiles that stay whole, and partial tiles that run in segments
  int32_t split_ragged;
  AttnTiles rest;           // kRounds: what the rest runs in
};

inline int attention_tile_rows(AttnTiles t) {
  switch (t) {
    case AttnTiles::kGroups32: return 32;
    case AttnTiles::kGroups64: return 64;
    case AttnTiles::kTiles128: case AttnTiles::kGroups128: case AttnTiles::kGroups128Wide: return 128;
    case AttnTiles::kTiles512: return kWideRows;
    default: return kAttnTileRows;
  }
}

// The tiles of the only or the last launch of a route.
inline AttnTiles last_tiles(const AttnRoute& r) { return r.tiles == AttnTiles::kRounds ? r.rest : r.tiles; }

// 128-row tiles that run at once (three workgroups per CU): a problem with no more of them runs those
constexpr int64_t kSmallTileRound = 768;

inline int64_t count_tiles(const int64_t* q_off, int H, int rows) {
  int64_t n = 0;
  for (int h = 0; h < H; ++h) n += (q_off[h + 1] - q_off[h] + rows - 1) / rows;
  return n;
}

// The same as the launch's grid deals them to the 8 XCDs, full tiles and the heads' partial ones each by themselves: 8 times
// those of the first XCD, which is what has to fit its share of the CUs.
inline int64_t count_dealt_tiles(const int64_t* q_off, int H, int rows) {
  int64_t full = 0, ragged = 0;
  for (int h = 0; h < H; ++h) {
    full += (q_off[h + 1] - q_off[h]) / rows;
    ragged += (q_off[h + 1] - q_off[h]) % rows != 0;
  }
  return 8 * ((full + 7) / 8 + (ragged + 7) / 8);
}

// Tiles of `rows` rows that are left of the heads when whole rounds of 256-row tiles, the heads' full
// ones in head order, have run.
inline int64_t count_rest_tiles(const int64_t* q_off, int H, int64_t cus, int rows) {
  int64_t full = 0, n = 0;
  for (int h = 0; h < H; ++h) full += (q_off[h + 1] - q_off[h]) / kAttnTileRows;
  int64_t keep = full / cus * cus;
  for (int h = 0; h < H; ++h) {
    const int64_t mq = q_off[h + 1] - q_off[h], nf = mq / kAttnTileRows, whole = nf < keep ? nf : keep;
    keep -= whole;
    n += (mq - whole * kAttnTileRows + rows - 1) / rows;
  }
  return n;
}

// At most one tile of 32, 64, 128 or 256 rows per CU whose waves share the keys, or at most two 128-row tiles of one key
// group per CU (`count(rows)` tiles): those that take the least time, in tenths of a us, for heads of at most kt key tiles.  A wave
// walks a quarter (half) of the keys of its tile; the groups' meeting is in the constant.  us at 16 heads (log2 keys), tiles
// of 32 / 64 / 128 / 128 wide / 256 rows / 128 rows of one group, x where there is more than one a CU:
//   250 x 250 5.5 / 6.7 / 7.8 / 9.5 / 11.4 / 7.1, 500 x 500 6.7 / 8.0 / 9.6 / 11.4 / 14.6 / 9.2, 500 x 4000 22.5 / 23.7 / 34.7 /
//   32.1 / 51 / 45.6, 1000 x 1000 x / 10.3 / 12.7 / 14.5 / 19.8 / 13.6, 1000 x 6000 x / 34.8 / 50 / 45 / 73 / 70, 1384 x 1384
//   x / x / 15.3 / 17.8 / 23.7 / 17.0, 2000 x 500 x / x / 10.2 / 12.0 / 15.1 / 9.8, 2000 x 4500 x / x / 40.1 / 39.2 / 57 / 53, 2000
//   x 14000 x / x / 108 / 99 / 156 / 150, 4000 x 500 x / x / x / x / 15.8 / 13.6, 4000 x 1500 x / x / x / x / 27.4 / 28.1.
// Plain keys take 5 to 15 % more everywhere.
struct AttnGroups {
  AttnTiles tiles;
  int64_t time;
};
// A workgroup with a full tile looks its head up, one after the other (from the ninth on a fortieth of a us each); one with
// a partial tile has it from a list, and heads of at most 64 rows leave half of a 128-row tile's waves out of the way: us, 32-row
// tiles / 128-row tiles of one group, 16 heads of 40 x 73 6.7 / 6.4, 32 of 33 x 66 7.1 / 6.3, 64 of 66 x 69 8.4 / 6.8, but 16 of
// 132 x 67 6.8 / 7.4.  `longest`: rows of the longest head.
template <typename Count>
inline AttnGroups choose_key_groups(Count count, int64_t cus, int64_t kt, int H, int64_t longest) {
  AttnGroups best = {AttnTiles::kTiles256, INT64_MAX};
  auto offer = [&](AttnTiles tiles, int rows, int64_t waves_of_tiles, int64_t time) {
    if (longest >= rows && H > 8) time += (H - 8) / 4;
    if (time < best.time && count(rows) <= waves_of_tiles * cus) best = {tiles, time};
  };
  const int64_t half = (kt + 1) / 2, quarter = (kt + 3) / 4;
  offer(AttnTiles::kGroups32, 32, 1, 45 + 11 * quarter);
  offer(AttnTiles::kGroups64, 64, 1, 58 + 11 * quarter);
  offer(AttnTiles::kGroups128, 128, 1, 60 + 19 * half / 2);
  offer(AttnTiles::kGroups128Wide, 128, 1, 86 + 17 * quarter);
  offer(AttnTiles::kGroups256, kAttnTileRows, 1, 95 + 15 * half);
  offer(AttnTiles::kTiles128, 128, 1, (longest <= 64 ? 44 : 49) + 11 * kt / 2);
  offer(AttnTiles::kTiles128, 128, 2, 60 + 9 * kt);
  return best;
}

// Keys of the shortest head from which on a launch may run in 512-row tiles.
constexpr int64_t kWideKeys = 2048;

// The query rows of a launch: `count` rows of every head from row `first` of the packed tensor.
struct HeadRows {
  int64_t first[HTTM_MAX_HEADS];
  int64_t count[HTTM_MAX_HEADS];
};
inline HeadRows all_rows(const int64_t* q_off, int H) {
  HeadRows r = {};
  for (int h = 0; h < H; ++h) {
    r.first[h] = q_off[h];
    r.count[h] = q_off[h + 1] - q_off[h];
  }
  return r;
}

// kRounds: the rows of the two launches.
inline void split_rounds(const int64_t* q_off, int H, int64_t cus, HeadRows* whole, HeadRows* rest) {
  *whole = *rest = all_rows(q_off, H);
  int64_t keep = 0;
  for (int h = 0; h < H; ++h) keep += whole->count[h] / kAttnTileRows;
  keep = keep / cus * cus;
  for (int h = 0; h < H; ++h) {
    const int64_t nf = whole->count[h] / kAttnTileRows, n = nf < keep ? nf : keep;
    keep -= n;
    whole->count[h] = n * kAttnTileRows;
    rest->first[h] += n * kAttnTileRows;
    rest->count[h] -= n * kAttnTileRows;
  }
}

// First row, inside head h of M rows, of the tile at `q0` of a launch whose rows of that head begin at row `first` of the
// packed tensor: a launch may have the last rows of a head only.
__host__ __device__ inline int row_in_head(int64_t first, int h, int64_t M, int q0) { return (int)(first - h * M) + q0; }

// Tiles of the only or the last launch of a route, dealt out as in count_dealt_tiles.
inline int64_t count_last_tiles(const AttnRoute& r, const int64_t* q_off, int H, int64_t cus) {
  const int rows = attention_tile_rows(last_tiles(r));
  if (r.tiles != AttnTiles::kRounds) return count_dealt_tiles(q_off, H, rows);
  HeadRows whole, rest;
  split_rounds(q_off, H, cus, &whole, &rest);
  int64_t off[HTTM_MAX_HEADS + 1] = {0};
  for (int h = 0; h < H; ++h) off[h + 1] = off[h] + rest.count[h];
  return count_dealt_tiles(off, H, rows);
}

// Log2 keys: whether a launch runs in 512-row tiles, and how it is split.  Both sides' times in ns: a pair of 256-row tiles
// takes 1517 a key tile and 5 us for its ends, segments and their sum 12 us; a 512-row tile in a round 1438 and 10 us, in a launch
// with segments 1454 and 11 us, segments and their sum 22 us (half a tile: a head's last one of at most 256 rows).  Rounds count as the
// grid deals the tiles to the XCDs: one tile more than an XCD has CUs is another round (6 heads of 21713 rows x 3974 keys, 256 tiles:
// 110 us in 256-row tiles, 181 in these).  Fitted to 980 random launches of 1 to 64 heads, each on two to five chips, on which the same
// launches differ by 2 % between the two kinds of tiles: those chosen take 0.983 of the time in 256-row tiles in the mean (0.975 on the
// better chips, 0.987 on the others), 6 % of them more than 1.01, 1.05 at most.  With 1462 and 7.5 us a tile and without the count of what
// is dealt a third took more than 1.01 on the others, 1.65 at most.  Every tile of a round has to be as long as the others:
// one workgroup on a CU leaves it idle behind a short one (12 heads of 36 000 rows against 7000 to 17 000 keys 1126 us in 256-row
// tiles, 1237 in these).  A plan that needs more slots than there are is dropped (kAttnScratchBytes).  us, 256-row tiles / these: 16 heads of
// 16384 x 4096 208 / 204, 16384 x 16384 794 / 759, 17600 x 17600 964 / 945, 23500 x 23500 1622 / 1575, 28650 x 28650 2527 / 2428, 31190 x 31190
// 2897 / 2775, 28380 x 83140 7249 / 6936, 8192 x 83140 2105 / 1897.
inline bool choose_wide_tiles(const int64_t* q_off, const int64_t* k_off, int H, int64_t cus, int64_t scratch_words, AttnRoute* out) {
  AttnRoute& r = *out;
  if ((q_off[H] - q_off[0]) / kWideRows + H < cus) return false;       // (the small launches, which the host's time is most of)
  int64_t min_keys = INT64_MAX, max_keys = 0, full = 0, ragged = 0, tiles256 = 0, work256 = 0;
  int64_t heads = 0, halves = 0, work = 0;    // half tiles, and times their key tiles
  for (int h = 0; h < H; ++h) {
    const int64_t mq = q_off[h + 1] - q_off[h], mk = k_off[h + 1] - k_off[h], kt = (mk + kAttnKeyTile - 1) / kAttnKeyTile;
    if (mq == 0) continue;
    ++heads;
    min_keys = std::min(min_keys, mk);
    max_keys = std::max(max_keys, mk);
    const int64_t n256 = (mq + kAttnTileRows - 1) / kAttnTileRows;
    full += mq / kWideRows;
    ragged += mq % kWideRows != 0;
    tiles256 += n256;
    const int64_t n = mq / kWideRows * 2 + (mq % kWideRows == 0 ? 0 : mq % kWideRows <= kAttnTileRows ? 1 : 2);
    halves += n;
    work += n * kt;
    work256 += n256 * kt;
  }
  const int64_t tiles = full + ragged;
  // (rounds of tiles, one a CU: all have to be of one length)
  if (tiles < cus || min_keys < kWideKeys || max_keys - min_keys > min_keys / 32) return false;
  r.tiles = AttnTiles::kTiles512;
  r.split.n_tiles = 0;
  if (scratch_words > 0) {
    plan_attention_split(q_off, k_off, H, cus, kWideRows, &r.split, &r.kept_full, &r.split_ragged);
    if (split_slots(r.split) * kAttnSlotWords > scratch_words) r.split.n_tiles = 0;
    // (less than an eighth of a round in segments: many short pieces of a tile, 12 heads of 22575 x 22575 and 31752 outliers, 28
    // tiles, 1582 : 1617)
    if (r.split.n_tiles > 0 && r.split.n_tiles * 8 < cus) return false;
  }
  const int64_t time256 = (work256 * 1517 + tiles256 * 5000) / 2 / cus + (tiles256 % cus ? 12000 : 0);
  const bool split = r.split.n_tiles > 0;
  if (split) {
    full = r.kept_full;
    ragged -= r.split_ragged;
  }
  const int64_t rounds = (8 * ((full + 7) / 8 + (ragged + 7) / 8) + cus - 1) / cus;       // (as count_dealt_tiles())
  if (split && rounds * cus > tiles - r.split.n_tiles) return false;
  // (heads of few tiles: an XCD's CUs walk the keys of four and more at a time, and so do the segments.  40 heads of 3685 x 18667 544 /
  // 583, 48 of 4203 x 16739 665 / 704; 12 such launches 1.013 in the mean, 0.96 from 32 768 keys on)
  if (split && tiles < 10 * heads && min_keys < 32768) return false;
  const int64_t time = split ? (work * 727 + tiles * 10800) / cus + 22200 : (work / halves * 1438 + 9860) * rounds;
  return split ? time * 301 <= time256 * 300 : time <= time256;
}

// The whole decision for a launch with room for `scratch_words` fp32 words of partial results (0: none).  `log2_keys`: one
// whose keys carry the logit scale, which may run in 512-row tiles.
inline void choose_attention_route(const int64_t* q_off, const int64_t* k_off, int H, int64_t cus, int64_t scratch_words,
                                   AttnRoute* out, bool log2_keys = false) {
  AttnRoute& r = *out;
  if (log2_keys && choose_wide_tiles(q_off, k_off, H, cus, scratch_words, out)) return;
  r.tiles = AttnTiles::kTiles256;
  r.split.n_tiles = 0;
  if (scratch_words > 0) plan_attention_split(q_off, k_off, H, cus, kAttnTileRows, &r.split, &r.kept_full, &r.split_ragged);
  int64_t full = 0, keys = 0, longest = 0;
  for (int h = 0; h < H; ++h) {
    longest = std::max(longest, q_off[h + 1] - q_off[h]);
    full += (q_off[h + 1] - q_off[h]) / kAttnTileRows;
    if (k_off[h + 1] - k_off[h] > keys) keys = k_off[h + 1] - k_off[h];
  }
  auto no_split = [&]() {
    r.split.n_tiles = r.split.n_groups = r.split.units = r.split.share_units = r.split.shares = r.split.span = r.split.slots = 0;
    r.kept_full = full;
    r.split_ragged = 0;
  };
  if (r.split.n_tiles == 0 || split_slots(r.split) * kAttnSlotWords > scratch_words) no_split();
  // Workgroups that share the keys among their waves walk a quarter (half) of them however many CUs are idle; segments
  // cut the walk over all CUs and cost a second kernel and the traffic of the partial results.  The shorter of the two, in
  // tenths of a us, fitted to 1700 shapes of 1 to 64 heads, 16 to 12000 rows and 200 to 40000 keys, each in every kind of
  // tiles (what this takes is 0.4 % above the best on average and for one in fifty more than 6 %):
  //  * segments: a step is the shorter the fewer of the tile's 256 rows there are, and the pieces of a tile are added up one
  //    after the other (24 heads of 68 x 6785 27 us, key groups 38; one head of 5646 x 5999 33, key groups 29).
  //  * groups in tiles of 32 and 64 rows read every key once a tile: 0.023 us for every key tile of every head, and long
  //    walks at full occupancy an eighth more (64 heads of 90 x 19556 148 us, segments 105; 8 of 1831 x 27212 139 : 126).
  //  * a tile too many on the first XCD is as long as all the others again (3 heads of 5423 x 23452, 252 full tiles of 64 rows
  //    and 3 partial ones: 226 us, segments 114).
  //  * segments that need more than the library's own array are those of keys so long that the estimate is too low for them:
  //    there by the lines 70 + 14, 80 + 16 a quarter, 60 + 15 a half (one head of 29824 x 35072 segments 277, groups 250, 24 of
  //    2346 x 56082 761 : 680, 12 of 2618 x 172602 1332 : 1176, 24 of 1064 x 45280 319 : 316, 8 of 3935 x 91614 583 : 601).
  //    httm_attention_log2_static accepts by them, too: what runs in key groups needs nothing of the array.
  const int64_t kt = (keys + kAttnKeyTile - 1) / kAttnKeyTile, half = (kt + 1) / 2, quarter = (kt + 3) / 4;
  const bool few = count_tiles(q_off, H, 64) <= cus;
  const bool lines = split_slots(r.split) * kAttnSlotWords * 4 > HTTM_STATIC_SCRATCH_BYTES;
  const AttnGroups groups = choose_key_groups(
      [&](int rows) { return lines ? count_tiles(q_off, H, rows) : count_dealt_tiles(q_off, H, rows); }, cus, kt, H, longest);
  const int64_t u = r.split.share_units;
  int64_t groups_time = groups.time, split_time = 0;
  if (lines) {
    groups_time = few ? 70 + 14 * quarter : count_tiles(q_off, H, 128) <= cus ? 80 + 16 * quarter
                : count_tiles(q_off, H, kAttnTileRows) <= cus ? 60 + 15 * half : INT64_MAX;
    split_time = 120 + split_slots(r.split) / 2 + (r.split.shares > cus ? 15 : 9) * u;
  } else if (r.split.n_tiles > 0) {
    int64_t rows = 0, all_kt = 0;
    for (int h = 0; h < H; ++h) {
      const int64_t mq = q_off[h + 1] - q_off[h];
      rows += mq;
      if (mq > 0) all_kt += (k_off[h + 1] - k_off[h] + kAttnKeyTile - 1) / kAttnKeyTile;
    }
    const int64_t tile_rows = kAttnTileRows * count_tiles(q_off, H, kAttnTileRows);
    split_time = 112 + 28 * split_slots(r.split) / 100 + (73 * u + (29 * u + 42 * kt / u) * rows / tile_rows) / 10;
    if (few && groups.tiles != AttnTiles::kTiles256) groups_time += std::max<int64_t>(groups.time - 300, 0) / 8 + 3 * all_kt / 128 - 8;
  }
  if (groups.tiles != AttnTiles::kTiles256 && (r.split.n_tiles == 0 || groups_time <= split_time)) {
    no_split();
    r.tiles = groups.tiles;
    return;
  }
  if (r.split.n_tiles > 0) return;
  // No split.  Whole rounds of 256-row tiles first; what is left - the last rows of the heads - in smaller tiles whose
  // keys are cut in four or two, if those are one round: a half (quarter) of a round instead
  // of a whole one.  From two rounds on (a lone tile on a CU has 0.8 of the rate of a pair): 16 heads of 9000
  // rows and keys 321 -> 294 us, 10186 x 15158 523 -> 495, 12500 579 -> 554; 5516 120 with 128-row tiles, 133 so.
  if (full >= 2 * cus && count_rest_tiles(q_off, H, cus, 128) <= cus) {
    r.tiles = AttnTiles::kRounds;
    r.rest = choose_key_groups([&](int rows) { return count_rest_tiles(q_off, H, cus, rows); }, cus, kt, H, longest).tiles;
    return;
  }
  // Otherwise a short problem that fits into one round of 128-row tiles (three workgroups per CU, 768 at a
  // time) runs those: they fill the chip where the big tiles leave a third of it idle.
  if (count_tiles(q_off, H, 128) <= kSmallTileRound) r.tiles = AttnTiles::kTiles128;
}

}  // namespace httm
