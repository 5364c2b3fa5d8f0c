// How feature tiles and units of work (row blocks, groups of rows, heavy lists) are dealt to the workgroups of a launch, and with them to the XCDs:
// workgroup ids go round robin to the eight XCDs.  Plain arithmetic, on the device and on the host.
#ifndef SPTIR_TILE_DEAL_H_
#define SPTIR_TILE_DEAL_H_

#include <stdint.h>

#include <algorithm>

#ifdef __HIPCC__
#define SPTIR_ANYWHERE __host__ __device__ __forceinline__
#else
#define SPTIR_ANYWHERE inline
#endif

namespace sptir {
namespace {

enum TileMap : int {
  kMapTilesPerXcd = 0,  // n_tiles multiple of 8: XCD x owns tiles x, x+8, ...
  kMapXcdsPerTile = 1,  // n_tiles in {1,2,4}: 8/n_tiles XCDs share a tile, split the units
  kMapPlain = 2,        // any other tile count: tile = id % n_tiles
  kMapRanges = 3        // as kMapXcdsPerTile, but each XCD of a tile takes consecutive units
};

SPTIR_ANYWHERE unsigned log2_of(unsigned power) { return 31u - (unsigned)__builtin_clz(power); }

// workgroup id -> (unit, feature tile); units are row blocks (hyb) or groups of rows (CSR).  It is the first thing that every workgroup does, and what a small
// graph's launch waits for: shifts where the counts are powers of two, one division for the others, and in decode_deal() nothing that the kernel's launches are
// never dealt by.  With divisions everywhere, of 64 bits for the ranges: 5,515 rows, 230,673 entries, 32 features 9.93 us, 9.67 like this; 50,021 rows,
// 1.5 M entries, 41 features 38.1, 37.9; from CSR 169,343 rows, 1.17 M entries, 128 features 117.1, 115.9.
template <typename Unit>
SPTIR_ANYWHERE void decode_block(unsigned bid, int map_mode, int map_param, int n_tiles, Unit* unit, int* tile) {
  const unsigned q = bid >> 3, x = bid & 7;
  if (map_mode == kMapXcdsPerTile) {
    *tile = (int)(x & ((unsigned)n_tiles - 1));
    *unit = (Unit)((q << log2_of((unsigned)map_param)) + (x >> log2_of((unsigned)n_tiles)));
  } else {
    const bool per_xcd = map_mode == kMapTilesPerXcd;
    const unsigned number = per_xcd ? q : bid, of = per_xcd ? (unsigned)map_param : (unsigned)n_tiles;
    const unsigned whole = number / of, rest = number - whole * of;
    *tile = (int)(per_xcd ? x + 8 * rest : rest);
    *unit = (Unit)whole;
  }
}

// launch geometry shared by both SpMM entry points
struct Geometry {
  int vec, lg, n_tiles, map_mode, map_param;
  int64_t grid;
};

// how n_tiles feature tiles (g->n_tiles) and n_units units are dealt to workgroups
inline bool plan_tiles(int64_t n_units, Geometry* g) {
  if (g->n_tiles % 8 == 0) {
    g->map_mode = kMapTilesPerXcd; g->map_param = g->n_tiles / 8;
    g->grid = n_units * g->n_tiles;
  } else if (8 % g->n_tiles == 0) {
    g->map_mode = kMapXcdsPerTile; g->map_param = 8 / g->n_tiles;
    g->grid = 8 * ((n_units + g->map_param - 1) / g->map_param);
  } else {
    g->map_mode = kMapPlain; g->map_param = 0;
    g->grid = n_units * g->n_tiles;
  }
  return g->grid <= 0x7FFFFFFF;
}

// The same for the launches on a hyb handle, which depart from it where X lies beyond L2 (below).
struct TileDeal {
  int32_t n_tiles, mode, param;
  int32_t n_units;
  int32_t slow_tile, moved;  // kMapXcdsPerTile: the last `moved` units of this tile go to the XCDs of the others
};

// (a unit past the last: nothing to do)  MAY_MOVE, MAY_RANGE: what a launch can be dealt by is known to its kernel, and the others' instructions are not in it.
template <bool MAY_MOVE = true, bool MAY_RANGE = true, typename Unit>
SPTIR_ANYWHERE void decode_deal(unsigned bid, const TileDeal& d, Unit* unit, int* tile) {
  const unsigned q = bid >> 3, x = bid & 7;
  if (MAY_RANGE && d.mode == kMapRanges) {
    const unsigned log2_tiles = log2_of((unsigned)d.n_tiles), log2_ranges = 3 - log2_tiles, h = x >> log2_tiles;
    const unsigned whole = (unsigned)d.n_units >> log2_ranges, rest = (unsigned)d.n_units & ((1u << log2_ranges) - 1);
    const unsigned lo = whole * h + (rest * h >> log2_ranges), hi = whole * (h + 1) + (rest * (h + 1) >> log2_ranges);
    *tile = (int)(x & ((unsigned)d.n_tiles - 1));
    *unit = (Unit)(q < hi - lo ? lo + q : (unsigned)d.n_units);
    return;
  }
  decode_block(bid, d.mode, d.param, d.n_tiles, unit, tile);
  if (MAY_MOVE && d.moved > 0) {  // (four tiles, two XCDs each: the six of the other tiles take turns)
    const unsigned n_units = (unsigned)d.n_units, kept = n_units - (unsigned)d.moved;
    const unsigned slow = (unsigned)d.slow_tile, t = (unsigned)*tile, h = x >> 2;
    if (t == slow) {
      if ((unsigned)*unit >= kept) *unit = (Unit)n_units;
    } else if ((unsigned)*unit >= n_units) {
      const unsigned own = (n_units - h + 1) >> 1;  // units of its own tile
      *tile = (int)slow;
      *unit = (Unit)(kept + (q - own) * 6 + h * 3 + t - (t > slow ? 1 : 0));
    }
  }
}

inline TileDeal deal_of(int64_t n_units, const Geometry& g) {
  return TileDeal{g.n_tiles, g.map_mode, g.map_param, (int32_t)std::min<int64_t>(n_units, 0x7FFFFFFF), 0, 0};
}

// Where the four tiles of a launch of chunk lists are the four lines of every 512 bytes of X, those of the last line are served
// more slowly from beyond L2, whichever XCD asks for them (a gather of 169,343 rows that no cache holds: 69, 79, 68 and 83 us for the
// XCDs of the four lines; one line at a time 49, 49, 49 and 53), and the two XCDs bound to that tile end when the others have been
// idle for a sixth of the launch.  So the others take units of its lists after their own: an eighth, and where heavy lists, which stay where they are, have
// more entries than these, a sixteenth of all entries' worth, up to a quarter of the units.  169,343 rows, 1.17 M entries, 128 features, operands that
// change from call to call: 178 -> 170 us for a product and the transposed one (a sixteenth 173, a tenth 171).  Of 128 features: 35 power-law graphs, both products,
// 1.024 times as fast as with none moved (a twelfth 1.019, a sixteenth 1.016); even lists whose columns are alike, 76 of them, 1.002 (0.95 to 1.07; a
// sixteenth 1.010), and which it is the handle does not know.  Over a single partition even lists lose 2 to 5 % by an eighth, nothing by a sixteenth.  Lists of
// fewer than 200 entries: 0.993 on 50 graphs (0.92 to 1.03), so none of those.  The fewest units, 512, when a unit had four lists; with one list each 35 graphs of
// 400 to 1900 of them 0.995, by their short lists.
// Not where an L2 holds most of a tile's column of X (132,534 rows in eight launches: 994 us, 1019 with it).  Only the last line gives units away: that the second
// one is late too (79 us) was seen, but nothing dealt by it yet.
// x: the address of the launch's first feature; n_cols: the rows of X that its entries range over; list_entries, heavy_entries: of the call's n_lists lists, and of
// its heavy ones; one_partition: so a launch ranges over
constexpr int64_t kMovedBytes = (int64_t)8 << 20, kMovedUnits = 512, kMovedEntries = 200;
// (Launches of rounds are too small for it: what a GPU holds at once are at most 256 workgroups of four lists for each of four tiles.)
inline void move_slow_units(uintptr_t x, int feat, int64_t n_cols, Geometry* g, TileDeal* d, int64_t list_entries = 1, int64_t heavy_entries = 1,
                            int64_t n_lists = 0, bool one_partition = false) {
  if (d->mode != kMapXcdsPerTile || d->n_tiles != 4 || g->vec * g->lg != 32 || feat % 128 != 0 || x % 128 != 0 ||
      n_cols * 128 < kMovedBytes || d->n_units < kMovedUnits || list_entries < 1 || list_entries < kMovedEntries * n_lists)
    return;
  const double share = std::max(one_partition ? 1. / 16 : 1. / 8, std::min(0.25, (1. + (double)heavy_entries / (double)list_entries) / 16));
  const int64_t moved = (int64_t)((double)d->n_units * share), helpers = 8 - d->param;
  const int64_t grid = g->grid + 8 * ((moved + helpers - 1) / helpers);
  if (grid > 0x7FFFFFFF) return;
  d->slow_tile = (int32_t)(3 - (x / 128 & 3));
  d->moved = (int32_t)moved;
  g->grid = grid;
}

// Heavy lists: an XCD of a tile's takes consecutive ones.  They are in partition order, so that it gathers from fewer columns of X
// than where the XCDs of a tile take turns.  25 power-law graphs with heavy lists and two or four tiles: 1.07 times as fast (1.00 to 1.17; in rounds 1.00, 1.03
// and 1.09).  144,465 rows, 1.04 M entries, 100 features 129 -> 110 us; 230,000 rows, 10 M entries, 128 features in a single launch 521 -> 513.  Not with a
// single tile, whose chunk lists and heavy lists then are in different partitions at a time (50,021 rows, 1.5 M entries, 41 features: 38.4 us, 42.1 with it).
inline void deal_ranges(TileDeal* d) {
  if (d->mode == kMapXcdsPerTile && d->n_tiles > 1) d->mode = kMapRanges;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_TILE_DEAL_H_
