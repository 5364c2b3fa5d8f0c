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

// workgroup id -> (unit, feature tile); units are row blocks (hyb) or groups of rows (CSR)
SPTIR_ANYWHERE void decode_block(unsigned bid, int map_mode, int map_param, int n_tiles, int64_t* unit, int* tile) {
  if (map_mode == kMapTilesPerXcd) {
    unsigned q = bid >> 3, x = bid & 7;
    *tile = (int)(x + 8 * (q % (unsigned)map_param));
    *unit = q / (unsigned)map_param;
  } else if (map_mode == kMapXcdsPerTile) {
    unsigned q = bid >> 3, x = bid & 7;
    *tile = (int)(x % (unsigned)n_tiles);
    *unit = (int64_t)q * map_param + x / (unsigned)n_tiles;
  } else {
    *tile = (int)(bid % (unsigned)n_tiles);
    *unit = bid / (unsigned)n_tiles;
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

// (a unit past the last: nothing to do)
SPTIR_ANYWHERE void decode_deal(unsigned bid, const TileDeal& d, int64_t* unit, int* tile) {
  const unsigned q = bid >> 3, x = bid & 7, n_tiles = (unsigned)d.n_tiles, param = (unsigned)d.param, n_units = (unsigned)d.n_units;
  if (d.mode == kMapRanges) {
    const unsigned h = x / n_tiles;
    const unsigned lo = (unsigned)((uint64_t)n_units * h / param), hi = (unsigned)((uint64_t)n_units * (h + 1) / param);
    *tile = (int)(x % n_tiles);
    *unit = q < hi - lo ? lo + q : n_units;
    return;
  }
  decode_block(bid, d.mode, d.param, d.n_tiles, unit, tile);
  if (d.moved > 0) {
    const unsigned slow = (unsigned)d.slow_tile, t = (unsigned)*tile, h = x / n_tiles, kept = n_units - (unsigned)d.moved;
    if (t == slow) {
      if (*unit >= kept) *unit = n_units;
    } else if (*unit >= n_units) {
      const unsigned own = (n_units - h + param - 1) / param;  // units of its own tile
      *tile = (int)slow;
      *unit = (int64_t)kept + (int64_t)(q - own) * (8 - param) + h * (n_tiles - 1) + t - (t > slow ? 1 : 0);
    }
  }
}

inline TileDeal deal_of(int64_t n_units, const Geometry& g) {
  return TileDeal{g.n_tiles, g.map_mode, g.map_param, (int32_t)std::min<int64_t>(n_units, 0x7FFFFFFF), 0, 0};
}

// Where the four tiles of a launch of chunk lists are the four lines of every 512 bytes of X, those of the last line are served
// more slowly from beyond L2, whichever XCD asks for them (a gather of 169,343 rows that no cache holds: 69, 79, 68 and 83 us for the
// XCDs of the four lines; one line at a time 49, 49, 49 and 53), and the two XCDs bound to that tile end when the others have been
// idle for a sixth of the launch.  So the others take an eighth of its units after their own.  169,343 rows, 1.17 M entries, 128
// features, operands that change from call to call: 186 -> 177 us for a product and the transposed one (a tenth 180, a fifth 176);
// other graphs of that size 101.7 -> 100.9 and 105.5 -> 104.2; 230,000 rows, 10 M entries in rounds 509 -> 489.  Not where an L2
// holds most of a tile's column of X (132,534 rows in eight launches: 994 us, 1019 with it).
// x: the address of the launch's first feature; n_cols: the rows of X that its entries range over
constexpr int64_t kMovedBytes = (int64_t)8 << 20, kMovedShare = 8, kMovedUnits = 512;
inline void move_slow_units(uintptr_t x, int feat, int64_t n_cols, Geometry* g, TileDeal* d) {
  if (d->mode != kMapXcdsPerTile || d->n_tiles != 4 || g->vec * g->lg != 32 || feat % 128 != 0 || x % 128 != 0 ||
      n_cols * 128 < kMovedBytes || d->n_units < kMovedUnits)
    return;
  const int64_t moved = d->n_units / kMovedShare, helpers = 8 - d->param;
  const int64_t grid = g->grid + 8 * ((moved + helpers - 1) / helpers);
  if (grid > 0x7FFFFFFF) return;
  d->slow_tile = (int32_t)(3 - (x / 128 & 3));
  d->moved = (int32_t)moved;
  g->grid = grid;
}

// Heavy lists: an XCD of a tile's takes consecutive ones.  They are in partition order, so that it gathers from fewer columns of X
// than where the XCDs of a tile take turns.  169,343 rows, 1.17 M entries, 128 features (two XCDs a tile, two partitions of four
// each) 105.5 -> 101.3 us, 64 features 1.02 times as fast, 230,000 rows, 10 M entries in rounds 509 -> 489; 50,000 x 60,000 columns, 0.9 M
// entries, two partitions 63 -> 60.  Not with a single tile, whose chunk lists and heavy lists then are in different
// partitions at a time (50,021 rows, 1.5 M entries, 41 features: 38.4 us, 42.1 with it).
inline void deal_ranges(TileDeal* d) {
  if (d->mode == kMapXcdsPerTile && d->n_tiles > 1) d->mode = kMapRanges;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_TILE_DEAL_H_
