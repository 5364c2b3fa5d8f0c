// The forms of decode_deal() (csrc/tile_deal.h, compiled alone) that kernels are built with, against the one that knows every way to deal, for
// test_tile_deal_forms.py: prints how many workgroups were compared, and fails where one differs.
//   forms KIND N_UNITS N_TILES   (KIND: plain, lists, heavy)
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "tile_deal.h"

namespace {
template <bool MAY_MOVE, bool MAY_RANGE>
bool same(unsigned bid, const sptir::TileDeal& d) {
  int64_t unit;
  int tile, tile_here;
  unsigned unit_here;
  sptir::decode_deal(bid, d, &unit, &tile);
  sptir::decode_deal<MAY_MOVE, MAY_RANGE>(bid, d, &unit_here, &tile_here);
  return (int64_t)unit_here == unit && (tile_here == tile || unit >= d.n_units);
}
}  // namespace

int main(int argc, char** argv) {
  if (argc != 4) return 1;
  const int64_t n_units = atoll(argv[2]);
  sptir::Geometry g{4, 8, atoi(argv[3]), 0, 0, 0};
  if (!sptir::plan_tiles(n_units, &g)) return 2;
  sptir::TileDeal d = sptir::deal_of(n_units, g);
  const bool lists = !strcmp(argv[1], "lists"), heavy = !strcmp(argv[1], "heavy");
  if (lists) sptir::move_slow_units(4096, 128, 1 << 16, &g, &d);
  if (heavy) sptir::deal_ranges(&d);
  const int64_t step = g.grid > 100000 ? g.grid / 50021 : 1;
  int64_t n = 0;
  for (int64_t bid = 0; bid < g.grid; bid += bid + 64 < g.grid ? step : 1, ++n) {
    const unsigned b = (unsigned)bid;
    if (!heavy && !same<true, false>(b, d)) return 3;
    if (!lists && !same<false, true>(b, d)) return 4;
    if (!heavy && d.moved == 0 && !same<false, false>(b, d)) return 5;
  }
  printf("%lld\n", (long long)n);
  return 0;
}
