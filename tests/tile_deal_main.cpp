// How units and feature tiles are dealt to workgroups (csrc/tile_deal.h, compiled alone), for test_tile_deal.py.
//   deal KIND N_UNITS N_TILES X FEAT N_COLS: prints "bid unit tile" of every workgroup that has a unit, and last "grid moved slow_tile"
//   KIND: plain, lists (chunk lists on the X at that address), heavy
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "tile_deal.h"

int main(int argc, char** argv) {
  if (argc != 8 || strcmp(argv[1], "deal")) return 1;
  const int64_t n_units = atoll(argv[3]);
  sptir::Geometry g{4, 8, atoi(argv[4]), 0, 0, 0};
  if (!sptir::plan_tiles(n_units, &g)) return 2;
  sptir::TileDeal d = sptir::deal_of(n_units, g);
  if (!strcmp(argv[2], "lists")) sptir::move_slow_units((uintptr_t)atoll(argv[5]), atoi(argv[6]), atoll(argv[7]), &g, &d);
  else if (!strcmp(argv[2], "heavy")) sptir::deal_ranges(&d);
  for (int64_t bid = 0; bid < g.grid; ++bid) {
    int64_t unit;
    int tile;
    sptir::decode_deal((unsigned)bid, d, &unit, &tile);
    if (unit < n_units) printf("%lld %lld %d\n", (long long)bid, (long long)unit, tile);
  }
  printf("%lld %d %d\n", (long long)g.grid, (int)d.moved, (int)d.slow_tile);
  return 0;
}
