// How many units of the slow line's tile move (csrc/tile_deal.h, compiled alone), for test_tile_deal_share.py.
//   share N_UNITS LIST_ENTRIES HEAVY_ENTRIES N_LISTS ONE_PARTITION: prints how many, after it has seen that every unit of the four tiles is dealt once
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "tile_deal.h"

int main(int argc, char** argv) {
  if (argc != 6) return 1;
  const int64_t n_units = atoll(argv[1]);
  sptir::Geometry g{4, 8, 4, 0, 0, 0};
  if (!sptir::plan_tiles(n_units, &g)) return 2;
  sptir::TileDeal d = sptir::deal_of(n_units, g);
  sptir::move_slow_units(0, 128, 1 << 16, &g, &d, atoll(argv[2]), atoll(argv[3]), atoll(argv[4]), atoi(argv[5]) != 0);
  std::vector<int> dealt(4 * (size_t)n_units, 0);
  for (int64_t bid = 0; bid < g.grid; ++bid) {
    unsigned unit;
    int tile;
    sptir::decode_deal<true, false>((unsigned)bid, d, &unit, &tile);
    if (unit < n_units) ++dealt[(size_t)tile * n_units + unit];
  }
  for (int n : dealt)
    if (n != 1) return 3;
  printf("%d\n", (int)d.moved);
  return 0;
}
