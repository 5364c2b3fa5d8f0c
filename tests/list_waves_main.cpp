// Wavefronts per workgroup of chunk lists (csrc/list_waves.h, compiled alone), for test_list_waves.py.
//   reads lines "rounds n_launches parts n_cols n_lists entries chunks longest feat tile_floats n_tiles" and prints the wavefronts of each
#include <stdio.h>

#include "list_waves.h"

int main() {
  long long v[11];
  for (;;) {
    for (int i = 0; i < 11; ++i)
      if (scanf("%lld", v + i) != 1) return i == 0 ? 0 : 1;
    printf("%d\n", sptir::list_waves({v[0] != 0, (int32_t)v[1], (int32_t)v[2], v[3], v[4], v[5], v[6], v[7], (int32_t)v[8], (int32_t)v[9],
                                      (int32_t)v[10]}));
  }
}
