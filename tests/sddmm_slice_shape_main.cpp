// Host rules of the column slices of an SDDMM plan, for test_sddmm_slice_shape.py.
//   shape MOST_HINT MOST_FEAT: prints "hint feat width lane_quads" for every feature size a plan can be made for and every
//                              size it may be called with
//   pay N_COLS FEAT N_LONG LONG_NNZ UNITS N_SEGS N_SLICES HALF_IN: prints whether slices are chosen, before and after the segments are counted
//   half N_SLICES PARTS: reads the same as `units`, and prints how many slices have half of the segments
//   long BEGIN END NNZ MIN_DEG: prints whether the row is one that slices may take
//   units N_SLICES PARTS MOST: reads the first segment of every part and slice, and the end, and prints "slice begin end" of every unit
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "sddmm_slice_shape.h"

int main(int argc, char** argv) {
  if (argc == 4 && !strcmp(argv[1], "shape")) {
    const int most_hint = atoi(argv[2]), most_feat = atoi(argv[3]);
    for (int hint = 1; hint <= most_hint; ++hint)
      for (int feat = 1; feat <= most_feat; ++feat) {
        const int32_t width = sptir::slice_width(hint);
        printf("%d %d %d %d\n", hint, feat, (int)width, width ? sptir::slice_lane_quads(width, feat) : 0);
      }
  } else if (argc == 10 && !strcmp(argv[1], "pay")) {
    long long v[10] = {0};
    for (int i = 2; i < 10; ++i) v[i] = atoll(argv[i]);
    printf("%d %d\n", sptir::slices_pay(v[2], v[3], v[4], v[5]) ? 1 : 0,
           sptir::slices_pay_as_counted(v[2], v[3], v[4], v[5], v[6], v[7], (int32_t)v[8], (int32_t)v[9]) ? 1 : 0);
  } else if (argc == 6 && !strcmp(argv[1], "long")) {
    printf("%d\n", sptir::is_long_row(atoll(argv[2]), atoll(argv[3]), atoll(argv[4]), atoll(argv[5])) ? 1 : 0);
  } else if ((argc == 5 && !strcmp(argv[1], "units")) || (argc == 4 && !strcmp(argv[1], "half"))) {
    const int n_slices = atoi(argv[2]), parts = atoi(argv[3]);
    std::vector<int32_t> begin((size_t)n_slices * parts + 1);
    for (int32_t& b : begin)
      if (scanf("%d", &b) != 1) return 1;
    if (argc == 4) {
      printf("%d\n", (int)sptir::slices_of_half(begin, n_slices, parts));
      return 0;
    }
    for (const sptir::SliceUnit& u : sptir::slice_units(begin, n_slices, parts, atoll(argv[4]))) printf("%d %d %d\n", u.slice, u.begin, u.end);
  } else {
    return 2;
  }
  return 0;
}
