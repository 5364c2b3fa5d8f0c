// Prints "hint feat width lane_quads" for every feature size a plan can be made for and every size it may be called with.
#include <stdio.h>
#include <stdlib.h>

#include "sddmm_slice_shape.h"

int main(int argc, char** argv) {
  const int most_hint = atoi(argv[1]), most_feat = atoi(argv[2]);
  (void)argc;
  for (int hint = 1; hint <= most_hint; ++hint)
    for (int feat = 1; feat <= most_feat; ++feat) {
      const int32_t width = sptir::slice_width(hint);
      printf("%d %d %d %d\n", hint, feat, (int)width, width ? sptir::slice_lane_quads(width, feat) : 0);
    }
  return 0;
}
