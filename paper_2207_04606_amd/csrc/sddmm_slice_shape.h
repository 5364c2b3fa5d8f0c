// Column slices of an SDDMM plan: their width, their layout in LDS, and which kernel takes a call.  No device code, so
// that the choice can be checked for every pair of feature sizes without a GPU.
#ifndef SPTIR_SDDMM_SLICE_SHAPE_H_
#define SPTIR_SDDMM_SLICE_SHAPE_H_

#include <stdint.h>

namespace sptir {

constexpr int kSliceBytes = 155 * 1024;  // of Yt in LDS; one workgroup a CU (two of 64 KB: 6 % slower, pieces half as long)
constexpr int kColumnBits = 13;          // of a column inside its slice (4 floats: 8192 columns)
constexpr int kLdsMostFeat = 256;        // floats of a row that the eight lanes of a group hold in eight float4 each

// Row to row in LDS, in float4: where all rows would begin in the same half of the 64 banks, half a row of banks more, or the
// lane groups meet in it (random 512-byte rows: 75 TB/s, 83 if half of them begin in the other half).
constexpr int slice_stride(int quads) { return quads % 16 == 0 ? quads + 8 : quads; }

// Columns per slice of a plan made for `feat` features; 0: no slices.
constexpr int32_t slice_width(int64_t feat) {
  if (feat > kLdsMostFeat) return 0;
  const int32_t fit = (int32_t)(kSliceBytes / (16 * slice_stride((int)(feat + 3) / 4))), most = 1 << kColumnBits;
  return fit < most ? fit : most;
}

// Float4 per lane of the kernel that takes a call from LDS, or 0: from memory (k_sddmm_segments), where a row has fewer than
// four floats, or more than a lane group holds, or the plan's slices have no room for it.
constexpr int slice_lane_quads(int32_t width, int32_t feat) {
  if (feat < 4 || feat > kLdsMostFeat) return 0;
  if ((int64_t)width * slice_stride((feat + 3) / 4) * 16 > kSliceBytes) return 0;
  return (feat + 31) / 32;
}

}  // namespace sptir

#endif  // SPTIR_SDDMM_SLICE_SHAPE_H_
