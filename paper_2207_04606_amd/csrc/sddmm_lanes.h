// What the SDDMM kernels share: the dot product of a lane and the reduction over the eight lanes of a group.
#ifndef SPTIR_SDDMM_LANES_H_
#define SPTIR_SDDMM_LANES_H_

#include <hip/hip_runtime.h>

namespace sptir {
namespace {

__device__ __forceinline__ float dot4(const float4& a, const float4& b, float acc) {
  acc = fmaf(a.x, b.x, acc);
  acc = fmaf(a.y, b.y, acc);
  acc = fmaf(a.z, b.z, acc);
  return fmaf(a.w, b.w, acc);
}

// the value of the lane that `ctrl` names (data-parallel primitive: no trip through LDS)
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Eight partial sums per lane -> lane fl of every 8-lane group ends with the group's total of p[fl].  The partners are lanes
// 7 - fl, fl ^ 2 and fl ^ 1, which DPP reaches and which together span the group.
__device__ __forceinline__ float reduce_scatter8(float (&p)[8], int fl) {
  constexpr int kMirror8 = 0x141, kXor2 = 0x4E, kXor1 = 0xB1;  // row_half_mirror, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
  float q[4], r[2];
  const bool hi4 = (fl & 4) != 0, hi2 = (fl & 2) != 0, hi1 = (fl & 1) != 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // the partner keeps the other half
    const float keep = hi4 ? p[i + 4] : p[i], give = hi4 ? p[i] : p[i + 4];
    q[i] = keep + from_lane<kMirror8>(give);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = hi2 ? q[i + 2] : q[i], give = hi2 ? q[i] : q[i + 2];
    r[i] = keep + from_lane<kXor2>(give);
  }
  const float keep = hi1 ? r[1] : r[0], give = hi1 ? r[0] : r[1];
  return keep + from_lane<kXor1>(give);
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_SDDMM_LANES_H_
