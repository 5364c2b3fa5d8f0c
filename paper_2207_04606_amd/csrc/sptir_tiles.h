// What the SpMM kernels share: lane loads and stores (and tile_deal.h: how feature tiles are dealt to the XCDs).
#ifndef SPTIR_TILES_H_
#define SPTIR_TILES_H_

#include "sptir_internal.h"
#include "tile_deal.h"

namespace sptir {
namespace {

template <int VEC> struct Vec;
template <> struct Vec<4> { using type = float4; };
template <> struct Vec<1> { using type = float; };

template <int VEC>
__device__ __forceinline__ void load_vec(float (&x)[VEC], const float* p) {
  typename Vec<VEC>::type v = *reinterpret_cast<const typename Vec<VEC>::type*>(p);
  if constexpr (VEC == 4) { x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
  else { x[0] = v; }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&x)[VEC]) {
  if constexpr (VEC == 4) *reinterpret_cast<float4*>(p) = make_float4(x[0], x[1], x[2], x[3]);
  else *p = x[0];
}

// Four floats at any 4-byte aligned address: one global_load/store_dwordx4 (the hardware takes it unaligned).
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

template <int VEC>
__device__ __forceinline__ void load_unaligned(float (&x)[VEC], const float* p) {
  if constexpr (VEC == 4) {
    const float4u v = *reinterpret_cast<const float4u*>(p);
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
  } else {
    static_assert(VEC == 1, "4 or 1 floats per lane");
    x[0] = *p;
  }
}
template <int VEC>
__device__ __forceinline__ void store_unaligned(float* p, const float (&x)[VEC]) {
  if constexpr (VEC == 4) *reinterpret_cast<float4u*>(p) = float4u{x[0], x[1], x[2], x[3]};
  else *p = x[0];
}

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + nb && b0 < a0 + na;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_TILES_H_
