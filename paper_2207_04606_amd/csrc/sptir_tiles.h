// What the SpMM kernels share: lane loads and stores, and how feature tiles are dealt to the XCDs.
#ifndef SPTIR_TILES_H_
#define SPTIR_TILES_H_

#include "sptir_internal.h"

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

enum TileMap : int {
  kMapTilesPerXcd = 0,  // n_tiles multiple of 8: XCD x owns tiles x, x+8, ...
  kMapXcdsPerTile = 1,  // n_tiles in {1,2,4}: 8/n_tiles XCDs share a tile, split the units
  kMapPlain = 2         // any other tile count: tile = id % n_tiles
};

// workgroup id -> (unit, feature tile); units are row blocks (hyb) or groups of rows (CSR)
__device__ __forceinline__ void decode_block(unsigned bid, int map_mode, int map_param, int n_tiles, int64_t* unit,
                                             int* tile) {
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
bool plan_tiles(int64_t n_units, Geometry* g) {
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

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + nb && b0 < a0 + na;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_TILES_H_
