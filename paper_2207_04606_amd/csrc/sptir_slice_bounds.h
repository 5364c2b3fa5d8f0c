// Where the long rows of a matrix cross its slices of columns (shared by the column slices of SpMM and of SDDMM plans).
#ifndef SPTIR_SLICE_BOUNDS_H_
#define SPTIR_SLICE_BOUNDS_H_

#include "sptir_internal.h"
#include "sptir_scan.h"

namespace sptir {
namespace {

constexpr int kBoundsBlock = 256;

// bound[s * room + p] = first entry of the p-th of `rows` whose column is in slice s (`width` columns) or later, s = 0 .. n_slices;
// 0 for p = n_long .. room - 1, rows of no entries.  Slices fastest over the lanes, so that the probes of a wavefront stay in a
// few rows, and through an LDS tile, so that the stores are runs of TILE rows.
template <int TILE>
__global__ __launch_bounds__(kBoundsBlock) void k_slice_bounds(int32_t n_slices, int32_t width, int32_t n_long, int32_t room,
                                                               const int32_t* __restrict__ rows,
                                                               const int32_t* __restrict__ indptr,
                                                               const int32_t* __restrict__ indices, int32_t* __restrict__ bound) {
  __shared__ int32_t tile[TILE][TILE + 1];
  const int n_sc = (n_slices + 1 + TILE - 1) / TILE;
  const int s0 = (int)(blockIdx.x % n_sc) * TILE, p0 = (int)(blockIdx.x / n_sc) * TILE;
  const int ns = min(TILE, n_slices + 1 - s0), np = min(TILE, room - p0);
  for (int i = threadIdx.x; i < np * ns; i += kBoundsBlock) {
    const int pl = i / ns, sl = i - pl * ns, s = s0 + sl;
    int at = 0;
    if (p0 + pl < n_long) {
      const int r = rows[p0 + pl], a = indptr[r], b = indptr[r + 1];
      at = s == 0 ? a : (s == n_slices ? b : lower_bound_col(indices, a, b, (int64_t)s * width));
    }
    tile[sl][pl] = at;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < ns * TILE; i += kBoundsBlock) {
    const int sl = i / TILE, pl = i % TILE;
    if (pl < np) bound[(int64_t)(s0 + sl) * room + p0 + pl] = tile[sl][pl];
  }
}

template <int TILE>
unsigned slice_bounds_workgroups(int32_t n_slices, int64_t room) {
  return (unsigned)(((int64_t)(n_slices + 1 + TILE - 1) / TILE) * ((room + TILE - 1) / TILE));
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_SLICE_BOUNDS_H_
