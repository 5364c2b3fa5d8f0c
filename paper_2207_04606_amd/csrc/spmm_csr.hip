// SpMM straight from CSR, one pass, no decomposition: the "no-hyb" variant
// that section 4.2.1 of arXiv 2207.04606 compares hyb against.
//
// Mapping (gfx950, wave64).  A workgroup of eight wavefronts owns 64 (a small
// dense matrix: 16 or 8) consecutive rows and one feature tile (32 floats, eight lanes of four), bound to XCDs like
// the tiles of the hyb kernels.  What a row costs is its gathers of X, so rows
// are treated by length:
//   short   (<= kShortRow) one lane group per row, eight rows per wavefront at
//           once, eight gathers in flight per lane.  A wavefront per row, as
//           this kernel began, leaves seven of eight lane groups re-reading
//           the same line on rows of seven entries;
//   medium  the wavefront takes the row alone, 64 entries per step;
//   long    (> kLongRow) all eight wavefronts share the row and meet in LDS: a
//           row of 13,000 entries on one wavefront took 0.6 ms, seven times
//           the rest of its graph together.
// Every wavefront loads the 64 row lengths itself (one coalesced load), so all
// of them know the long rows without a barrier, and a workgroup without long
// rows never meets one.  Where rows are short in the mean, the long ones are taken
// by workgroups that come before all others instead.  Sums have a fixed order: results are reproducible.
// The fourth lane of a tail reads (and writes) the last four floats of the
// row, so any feature size of four or more uses 16-byte accesses; they need
// only 4-byte alignment.
// Measured (169,343 rows, 1,166,243 entries, 128 features): 0.65 -> 0.114 ms on
// operands that change from call to call (0.107 on the same ones), 5.2 TB/s of
// gathered rows of which a quarter hit L2; the memory-side cache delivers 7.9 at
// random.
#include <algorithm>
#include <type_traits>

#include "sptir_internal.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

struct CsrArgs {
  const int32_t* indptr;
  const int32_t* indices;
  const float* values;
  const float* X;
  float* Y;
  int32_t n_rows;
  int32_t feat;
  int32_t n_tiles;
  int32_t map_mode;
  int32_t map_param;
  // LONG_FIRST: the workgroups before the others (a multiple of 8), and among them those of a tile
  uint32_t long_grid;
  int32_t long_mode, long_param, long_units;
};

constexpr int kCsrRows = 64;     // most rows per workgroup: one per lane when their lengths are loaded
constexpr int kShortRow = 32;    // four steps of one lane group: 16..48 measured alike
constexpr int kLongRow = 512;    // eight steps of one wavefront (1024: 5 % slower on power-law rows, 256: the same); half
                                 // of it with 16 rows per workgroup, twice of it where every wavefront has one row
                                 // (3,576 rows, 514,589 entries: 14 us against 17)

// LONG_FIRST: workgroups of their own take the long rows, before the others begin
template <int VEC, int LG, int ROWS, bool LONG_FIRST>
__global__ __launch_bounds__(512) void k_spmm_csr(CsrArgs a) {
  constexpr int kGroups = 64 / LG, kWaves = 8, kRowsPerWave = ROWS / kWaves;
  constexpr int UB = LG < 8 ? LG : 8, kTile = VEC * LG;
  static_assert(kRowsPerWave % kGroups == 0 || kGroups % kRowsPerWave == 0, "rows of a wavefront in whole passes");
  __shared__ __align__(16) float part[kWaves][kTile];
  int64_t unit;
  int tile_id;
  const bool for_long = LONG_FIRST && blockIdx.x < a.long_grid;
  if (for_long) decode_block(blockIdx.x, a.long_mode, a.long_param, a.n_tiles, &unit, &tile_id);
  else decode_block(blockIdx.x - (LONG_FIRST ? a.long_grid : 0u), a.map_mode, a.map_param, a.n_tiles, &unit, &tile_id);
  const int64_t row0 = for_long ? 0 : unit * ROWS;
  if (row0 >= a.n_rows || (for_long && unit >= a.long_units)) return;
  const int lane = threadIdx.x & 63, g = lane / LG, fl = lane & (LG - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int f_nominal = tile_id * kTile + fl * VEC;
  const bool f_active = f_nominal < a.feat;
  const int f0 = f_nominal + VEC <= a.feat ? f_nominal : a.feat - VEC;  // (a tail lane repeats floats of its neighbour)
  const float* Xf = a.X + (f_active ? f0 : 0);
  float* Yf = a.Y + f0;
  const size_t feat = (size_t)a.feat;

  // lane l: first entry and length of row row0 + l
  int row_begin = 0, row_len = 0;
  if (!for_long && lane < ROWS && row0 + lane < a.n_rows) {
    row_begin = a.indptr[row0 + lane];
    row_len = a.indptr[row0 + lane + 1] - row_begin;
  }

  constexpr int kLong = ROWS == 8 ? 2 * kLongRow : ROWS == 16 ? kLongRow / 2 : kLongRow;
  float acc[VEC];
  // entries [first, first + left) of a row summed by this lane group, `stride` entries apart from step to step; the
  // next step's entries are fetched while this one's gathers are in flight (two steps of gathers in flight measured
  // no faster: 0.144 against 0.122 ms, half the wavefronts)
  auto walk = [&](int first, int left, int stride) {
    if (!__any(left > 0)) return;
    int c = 0;
    float v = 0.f;
    auto fetch = [&]() {
      const bool ok = fl < UB && fl < left;
      c = ok ? a.indices[first + fl] : 0;
      v = ok ? a.values[first + fl] : 0.f;
    };
    fetch();
    do {
      float x[UB][VEC];
      float vu[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int cu = __shfl(c, g * LG + u, 64);
        vu[u] = __shfl(v, g * LG + u, 64);
        if (f_active && u < left) load_unaligned<VEC>(x[u], Xf + (size_t)cu * feat);
        else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) x[u][e] = 0.f;
        }
      }
      first += stride;
      left -= stride;
      fetch();
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = fmaf(vu[u], x[u][e], acc[e]);
    } while (__any(left > 0));
  };
  auto clear = [&]() {
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  };
  auto sum_lane_groups = [&]() {
#pragma unroll
    for (int d = LG; d < 64; d <<= 1)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += __shfl_xor(acc[e], d, 64);
  };

  // a long row, by the whole workgroup
  auto long_row = [&](int64_t row, int first, int len) {
    const int o = (wave * kGroups + g) * UB;
    clear();
    walk(first + o, len - o, kWaves * kGroups * UB);
    sum_lane_groups();
    if (g == 0) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) part[wave][fl * VEC + e] = acc[e];
    }
    __syncthreads();
    if (wave == 0 && g == 0 && f_active) {
#pragma unroll
      for (int w = 1; w < kWaves; ++w)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += part[w][fl * VEC + e];
      store_unaligned<VEC>(Yf + (size_t)row * feat, acc);
    }
    __syncthreads();
  };
  if constexpr (LONG_FIRST) {
    if (for_long) {
      __shared__ unsigned long long span_long[2][kWaves];
      int turn = 0;
      // 512 rows at a time, one per thread and a.long_units apart: where long rows are neighbours (rows in the order of their
      // lengths) each of these workgroups has its share.  (512 in a row: 169,343 rows so ordered 1247 us, 113 in no order.)
      const int64_t step = a.long_units;
      for (int64_t r0 = unit; r0 < a.n_rows; r0 += 512 * step, turn ^= 1) {
        const int64_t r = r0 + threadIdx.x * step;
        const int len = r < a.n_rows ? a.indptr[r + 1] - a.indptr[r] : 0;
        const unsigned long long mine = __ballot(len > kLong);
        if (lane == 0) span_long[turn][wave] = mine;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w)
          for (unsigned long long left = span_long[turn][w]; left; left &= left - 1) {
            const int64_t row = r0 + (w * 64 + __builtin_ctzll(left)) * step;
            const int first = __builtin_amdgcn_readfirstlane(a.indptr[row]);
            long_row(row, first, __builtin_amdgcn_readfirstlane(a.indptr[row + 1]) - first);
          }
      }
      return;
    }
  } else {
    // (every wavefront sees the same mask)
    for (unsigned long long long_rows = __ballot(row_len > kLong); long_rows; long_rows &= long_rows - 1) {
      const int src = __builtin_ctzll(long_rows);
      long_row(row0 + src, __builtin_amdgcn_readlane(row_begin, src), __builtin_amdgcn_readlane(row_len, src));
    }
  }
  // short rows: a lane group each
  constexpr int kPasses = (kRowsPerWave + kGroups - 1) / kGroups;
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    const int in_wave = p * kGroups + g;
    const int src = wave * kRowsPerWave + (in_wave < kRowsPerWave ? in_wave : 0);
    const int first = __shfl(row_begin, src, 64), len = __shfl(row_len, src, 64);
    const bool mine = in_wave < kRowsPerWave && len <= kShortRow && row0 + src < a.n_rows;
    clear();
    walk(first, mine ? len : 0, UB);
    if (mine && f_active) store_unaligned<VEC>(Yf + (size_t)(row0 + src) * feat, acc);
  }
  // medium rows: the wavefront each
  unsigned long long medium = __ballot(row_len > kShortRow && row_len <= kLong) &
                              (((1ull << kRowsPerWave) - 1) << (wave * kRowsPerWave));
  while (medium) {
    const int src = __builtin_ctzll(medium);
    medium &= medium - 1;
    const int first = __builtin_amdgcn_readlane(row_begin, src), len = __builtin_amdgcn_readlane(row_len, src);
    clear();
    walk(first + g * UB, len - g * UB, kGroups * UB);
    sum_lane_groups();
    if (g == 0 && f_active) store_unaligned<VEC>(Yf + (size_t)(row0 + src) * feat, acc);
  }
}

}  // namespace
}  // namespace sptir

using namespace sptir;

extern "C" sptir_status_t sptir_spmm_csr(const sptir_csr_t* csr, const float* X, float* Y, int32_t feat,
                                         void* stream_) {
  if (!csr || feat < 1 || csr->n_rows < 0 || csr->n_cols < 0 || csr->nnz < 0) return SPTIR_ERR_INVALID_ARG;
  if (!csr->indptr || (csr->nnz > 0 && (!csr->indices || !csr->values))) return SPTIR_ERR_INVALID_ARG;
  if ((csr->n_cols > 0 && !X) || (csr->n_rows > 0 && !Y)) return SPTIR_ERR_INVALID_ARG;
  const size_t x_bytes = sizeof(float) * (size_t)csr->n_cols * feat, y_bytes = sizeof(float) * (size_t)csr->n_rows * feat;
  if (x_bytes && y_bytes && overlaps(X, x_bytes, Y, y_bytes)) return SPTIR_ERR_INVALID_ARG;
  if (csr->n_rows == 0) return SPTIR_OK;
  Geometry g;
  g.vec = feat >= 4 ? 4 : 1;
  g.lg = feat >= 4 && feat <= 16 ? 4 : 8;
  // A row of X that is not whole 128-byte lines has its tiles across line ends: tiles of 64 floats then touch fewer
  // lines per row than tiles of 32 (41 features on 132,534 rows: 0.217 -> 0.143 ms).  Where X is small enough for
  // L2 the lines are cheap and the narrower lane groups keep more rows in flight (20,000 rows, 41 features: 24 against
  // 27 us); they change over near 8 MB.  (120 graphs: above it the wide tiles are 1.16 times as fast in the mean, 0.74 to 1.6;
  // from 4 to 8 MB the two are alike; below the narrow ones are 1.18 times as fast, 0.67 to 1.8.)
  if (feat > 32 && feat % 32 != 0 && x_bytes > ((size_t)8 << 20)) g.lg = 16;
  g.n_tiles = (feat + g.vec * g.lg - 1) / (g.vec * g.lg);
  // Rows per workgroup: 64, or fewer where workgroups of 64 would leave CUs idle and rows are long enough for a wavefront
  // each (a small dense graph: 4,168 rows, 603,937 entries, 32 features: 43 -> 17 us with 8 rows; 8,382 rows, 1.2 M, 64
  // features: 44 -> 29 with 16).  Short rows want eight of them per wavefront however few there are (10,403 rows of 20
  // entries: 9 us against 14).  On 120 graphs: long rows in few workgroups, 16 rows 1.35 times as fast as 64 (0.9 to 2);
  // long rows in 512 workgroups and more, 64 and 16 alike; short rows, 64 rows 1.18 times as fast as 16 (from 512
  // workgroups on 1.29, below 0.91) and 1.7 times as fast as 8.
  const int64_t n_wg = ((int64_t)csr->n_rows + kCsrRows - 1) / kCsrRows * g.n_tiles;
  const bool dense = csr->nnz >= 40 * (int64_t)csr->n_rows;
  const int rows = !dense || n_wg >= 512 ? kCsrRows : n_wg >= 128 ? 16 : 8;
  if (!plan_tiles(((int64_t)csr->n_rows + rows - 1) / rows, &g)) return SPTIR_ERR_OVERFLOW;
  CsrArgs a;
  a.indptr = csr->indptr; a.indices = csr->indices; a.values = csr->values; a.X = X; a.Y = Y;
  a.n_rows = csr->n_rows; a.feat = feat; a.n_tiles = g.n_tiles; a.map_mode = g.map_mode; a.map_param = g.map_param;
  // Long rows first, by workgroups of their own (up to 512 over all tiles, which look through all rows): a long row that a workgroup
  // in the middle of the grid meets is worked on when the others have ended (169,343 rows, 13,000 entries the longest: 113 -> 104
  // us).  One of them per 128 rows: 160 graphs of 3.5 to 24 entries a row, against none, power-law rows 1.16 times as fast (0.91 to
  // 1.7), in the order of their lengths 3.3 (1.0 to 14), even rows 0.98 (0.9 to 1.05); one per 512 rows 1.08, 3.4 and 0.98.
  // Longer rows are long too often for 512 workgroups (mean of 24 to 100 entries: 0.7 to 1.07).
  const bool long_first = csr->nnz < 24 * (int64_t)csr->n_rows;
  int64_t long_grid = 0;
  if (long_first) {
    Geometry first = g;
    a.long_units = (int32_t)std::max<int64_t>(1, std::min<int64_t>(512 / g.n_tiles, ((int64_t)csr->n_rows + 127) / 128));
    if (!plan_tiles(a.long_units, &first)) return SPTIR_ERR_OVERFLOW;
    long_grid = (first.grid + 7) / 8 * 8;
    a.long_grid = (uint32_t)long_grid; a.long_mode = first.map_mode; a.long_param = first.map_param;
    if (long_grid + g.grid > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  }
  dim3 grid((unsigned)(long_grid + g.grid)), block(512);
  hipStream_t stream = (hipStream_t)stream_;
  auto launch = [&](auto n) {
    constexpr int kRows = decltype(n)::value;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, a); };
    auto shape = [&](auto first) {
      constexpr bool kFirst = decltype(first)::value;
      if (g.vec == 1) go(k_spmm_csr<1, 8, kRows, kFirst>);
      else if (g.lg == 4) go(k_spmm_csr<4, 4, kRows, kFirst>);
      else if (g.lg == 16) go(k_spmm_csr<4, 16, kRows, kFirst>);
      else go(k_spmm_csr<4, 8, kRows, kFirst>);
    };
    if (kRows == kCsrRows && long_first) shape(std::integral_constant<bool, kRows == kCsrRows>{});
    else shape(std::false_type{});
  };
  if (rows == kCsrRows) launch(std::integral_constant<int, kCsrRows>{});
  else if (rows == 16) launch(std::integral_constant<int, 16>{});
  else launch(std::integral_constant<int, 8>{});
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}
