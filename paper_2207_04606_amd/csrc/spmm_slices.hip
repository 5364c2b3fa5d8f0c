// SpMM of the long rows of a hyb handle, from column slices in LDS.
//
// A gathered row of X costs L1 time wherever it comes from: 32 TB/s of them arrive from an XCD's L2, 28 in k_spmm_heavy.  LDS
// delivers random rows of 128 bytes at 76 TB/s, of 64 at 70, of 32 at 58.  A row of A that has entries in every slice of columns
// that fits LDS can take its rows of X from there.
//
// Mapping.  A slice is kSliceCols columns, their features a tile of 16 (64 bytes: narrower tiles hold more columns, so that a
// row has more of its entries in one slice, but lose more to bank conflicts).  The long rows, longest first, are cut into blocks of 16, one
// row per lane group of four lanes, and the blocks into panels of up to 128.  A workgroup takes a panel, a tile and a range of
// slices; a wavefront takes every 16th block of the panel and keeps the sums of its rows in registers from the first slice to
// the last, so that what it leaves, a partial sum per row and range, is a hundredth of what it gathers.  The panel is as large as
// it has to be for the gathers of a slice to outweigh the loading of it.
//
// The entries lie in steps: the next eight columns (16 bits each) of the 16 rows of a block, a load of 16 bytes per lane group.
// The rows of a block are of like length, so they have about as many steps in a slice; what the shorter ones lack points at a
// row of zeros after the slice's last (a fifth of what is read; the last step may have half).  The steps of a wavefront follow each
// other from slice to slice, whatever the block, and are asked for two steps ahead.
//
// 232,965 rows, 114.6 M entries, 128 features: the call 2.39 -> 1.80 ms.  87 M entries in 0.98 ms, 46 TB/s of gathered rows (28.5
// in k_spmm_heavy; 1.2 times as many slots), vector ALU issuing 68 % of it, bank conflicts 34 %; the rest is loading slices and
// wavefronts that wait there for the last.
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_slice_bounds.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

constexpr int kThreads = 1024, kWavesHere = kThreads / 64;
constexpr int kLanes = 4, kTileFloats = 4 * kLanes;     // a lane group and its features
constexpr int kBlockRows = 64 / kLanes;
constexpr int kMaxBlocksPerWave = 8;                    // sums: 4 registers each
constexpr int kMaxPanelBlocks = kWavesHere * kMaxBlocksPerWave;
constexpr int kAhead = 2;                               // steps between the request for one and its use
// Most slots walked per entry (8 x 16 a step).  A block takes as many steps in a slice as its longest row there, and its rows have
// nothing in common but their length: 1.1 to 1.45 where columns are close to uniform or fall in popularity, 4 to 9 where rows
// have 30 to 80 % of their entries in one of 50 ranges of columns (232,965 rows, 80 %: 2.1 ms a product without slices, 6.2 with).
// At 2 the entries take as many bytes as in the stream.  80 drawn graphs, 3 to 25 % of a row's entries in such a range or all in
// a band, products against no slices: up to 1.5 slots 1.65 times as fast (0.86 to 3.2), to 2 1.49 (0.93 to 3.0; 1.0 and more from 12 M
// long entries on), to 2.5 1.33 (0.79 to 3.2), to 3.7 1.06 (0.6 to 2.5).
constexpr double kMostSlotsPerEntry = 2.0;
// Nor where one slice has more than so many times the mean's steps: a panel is one workgroup there, and panels small enough for all
// CUs to have some load every other slice for little.  80 graphs of 13 M entries and more, columns skewed, hot in a range, in bands or
// uniform, products against no slices: 1.31 times as fast up to 16 (0.91 to 2.8), beyond 0.80 and 0.91.
constexpr double kMostOfMean = 16.0;
constexpr size_t kSliceLds = sizeof(float4) * kLanes * (kSliceCols + 1);

struct Unit {
  int32_t first;          // of the panel's words of step_of
  int32_t blocks_per_wave, n_blocks;
  int32_t slice0, slice1;
  int32_t partial0;       // partial-sum row of the panel's first row in this range
};

struct SliceArgs {
  const Unit* units;
  const int32_t* step_of;  // [panel][wavefront][slice][block of the wavefront]: its first step << 1 | its last step has half
  const uint4* cols;       // [step][16]
  const float4* vals;      // [step][16][2]; NULL: every entry counts 1
  const float* X;
  float* partial;
  int32_t n_units, n_slices, n_cols, feat;
  int32_t feat0, n_tiles, partial_feat;
};

// Byte offset in LDS of a lane's floats of the column in one half of w (the compiler takes two instructions for it)
__device__ __forceinline__ unsigned row_at(unsigned w, int upper, unsigned lane_bytes) {
  static_assert(sizeof(float4) * kLanes == 64, "the factor below");
  unsigned at;
  if (upper) asm("v_mad_u32_u16 %0, %1, 64, %2 op_sel:[1,0,0,0]" : "=v"(at) : "v"(w), "v"(lane_bytes));
  else asm("v_mad_u32_u16 %0, %1, 64, %2" : "=v"(at) : "v"(w), "v"(lane_bytes));
  return at;
}

template <bool UNIT>
__global__ __launch_bounds__(kThreads) void k_spmm_slices(SliceArgs a) {
  extern __shared__ __align__(16) float4 xs[];  // [kSliceCols + 1][kLanes]
  const int lane = threadIdx.x & 63, g = lane / kLanes, fl = lane & (kLanes - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // the tiles of a unit go to one XCD, next to each other: they read the same steps
  const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int unit_id = q / a.n_tiles * 8 + x, tile = q % a.n_tiles;
  if (unit_id >= a.n_units) return;
  const Unit u = a.units[unit_id];
  const int f_tile = a.feat0 + tile * kTileFloats;
  if (threadIdx.x < kLanes) xs[kSliceCols * kLanes + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);

  const int words = u.blocks_per_wave * a.n_slices;  // of step_of, per wavefront
  const int32_t* step_of = a.step_of + u.first + wave * words;
  auto word = [&](int i) { return __builtin_amdgcn_readfirstlane(step_of[i]); };
  int at = word(u.slice0 * u.blocks_per_wave) >> 1;  // the step that is worked on; the array ends in kAhead spare ones
  uint4 ahead[kAhead];
  float4 v_ahead[UNIT ? 1 : kAhead][2];
  auto request = [&](int step, uint4& c, float4 (&v)[2]) {
    c = (a.cols + (size_t)step * kBlockRows)[g];
    if constexpr (!UNIT) {
      const float4* p = a.vals + (size_t)step * kBlockRows * 2;
      v[0] = p[2 * g]; v[1] = p[2 * g + 1];
    }
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i) request(at + i, ahead[i], v_ahead[UNIT ? 0 : i]);
  const unsigned lane_bytes = 16u * fl;
  float total[kMaxBlocksPerWave][4];
#pragma unroll
  for (int r = 0; r < kMaxBlocksPerWave; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) total[r][e] = 0.f;

  // Rows of X of a slice, through registers to LDS.  (Asked for while the slice before is worked on they spill: twice as long.)
  constexpr int kStaged = (kSliceCols * kLanes + kThreads - 1) / kThreads;
  float4u staged[kStaged];
  const int q_mine = (int)threadIdx.x & (kLanes - 1), f_mine = f_tile + 4 * q_mine;
  auto n_cols_of = [&](int s) { return (int)min((int64_t)kSliceCols, (int64_t)a.n_cols - (int64_t)s * kSliceCols); };
  auto get_slice = [&](int s, float4u (&v)[kStaged]) {
    const int n = n_cols_of(s);
    const float* src = a.X + (size_t)s * kSliceCols * a.feat;
    if (a.feat >= 4) {
      // (a row's last float4 is its last four floats, whatever its number; past the end it is never written to Y)
      src += min(f_mine, a.feat - 4);
#pragma unroll
      for (int k = 0; k < kStaged; ++k)
        v[k] = *reinterpret_cast<const float4u*>(src + (size_t)min(((int)threadIdx.x + k * kThreads) / kLanes, n - 1) * a.feat);
    } else {
#pragma unroll
      for (int k = 0; k < kStaged; ++k) {
        const float* p = src + (size_t)min(((int)threadIdx.x + k * kThreads) / kLanes, n - 1) * a.feat;
        v[k] = float4u{0.f, 0.f, 0.f, 0.f};
        if (f_mine < a.feat) v[k].x = p[f_mine];
        if (f_mine + 1 < a.feat) v[k].y = p[f_mine + 1];
        if (f_mine + 2 < a.feat) v[k].z = p[f_mine + 2];
      }
    }
  };
  auto put_slice = [&](int s, const float4u (&v)[kStaged]) {
    const int n = n_cols_of(s) * kLanes;
#pragma unroll
    for (int k = 0; k < kStaged; ++k) {
      const int i = (int)threadIdx.x + k * kThreads;
      if (i < n) xs[i] = make_float4(v[k].x, v[k].y, v[k].z, v[k].w);
    }
  };
  for (int s = u.slice0; s < u.slice1; ++s) {
    int bound[kMaxBlocksPerWave + 1];
#pragma unroll
    for (int r = 0; r <= kMaxBlocksPerWave; ++r) bound[r] = word(s * u.blocks_per_wave + min(r, u.blocks_per_wave));
    get_slice(s, staged);  // (wavefronts that are done load while others work: with the load after the barrier the call of the header took 1.82 ms)
    __syncthreads();       // (the slice before is no longer read)
    put_slice(s, staged);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kMaxBlocksPerWave; ++r) {
      if (r >= u.blocks_per_wave) continue;
      // the entries of one row and slice, in two running sums (a sum over all slices at once would be longer and less exact)
      float sum[2][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[0][e] = sum[1][e] = 0.f;
      auto step = [&](int n_here) {
        const uint4 c = ahead[0];
        float v[8];
        if constexpr (!UNIT) {
          const float4 v0 = v_ahead[0][0], v1 = v_ahead[0][1];
          v[0] = v0.x; v[1] = v0.y; v[2] = v0.z; v[3] = v0.w; v[4] = v1.x; v[5] = v1.y; v[6] = v1.z; v[7] = v1.w;
        }
#pragma unroll
        for (int i = 0; i + 1 < kAhead; ++i) {
          ahead[i] = ahead[i + 1];
          if constexpr (!UNIT) { v_ahead[i][0] = v_ahead[i + 1][0]; v_ahead[i][1] = v_ahead[i + 1][1]; }
        }
        request(at + kAhead, ahead[kAhead - 1], v_ahead[UNIT ? 0 : kAhead - 1]);
#pragma unroll
        for (int i = 0; i < n_here; ++i) {
          const unsigned w = i < 2 ? c.x : (i < 4 ? c.y : (i < 6 ? c.z : c.w));
          const float4 xv = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(xs) + row_at(w, i & 1, lane_bytes));
          float (&acc)[4] = sum[i & 1];
          if constexpr (UNIT) {
            acc[0] += xv.x; acc[1] += xv.y; acc[2] += xv.z; acc[3] += xv.w;
          } else {
            acc[0] = fmaf(v[i], xv.x, acc[0]); acc[1] = fmaf(v[i], xv.y, acc[1]);
            acc[2] = fmaf(v[i], xv.z, acc[2]); acc[3] = fmaf(v[i], xv.w, acc[3]);
          }
        }
        ++at;
      };
      const int half = bound[r] & 1, whole_end = (bound[r + 1] >> 1) - half;
      while (at < whole_end) step(8);
      if (half) step(4);
#pragma unroll
      for (int e = 0; e < 4; ++e) total[r][e] += sum[0][e] + sum[1][e];
    }
  }
  float* out = a.partial + (size_t)u.partial0 * a.partial_feat + tile * kTileFloats + fl * 4;
#pragma unroll
  for (int r = 0; r < kMaxBlocksPerWave; ++r) {
    const int block = r * kWavesHere + wave;
    if (block < u.n_blocks)
      *reinterpret_cast<float4*>(out + (size_t)(block * kBlockRows + g) * a.partial_feat) =
          make_float4(total[r][0], total[r][1], total[r][2], total[r][3]);
  }
}

struct Panel {
  int32_t block0, n_blocks, blocks_per_wave;
  int32_t first;      // words of step_of before it
  int32_t partial0;   // partial-sum rows before it
  int32_t n_ranges;
};

// Y[r] = (row_val[r] *) the partial sums of long row r, range after range: the row has no other entries
__global__ __launch_bounds__(256) void k_slice_sums(const int32_t* __restrict__ rows, int32_t n_long,
                                                    const Panel* __restrict__ panels, const int32_t* __restrict__ panel_of,
                                                    const float* __restrict__ partial, const float* __restrict__ row_val, float* Y,
                                                    int32_t feat, int32_t feat0, int32_t width, int32_t partial_feat) {
  const int per_row = (width + 3) / 4, in_wg = 256 / per_row;
  const int row_here = (int)threadIdx.x / per_row, f = ((int)threadIdx.x % per_row) * 4;
  const int64_t p = (int64_t)blockIdx.x * in_wg + row_here;
  if (row_here >= in_wg || p >= n_long) return;
  const int r = rows[p];
  const Panel panel = panels[panel_of[p / kBlockRows]];
  const size_t step = (size_t)panel.n_blocks * kBlockRows * partial_feat;
  const float* src = partial + ((size_t)panel.partial0 + (size_t)(p - (int64_t)panel.block0 * kBlockRows)) * partial_feat + f;
  float acc[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[k][e] = 0.f;
  for (int i = 0; i < panel.n_ranges; i += 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k < panel.n_ranges) {
        float v[4];
        load_vec<4>(v, src + (size_t)(i + k) * step);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[k][e] += v[e];
      }
  }
  const float scale = row_val ? row_val[r] : 1.f;
  float out[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = scale * ((acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]));
  const int f_nominal = feat0 + f;
  const int f_here = feat >= 4 ? min(f_nominal, feat - 4) : 0, again = f_nominal - f_here;
  float* y = Y + (size_t)r * (size_t)feat + f_here;
  if (again == 0 && feat >= 4) {
    store_unaligned<4>(y, out);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e >= again && f_here + e < feat) y[e] = out[e];
  }
}

// ------------------------------------------------------------------- build
// A workgroup per block of rows: count[block * n_slices + s] = half steps in slice s, those of its longest row;
// block_steps[block]: its steps (in host memory)
__global__ __launch_bounds__(256) void k_count_steps(int32_t n_slices, int32_t room, const int32_t* __restrict__ bound, int32_t* count,
                                                     int32_t* block_steps) {
  __shared__ int32_t total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  const int row = (int)threadIdx.x & (kBlockRows - 1), s_here = (int)threadIdx.x / kBlockRows;
  const int64_t p = (int64_t)blockIdx.x * kBlockRows + row;
  int mine = 0;
  for (int s0 = 0; s0 < n_slices; s0 += 256 / kBlockRows) {
    const int s = s0 + s_here;
    int steps = s < n_slices ? (bound[(int64_t)(s + 1) * room + p] - bound[(int64_t)s * room + p] + 3) / 4 : 0;  // (halves)
#pragma unroll
    for (int d = 1; d < kBlockRows; d <<= 1) steps = max(steps, __shfl_xor(steps, d, kBlockRows));
    if (row == 0 && s < n_slices) {
      count[(int64_t)blockIdx.x * n_slices + s] = steps;
      mine += (steps + 1) / 2;
    }
  }
  if (mine) atomicAdd(&total, mine);
  __syncthreads();
  if (threadIdx.x == 0) block_steps[blockIdx.x] = total;
}

// A workgroup per slice: steps of all blocks in it
__global__ __launch_bounds__(256) void k_slice_steps(int32_t n_slices, int32_t n_blocks, const int32_t* __restrict__ count,
                                                     int32_t* slice_steps) {
  __shared__ int32_t total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  int mine = 0;
  for (int b = threadIdx.x; b < n_blocks; b += 256) mine += (count[(int64_t)b * n_slices + blockIdx.x] + 1) / 2;
  if (mine) atomicAdd(&total, mine);
  __syncthreads();
  if (threadIdx.x == 0) slice_steps[blockIdx.x] = total;
}

__device__ __forceinline__ int64_t word_of(const Panel& p, int block, int s, int n_slices) {
  const int b = block - p.block0;
  return (int64_t)p.first + ((int64_t)(b % kWavesHere) * n_slices + s) * p.blocks_per_wave + b / kWavesHere;
}

__host__ __device__ __forceinline__ int64_t panel_words_end(const Panel& p, int n_slices) {
  return (int64_t)p.first + (int64_t)kWavesHere * p.blocks_per_wave * n_slices;
}

// the numbers of steps to their words, and none to those of the wavefronts that have a block less
__global__ __launch_bounds__(256) void k_order_steps(int64_t n, int32_t n_slices, const Panel* __restrict__ panels,
                                                     const int32_t* __restrict__ panel_of, const int32_t* __restrict__ count,
                                                     int32_t* first_step) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int block = (int)(i / n_slices), s = (int)(i % n_slices);
  const Panel p = panels[panel_of[block]];
  first_step[word_of(p, block, s, n_slices)] = (count[i] + 1) / 2;
  if (block != p.block0 + p.n_blocks - 1) return;
  for (int b = block + 1; b < p.block0 + p.blocks_per_wave * kWavesHere; ++b) first_step[word_of(p, b, s, n_slices)] = 0;
}

template <typename T>
__device__ __forceinline__ void load_eight(T (&out)[8], const T* p) {
  float a[4], b[4];
  load_unaligned<4>(a, reinterpret_cast<const float*>(p));
  load_unaligned<4>(b, reinterpret_cast<const float*>(p) + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[i] = __builtin_bit_cast(T, a[i]);
    out[4 + i] = __builtin_bit_cast(T, b[i]);
  }
}

struct FillArgs {
  int64_t n, nnz, n_steps;      // n: blocks x slices
  int32_t n_slices, room, n_long;
  const Panel* panels;
  const int32_t *panel_of, *count, *first_step, *bound, *order, *indices;
  const float* values;
  int32_t *step_of, *rows;
  uint4* cols;
  float4* vals;                 // NULL: none
};

// The steps of a (block, slice) by a wavefront, four steps of its 16 rows at a time, and its word
__global__ __launch_bounds__(256) void k_fill_steps(FillArgs a) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t i = t / 64;
  if (t < kAhead * kBlockRows) {  // what the loops read ahead past the last step
    const size_t at = (size_t)a.n_steps * kBlockRows + t;
    const unsigned c = (unsigned)kSliceCols | (unsigned)kSliceCols << 16;
    a.cols[at] = make_uint4(c, c, c, c);
    if (a.vals) a.vals[2 * at] = a.vals[2 * at + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (i >= a.n) return;
  const int row = (int)(t % kBlockRows), turn = (int)(t % 64) / kBlockRows;
  // (slices fastest: the pieces of a row follow each other in memory)
  const int64_t n_blocks = a.n / a.n_slices;
  const int s = (int)(i % a.n_slices), block = (int)(i / a.n_slices);
  const int halves = a.count[(int64_t)block * a.n_slices + s], steps = (halves + 1) / 2;
  const int64_t p = (int64_t)block * kBlockRows + row;
  const int lo = a.bound[(int64_t)s * a.room + p], len = a.bound[(int64_t)(s + 1) * a.room + p] - lo;
  const Panel panel = a.panels[a.panel_of[block]];
  const int64_t word = word_of(panel, block, s, a.n_slices);
  const int64_t first = a.first_step[word];
  if (t % 64 == 0) {
    a.step_of[word] = (int32_t)(first << 1) | (halves & 1);
    if (block == panel.block0 + panel.n_blocks - 1)  // also for the wavefronts that have a block less
      for (int b = block + 1; b < panel.block0 + panel.blocks_per_wave * kWavesHere; ++b) {
        const int64_t w = word_of(panel, b, s, a.n_slices);
        a.step_of[w] = a.first_step[w] << 1;
      }
    if (t == 0) a.step_of[(int64_t)panel_words_end(a.panels[a.panel_of[n_blocks - 1]], a.n_slices)] = (int32_t)(a.n_steps << 1);
  }
  if (s == 0 && turn == 0 && p < a.n_long) a.rows[p] = a.order[p];
  const bool inside = (int64_t)lo + (int64_t)steps * 8 <= a.nnz;
  for (int j = turn; j < steps; j += 64 / kBlockRows) {
    const int e0 = lo + j * 8, left = len - j * 8;
    int c[8];
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = 0.f;
    if (inside) {  // (16 bytes at a time, into the next row if need be: L1 does not hold the lines of a wavefront's 64 pieces)
      load_eight(c, a.indices + e0);
      if (a.vals) load_eight(v, a.values + e0);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        c[k] = k < left ? a.indices[e0 + k] : 0;
        if (a.vals && k < left) v[k] = a.values[e0 + k];
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      c[k] = k < left ? c[k] - s * kSliceCols : kSliceCols;
      v[k] = k < left ? v[k] : 0.f;
    }
    const size_t at = (size_t)(first + j) * kBlockRows + row;
    a.cols[at] = make_uint4((unsigned)(c[0] | c[1] << 16), (unsigned)(c[2] | c[3] << 16), (unsigned)(c[4] | c[5] << 16),
                            (unsigned)(c[6] | c[7] << 16));
    if (a.vals) {
      a.vals[2 * at] = make_float4(v[0], v[1], v[2], v[3]);
      a.vals[2 * at + 1] = make_float4(v[4], v[5], v[6], v[7]);
    }
  }
}

template <bool UNIT>
void launch_gather(const SliceArgs& a, unsigned grid, hipStream_t stream) {
  auto* kernel = &k_spmm_slices<UNIT>;
  static OncePerDevice allowed;
  allow_dynamic_lds(reinterpret_cast<const void*>(kernel), kSliceLds, allowed);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), kSliceLds, stream, a);
}

size_t up(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

}  // namespace

int64_t slice_min_degree(int32_t n_cols) { return std::max<int64_t>(kChunkSlots, (int64_t)kMinSlicePiece * n_cols / kSliceCols); }

// First part of the build: everything up to the numbers of steps, which land in b->host; only enqueues work.
sptir_status_t spmm_slices_count(SpmmSliceBuild* b, const sptir_csr_t* csr, int32_t min_deg, int32_t n_long, int64_t longest,
                                 sptir_alloc_fn alloc, void* actx, hipStream_t stream) {
  b->n_long = n_long;
  b->n_blocks = (n_long + kBlockRows - 1) / kBlockRows;
  b->n_slices = (int32_t)(((int64_t)csr->n_cols + kSliceCols - 1) / kSliceCols);
  const size_t room = (size_t)b->n_blocks * kBlockRows, words = (size_t)b->n_blocks * b->n_slices;
  if (words * 64 > (size_t)0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  const size_t o_bound = up(sizeof(int32_t) * (size_t)csr->n_rows), o_count = o_bound + up(sizeof(int32_t) * (words * kBlockRows + room));
  const size_t o_sort = o_count + up(sizeof(int32_t) * words);
  b->temporary = scratch_alloc(o_sort + order_rows_scratch(csr->n_rows), alloc, actx, stream);
  b->host = pinned_acquire(sizeof(int32_t) * ((size_t)b->n_blocks + b->n_slices));
  if (!b->temporary || !b->host.p) return SPTIR_ERR_ALLOC;
  char* t = (char*)b->temporary;
  b->order = (int32_t*)t; b->bound = (int32_t*)(t + o_bound); b->count = (int32_t*)(t + o_count);
  int32_t* block_steps = (int32_t*)b->host.p;
  const sptir_status_t st = order_rows_by_class(csr->indptr, csr->n_rows, min_deg, longest, b->order, t + o_sort, stream);
  if (st != SPTIR_OK) return st;
  constexpr int kTile = 32;
  hipLaunchKernelGGL(k_slice_bounds<kTile>, dim3(slice_bounds_workgroups<kTile>(b->n_slices, (int64_t)room)), dim3(kBoundsBlock), 0,
                     stream, b->n_slices, kSliceCols, n_long, (int32_t)room, b->order, csr->indptr, csr->indices, b->bound);
  hipLaunchKernelGGL(k_count_steps, dim3((unsigned)b->n_blocks), dim3(256), 0, stream, b->n_slices, (int32_t)room, b->bound, b->count,
                     block_steps);
  hipLaunchKernelGGL(k_slice_steps, dim3((unsigned)b->n_slices), dim3(256), 0, stream, b->n_slices, b->n_blocks, b->count,
                     block_steps + b->n_blocks);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

// The steps that were counted, once the stream has been waited for
int64_t spmm_slices_steps(const SpmmSliceBuild& b) {
  const int32_t* block_steps = (const int32_t*)b.host.p;
  int64_t n_steps = 0;
  for (int32_t i = 0; i < b.n_blocks; ++i) n_steps += block_steps[i];
  return n_steps;
}

// The share of all steps that the slice with most of them has
static double hottest_slice(const SpmmSliceBuild& b, int64_t n_steps) {
  const int32_t* slice_steps = (const int32_t*)b.host.p + b.n_blocks;
  return *std::max_element(slice_steps, slice_steps + b.n_slices) / (double)std::max<int64_t>(1, n_steps);
}

bool spmm_slices_even(const SpmmSliceBuild& b, int64_t long_nnz) {
  const int64_t n_steps = spmm_slices_steps(b);
  return (double)n_steps * (8 * kBlockRows) <= kMostSlotsPerEntry * (double)long_nnz &&
         hottest_slice(b, n_steps) * b.n_slices <= kMostOfMean;
}

// Then: panels, units and the handle's memory.  Host work only; where it does not succeed nothing has been enqueued.
sptir_status_t spmm_slices_plan(SpmmSliceBuild* b, int32_t feat_hint, bool with_values, SpmmSlices* out, sptir_alloc_fn alloc,
                                void* actx, hipStream_t stream) try {
  const int32_t* block_steps = (const int32_t*)b->host.p;
  const int32_t* slice_steps = block_steps + b->n_blocks;
  const int64_t n_steps = spmm_slices_steps(*b);
  if (n_steps + kAhead > 0x3FFFFFFF) return SPTIR_ERR_OVERFLOW;
  // In units of what a step costs where LDS binds (8 KB): loading a slice, and the steps of a panel in a slice that outweigh it,
  // fewer where there would not be enough units for every CU (9,306 rows, 4.6 M entries, 32 features: 81 us with 2048, 34 with this)
  constexpr double kLoad = 64.0, kMostWorth = 2048.0, kLeastWorth = 128.0;
  const double tiles = std::max(1, ((feat_hint > 0 ? std::min(feat_hint, kPartialFeat) : 64) + kTileFloats - 1) / kTileFloats);
  const double worth = std::max(kLeastWorth, std::min(kMostWorth, (double)n_steps * tiles / (256.0 * 4.0)));
  // ... and no more in the hottest slice than half of what a CU has to do.  (79 of those graphs against panels without this limit:
  // 1.09 times as fast in the mean, 0.88 to 1.8; uniform columns alike.)
  const double panel_most = std::min(worth * b->n_slices, 0.5 * n_steps * tiles / 256.0 / hottest_slice(*b, n_steps));
  std::vector<Panel> panels;
  std::vector<int32_t> panel_of((size_t)b->n_blocks);
  std::vector<double> panel_steps;
  int64_t words = 0;
  for (int32_t at = 0; at < b->n_blocks;) {
    Panel p{at, 0, 0, (int32_t)words, 0, 0};
    double steps = 0;
    while (at < b->n_blocks && p.n_blocks < kMaxPanelBlocks &&
           (p.n_blocks % kWavesHere != 0 || p.n_blocks == 0 || steps < panel_most)) {
      steps += block_steps[at];
      panel_of[(size_t)at] = (int32_t)panels.size();
      ++at; ++p.n_blocks;
    }
    p.blocks_per_wave = (p.n_blocks + kWavesHere - 1) / kWavesHere;
    words += (int64_t)kWavesHere * p.blocks_per_wave * b->n_slices;
    panels.push_back(p);
    panel_steps.push_back(steps);
  }
  if (words + 1 > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  // Units: ranges of slices of a panel.  A third of what is left for a CU, over the feature tiles of a call, at a time: the last
  // ones are small, and the CUs end together.  (Units of one size leave up to one of them idle at the end: 5 a CU 1.84 ms.)
  double left = 0;
  for (double s : panel_steps) left += s + kLoad * b->n_slices;
  struct Ranked { double cost; Unit u; };
  std::vector<Ranked> ranked;
  int64_t partial_rows = 0;
  for (size_t i = panels.size(); i-- > 0;) {  // (large panels, whose partial sums are many, in few and large units)
    Panel& p = panels[i];
    p.partial0 = (int32_t)partial_rows;
    for (int32_t s = 0; s < b->n_slices;) {
      const double most = left * tiles / (256.0 * 3.0);
      double here = 0;
      const int32_t s0 = s;
      do {
        here += kLoad + (n_steps > 0 ? panel_steps[i] * slice_steps[s] / (double)n_steps : 0.0);
        ++s;
      } while (s < b->n_slices && here + kLoad + panel_steps[i] * slice_steps[s] / (double)std::max<int64_t>(1, n_steps) <= most);
      left -= here;
      ranked.push_back({here, Unit{p.first, p.blocks_per_wave, p.n_blocks, s0, s, (int32_t)partial_rows}});
      partial_rows += (int64_t)p.n_blocks * kBlockRows;
      ++p.n_ranges;
      if (partial_rows > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
    }
  }
  std::stable_sort(ranked.begin(), ranked.end(), [](const Ranked& x, const Ranked& y) { return x.cost > y.cost; });
  // ---- the handle's arrays, and the tables through pinned memory
  const size_t room = (size_t)b->n_blocks * kBlockRows;
  const size_t n_words = scan_room(words);
  const size_t table_sizes[] = {sizeof(Unit) * ranked.size(), sizeof(Panel) * panels.size(), sizeof(int32_t) * panel_of.size()};
  size_t table_bytes = 0;
  for (size_t t : table_sizes) table_bytes += up(t);
  const size_t steps_room = (size_t)n_steps + kAhead;
  const size_t o_rows = table_bytes, o_words = o_rows + up(sizeof(int32_t) * room), o_first = o_words + up(sizeof(int32_t) * (size_t)(words + 1));
  const size_t o_seq = o_first + up(sizeof(int32_t) * n_words);
  const size_t o_cols = o_seq + up(sizeof(int32_t) * (n_words / kScanSeq + 1));
  const size_t o_vals = o_cols + up(sizeof(uint4) * kBlockRows * steps_room);
  const size_t o_partial = o_vals + (with_values ? up(2 * sizeof(float4) * kBlockRows * steps_room) : 0);
  const size_t bytes = o_partial + up(sizeof(float) * kPartialFeat * (size_t)partial_rows);
  size_t got = 0;
  char* base = (char*)scratch_alloc(bytes, alloc, actx, stream, &got);
  if (!base) return SPTIR_ERR_ALLOC;
  out->blob = base; out->device_bytes = got;
  b->tables = pinned_acquire(table_bytes);
  if (!b->tables.p) return SPTIR_ERR_ALLOC;
  char* t = b->tables.p;
  for (size_t i = 0; i < ranked.size(); ++i) memcpy(t + sizeof(Unit) * i, &ranked[i].u, sizeof(Unit));
  memcpy(t + up(table_sizes[0]), panels.data(), table_sizes[1]);
  memcpy(t + up(table_sizes[0]) + up(table_sizes[1]), panel_of.data(), table_sizes[2]);
  b->n_steps = n_steps; b->words = words; b->table_bytes = table_bytes;
  b->first_step = (int32_t*)(base + o_first); b->seq_base = (int32_t*)(base + o_seq);
  out->n_long = b->n_long; out->n_units = (int32_t)ranked.size(); out->n_slices = b->n_slices;
  out->units = base; out->panels = base + up(table_sizes[0]);
  out->panel_of = (const int32_t*)(base + up(table_sizes[0]) + up(table_sizes[1]));
  out->rows = (int32_t*)(base + o_rows); out->step_of = (int32_t*)(base + o_words);
  out->cols = (uint4*)(base + o_cols); out->vals = with_values ? (float4*)(base + o_vals) : nullptr;
  out->partial = (float*)(base + o_partial);
  return SPTIR_OK;
} catch (const std::bad_alloc&) {  // (the tables of units and panels)
  return SPTIR_ERR_ALLOC;
}

// Last: the contents of the handle's arrays.  The host side of `b` has to stay until the stream has drained.
sptir_status_t spmm_slices_fill(const SpmmSliceBuild& b, const sptir_csr_t* csr, const SpmmSlices& s, hipStream_t stream) {
  SPTIR_HIP(hipMemcpyAsync(s.blob, b.tables.p, b.table_bytes, hipMemcpyHostToDevice, stream));
  FillArgs f;
  f.n = (int64_t)b.n_blocks * b.n_slices; f.nnz = csr->nnz; f.n_steps = b.n_steps;
  f.n_slices = b.n_slices; f.room = b.n_blocks * kBlockRows; f.n_long = b.n_long;
  f.panels = (const Panel*)s.panels; f.panel_of = s.panel_of; f.count = b.count; f.first_step = b.first_step; f.bound = b.bound;
  f.order = b.order; f.indices = csr->indices; f.values = csr->values;
  f.step_of = s.step_of; f.rows = s.rows; f.cols = s.cols; f.vals = s.vals;
  hipLaunchKernelGGL(k_order_steps, dim3((unsigned)((f.n + 255) / 256)), dim3(256), 0, stream, f.n, b.n_slices, f.panels,
                     f.panel_of, b.count, b.first_step);
  if (b.words <= kScanOneMost) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanThreads), 0, stream, b.first_step, (int32_t)b.words);
  } else {
    const sptir_status_t st = device_exclusive_scan(b.first_step, b.words, b.seq_base, stream);
    if (st != SPTIR_OK) return st;
  }
  hipLaunchKernelGGL(k_fill_steps, dim3((unsigned)((f.n * 64 + 255) / 256)), dim3(256), 0, stream, f);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

void spmm_slices_done(SpmmSliceBuild* b, sptir_free_fn free_, void* actx) {
  scratch_free(b->temporary, free_, actx);
  pinned_release(b->host);
  pinned_release(b->tables);
  *b = SpmmSliceBuild();
}

// features feat0 .. feat0 + width - 1 (at most kPartialFeat of them): the launch that gathers, the launch that adds up
sptir_status_t spmm_slices_gather(const SpmmSlices& s, int32_t n_cols, const float* X, int32_t feat, int32_t feat0, int32_t width,
                                  hipStream_t stream) {
  SliceArgs a;
  a.units = (const Unit*)s.units; a.step_of = s.step_of; a.cols = s.cols; a.vals = s.vals; a.X = X; a.partial = s.partial;
  a.n_units = s.n_units; a.n_slices = s.n_slices; a.n_cols = n_cols; a.feat = feat; a.feat0 = feat0;
  a.n_tiles = (width + kTileFloats - 1) / kTileFloats; a.partial_feat = a.n_tiles * kTileFloats;
  const int64_t grid = ((int64_t)s.n_units + 7) / 8 * 8 * a.n_tiles;
  if (grid > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  if (s.vals) launch_gather<false>(a, (unsigned)grid, stream);
  else launch_gather<true>(a, (unsigned)grid, stream);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

sptir_status_t spmm_slices_add(const SpmmSlices& s, const float* row_val, float* Y, int32_t feat, int32_t feat0, int32_t width,
                               hipStream_t stream) {
  const int n_tiles = (width + kTileFloats - 1) / kTileFloats;
  const int in_wg = 256 / ((width + 3) / 4);
  hipLaunchKernelGGL(k_slice_sums, dim3((unsigned)((s.n_long + in_wg - 1) / in_wg)), dim3(256), 0, stream, s.rows, s.n_long,
                     (const Panel*)s.panels, s.panel_of, s.partial, row_val, Y, feat, feat0, width, n_tiles * kTileFloats);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

}  // namespace sptir
