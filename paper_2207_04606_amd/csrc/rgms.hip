// Relational gather-matmul-scatter (RGMS, section 4.4 of arXiv 2207.04606):
//     Y[i,l] = sum_r sum_j sum_k A[r,i,j] * X[j,k] * W[r,k,l].
// The paper decomposes every relation's matrix into hyb(1, 5), gathers the
// rows of X, multiplies by W[r] on the matrix cores and scatters into Y, all in
// one kernel, so that T[r] = X W[r] never exists in memory.
//
// Here the kernel is stationary in Y instead of in r.  A arrives as one CSR
// over stacked rows r*n + i.  Rows of Y are cut into blocks; a
// workgroup owns a block, keeps its rows of Y in LDS, walks the block's pairs
// (r, i) relation after relation and writes Y once.  The scatter of the
// relation-stationary order (a float atomic per element of every pair's product
// row, at L2) was what bound it; over 250 graphs and feature sizes it took 1.22 times as long as a first kernel in this one.
//
// A *piece* is up to 4 entries of one (relation, row) pair, a *quad* four pieces of one relation in one block, a *tile*
// up to four quads.  The pieces of a (relation, block) are sorted by length, so that the pieces of a quad are alike, and
// the entries are stored in *steps* of four, one for each piece of a quad.  Pieces of one pair lie in the same place of two or four quads of a
// tile, as far as they fill tiles, and meet before the product: a pair of many entries is multiplied by W[r] once for sixteen or eight of
// them.  (Once for four: 20,000 rows, 20 relations, 3.2 M entries, 32 x 256 features 265 -> 203 us, 64 x 128 249 -> 196, 32 x 32 52 -> 46; with
// pieces of eight entries, for which W[r] is read half as often, the kernel of 16-row products below took 192, 212 and 77.)  A wavefront takes a tile:
//   gather    Z[i] = sum of value x row of X over the entries of piece i: 16 lanes for each of a step's four entries, whole rows
//             of X and plain multiply-adds;
//   multiply  Z W[r], v_mfma_f32_4x4x1_f32 with 16 blocks: float32 throughout, four rows at a time; W[r] from L1 / L2, for 32
//             features kept in registers over the tiles of a relation;
//   add       four rows x 32 results to the block's rows in LDS, as float64 atomics: ds_add_f64 takes 9 cycles a
//             wavefront, ds_add_f32 193 (measured), and the sums lose nothing.
// float32 matrix instructions are issued to the vector units: four 16x16x4 products take 134 cycles of a SIMD, 32 multiply-adds 88, and
// both together 237.  An earlier form gathered by selection matrices and multiplied 16 rows at a time; without any of its loads
// of X and W and without its adds it took 94 % of its time.  Now a relation with few pairs in a block does not pay for
// rows that it has not got, and the gather is two instructions a step.  What counts beside that: a tile's loads depend on each other and are
// waited for one tile later, so whatever makes the compiler wait for the newest load (a copy of a register that is being loaded, a
// count of loads that depends on a branch) costs a trip past L2 a tile; and wavefronts (32 x 32 features, 94 K rows, 51 relations, 4.76 M
// entries: six per SIMD 1.12 times as fast as five).  That graph 161 -> 107 us (99 with the longest blocks first),
// 1.9 M rows, 96 relations, 5.7 M entries 439 -> 342; 27,163 rows, 46 relations, 148,100 entries, 64 x 64: 39 -> 30 (27 with a block for every CU).  130 drawn graphs and feature sizes, 1.3 to 40 entries a pair: 1.21 times as fast up
// to 128 columns of Y (0.97 to 1.85), 1.06 for 256 and 512 (0.88 to 1.31: 16 entries a pair, for which W[r] is read twice as often).
// Blocks are as large as gives (relation, block) enough pieces, and small enough that there are workgroups
// for all CUs; a block with far more tiles than the others is several work items, whose sums meet in Y by global atomics.
//
// The order of the adds is not fixed (the last float32 bit may differ from call to call) unless the handle was built
// with a workspace: then every tile waits for its predecessor before it adds, item sums meet in the workspace,
// and results are reproducible bit for bit.
#include <string.h>

#include <algorithm>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "rgms_blocks.h"
#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

constexpr int kTileRows = 16;      // pieces per tile
constexpr int kPieceEntries = 4;   // most entries per piece: a tile has 16 steps at most, 64 entries, a lane each
constexpr int kPad = -1;           // the column of a place without an entry: past the end of X, where a buffer load gives 0

struct RgmsItem {
  int32_t block;    // rows block * block_rows .. of Y
  int32_t tile0;
  int32_t n_tiles;
  int32_t part;     // -1: the whole block; otherwise number of this item among the items of divided blocks
};

struct RgmsTile {
  int32_t first;       // its first step: entries 4 first ..
  int32_t rel;
  // bits 3e .. + 2: quads that have more than e steps (the longest are first); bits 12 + 4e .. + 3: steps for entries before e; bits 28, 29: quads
  // that hold pieces of the same rows, place for place, are 1 << so many (their sums meet before the product, and `rows` has them once)
  uint32_t shape;
  int32_t n_steps;
  uint16_t rows[kTileRows];  // of its pieces, in the block; block_rows: none
};
constexpr int kTileWords = sizeof(RgmsTile) / 4;

struct RgmsArgs {
  const RgmsItem* items;
  const RgmsTile* tiles;
  const int2* entries;       // [steps][4]: column, value bits; a step: entry e of each piece of a quad; inside a tile e major
  const float* X;
  const float* W;
  float* Y;
  float* partial;           // ORDERED: sums of the items of divided blocks
  int32_t n_rows;
  int32_t block_rows;
  int32_t d_out;
  int32_t width;            // columns of Y per workgroup, a multiple of 32
  int32_t n_waves;          // per workgroup
  int32_t sharers;          // workgroups per item
  uint32_t x_bytes;
};

typedef float floatx4 __attribute__((ext_vector_type(4)));

// f(0) .. f(N - 1) with the number as a type
template <int N, typename F, int I = 0>
__device__ __forceinline__ void for_steps(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    for_steps<N, F, I + 1>(std::forward<F>(f));
  }
}

// lane S of every 16
template <int S>
__device__ __forceinline__ int bcast16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + S, 0xF, 0xF, true);  // row_newbcast:S
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ int from_lane(int byte, int v) { return __builtin_amdgcn_ds_bpermute(byte, v); }

constexpr int kPass = 32;       // columns of Y per pass

__device__ float zero_row[128];  // what a place without an entry names where X has 4 GB or more (never written)

// TIN: d_in / 32.  In a 4x4x1 product of 16 blocks lane 4 b + i holds row i of block b's A, or column i of its B, and column i
// of all four rows of its result; A can be one block's for eight blocks together (cbsz 3).  So lanes 0 .. 31 form a product of
// four rows, one feature and 32 columns, lanes 32 .. 63 another one, with the feature that lies kHalf further on, and the two meet at
// the end.  W[r] is loaded in whole rows of 32 columns.  The gather leaves piece i's row in lanes 16 i .. + 15 (a load of 16 lanes
// that name four rows takes four times the lines: 246 against 206 us); lane 16 i + b's features go to lane 4 b + i, once a quad.
// WIDE_X: X has 4 GB or more.  (32 features: six wavefronts per SIMD, 80 registers, for which ORDERED spills two; with five, 3.2 M entries, 20
// relations, 20,000 rows, 32 x 32 took 92 us, with six 65.)
template <int TIN, bool ORDERED, bool WIDE_X>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(TIN == 1 ? 6 : 4))) void k_rgms(RgmsArgs a) {
  constexpr int VW = TIN == 1 ? 2 : 4;              // floats per lane and load of a row of X
  constexpr int kGroups = 2 * TIN / VW;             // loads per row
  constexpr int kZ = 2 * TIN;                       // registers per row
  constexpr int kDin = 32 * TIN, kRowBytes = 4 * kDin, kLog2RowBytes = TIN == 1 ? 7 : TIN == 2 ? 8 : 9;
  constexpr bool kTwoAhead = TIN == 1;              // rows for the first two entries of a tile's pieces are loaded ahead, or for one
  constexpr bool kInTurns = ORDERED || TIN > 1;     // the wavefronts take tiles in turns, not a run each
  constexpr int kHalf = 8 * VW;                     // of the features of a load, those of lanes 0 .. 31 of a product
  // Rows of W (and as many of the other half) that are loaded together: all of a pass, or 4, of which two lots are held.
  // (8, which spills 2 registers for 128 features: 94,806 rows, 96 relations, 670 K entries, 64 x 64 features 102 -> 106 us, 128 x 128
  // 327 -> 338; 16 spills 6 for 64 features, 127 for 128: 128 and 719 us.)
  constexpr int kChunk = TIN == 1 ? 16 : 4;
  constexpr int kChunks = kDin / 2 / kChunk;        // per pass
  extern __shared__ __align__(16) double y_tile[];  // [rows + 1][width] (the last for pieces that are none), then ORDERED: turn[width / kPass]
  RgmsItem item = a.items[blockIdx.x / (unsigned)a.sharers];
  if (a.sharers > 1) {
    const unsigned part = blockIdx.x % (unsigned)a.sharers, n = (unsigned)item.n_tiles;
    const unsigned lo = n * part / (unsigned)a.sharers;
    item.n_tiles = (int)(n * (part + 1) / (unsigned)a.sharers - lo);
    item.tile0 += (int)lo;
    item.part = 0;  // (its sums are added to Y)
  }
  const int rows = a.block_rows, width = a.width;
  const int n0 = blockIdx.y * width;
  const int cols = min(width, a.d_out - n0);
  int* turn = reinterpret_cast<int*>(y_tile + (rows + 1) * width);
  using std::integral_constant;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), n_waves = a.n_waves;

  // The wavefront's tiles: a run of them, so that one W[r] serves many; where they take turns, every n_waves-th.
  const int stride = kInTurns ? n_waves : 1;
  // (an item has at most 2^26 tiles, so 32 bits hold sixteen times as many; divisions of 64 bits are 150 instructions of a scalar unit each)
  const unsigned n_tiles = (unsigned)item.n_tiles;
  const int tile_lo = kInTurns ? wave : (int)(n_tiles * (unsigned)wave / (unsigned)n_waves);
  const int tile_hi = kInTurns ? item.n_tiles : (int)(n_tiles * (unsigned)(wave + 1) / (unsigned)n_waves);

  // A tile's loads depend on each other (the tile, its entries, the rows those name), each a trip past L2, so they run
  // ahead by three tiles, two and one: what is issued while tile t is multiplied has arrived when t + 1 begins.
  const char* tiles = reinterpret_cast<const char*>(a.tiles + item.tile0);
  const unsigned tile_word = 4u * min(lane, kTileWords - 1);
  auto load_tile = [&](int t) -> int {  // lane i: word i
    return *reinterpret_cast<const int*>(tiles + ((unsigned)(t < tile_hi ? t : tile_lo) * (unsigned)sizeof(RgmsTile) + tile_word));
  };
  auto first_of = [&](int tile) { return __builtin_amdgcn_readlane(tile, 0); };
  auto rel_of = [&](int tile) { return __builtin_amdgcn_readlane(tile, 1); };
  auto shape_of = [&](int tile) { return __builtin_amdgcn_readlane(tile, 2); };
  auto steps_of = [&](int tile) { return __builtin_amdgcn_readlane(tile, 3); };
  auto load_entries = [&](int first, int shape, int steps) -> int2 {  // lane 16 i + 4 e + q: entry e of piece i of quad q
    const int at = __builtin_amdgcn_ubfe(shape, 12 + (lane & 12), 4) + (lane & 3);
    const char* from = reinterpret_cast<const char*>(a.entries + (size_t)first * 4);
    return *reinterpret_cast<const int2*>(from + (unsigned)(min(at, steps - 1) * 32 + (lane >> 4) * 8));
  };
  auto wait_for_loads = [] { __builtin_amdgcn_s_waitcnt(0x0F70); };  // vmcnt(0)
  // (values that only some turns set: without this they would be kept from turn to turn)
  auto undefined = [](float (&v)[4][kZ]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < kZ; ++k) asm volatile("" : "=v"(v[q][k]));
  };
  // (a loaded value moves on here, and not where the load that takes its place would be waited for)
  auto moved = [](int v) { asm volatile("" : "+v"(v)); return v; };
  const __amdgpu_buffer_rsrc_t x_buf = buffer_of(a.X, a.x_bytes);
  const unsigned x_lane = (unsigned)(lane & 15) * (4 * VW);
  // (kPad: past the last row that an X below 4 GB can have)
  auto x_place = [&](int col) { return WIDE_X ? col : (int)((unsigned)col << kLog2RowBytes); };
  auto load_x = [&](int place, float (&x)[kZ]) {
    typedef float vec __attribute__((ext_vector_type(VW)));
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      vec v;
      if constexpr (WIDE_X)
        v = *reinterpret_cast<const vec*>((place == kPad ? zero_row : a.X + (size_t)place * kDin) + (lane & 15) * VW + 16 * VW * g);
      else if constexpr (VW == 2)
        v = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(x_buf, (int)((unsigned)place + x_lane), 0, 0));
      else
        v = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(x_buf, (int)((unsigned)place + x_lane), 256 * g, 0));
#pragma unroll
      for (int l = 0; l < VW; ++l) x[VW * g + l] = v[l];
    }
  };
  int tile = 0, tile_1 = 0, tile_2 = 0;
  int2 e = make_int2(0, 0), e_1 = e;
  float xa[4][kZ], xb[4][kZ];
  float w[2][kChunk];
  // entry E of the pieces of the first n quads
  auto load_rows = [&](auto entry, float (&x)[4][kZ], const int2& e, int n) {
    for_steps<4>([&](auto q) {
      constexpr int Q = decltype(q)::value;
      if (Q < n) load_x(bcast16<4 * decltype(entry)::value + Q>(e.x), x[Q]);
    });
  };
  auto sum_rows = [&](auto entry, const float (&x)[4][kZ], const int2& e, int n, float (&z)[4][kZ]) {
    for_steps<4>([&](auto q) {
      constexpr int Q = decltype(q)::value, E = decltype(entry)::value;
      if (Q < n) {
#pragma unroll
        for (int k = 0; k < kZ; ++k) {
          const float v = __int_as_float(bcast16<4 * E + Q>(e.y));
          z[Q][k] = E == 0 ? v * x[Q][k] : fmaf(v, x[Q][k], z[Q][k]);
        }
      }
    });
  };
  // W[r], chunk c of the pass at c0: w[i] is one row of the lower half in lanes 0 .. 31 and one of the upper half in the others
  const int w_lane = 4 * ((lane >> 5) * kHalf * a.d_out + (lane & 31));
  auto load_w = [&](int rel, int c0, int c, float (&w)[kChunk]) {
    const __amdgpu_buffer_rsrc_t w_buf = buffer_of(a.W + (size_t)rel * kDin * (size_t)a.d_out, (uint32_t)(kRowBytes * a.d_out));
    const int j = c * kChunk;
    int at = 4 * ((2 * kHalf * (j / kHalf) + j % kHalf) * a.d_out + n0 + c0);
    asm volatile("" : "+s"(at));  // (or the places of all rows are kept in registers)
#pragma unroll
    for (int i = 0; i < kChunk; ++i, at += 4 * a.d_out)
      w[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(w_buf, w_lane, at, 0));
  };

  // the place in LDS of the lane's column `lane_place` of a row, the upper or lower half of `two`: one instruction
  const unsigned row_bytes = 8 * width;
  auto place_of_row = [&](int two, auto which, unsigned lane_place) {
    unsigned at;
    if constexpr (decltype(which)::value % 2)
      asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(at) : "v"(two), "s"(row_bytes), "v"(lane_place));
    else
      asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(two), "s"(row_bytes), "v"(lane_place));
    return at;
  };
  // rows of X for the next tile.  (Where W[r] streams in behind them they are four whatever the tile holds: a load can only be
  // waited for by the number of those after it.)
  auto load_next = [&](int shape) {
    load_rows(integral_constant<int, 0>{}, xa, e, kChunks == 1 ? shape & 7 : 4);
    if constexpr (kTwoAhead) load_rows(integral_constant<int, 1>{}, xb, e, shape >> 3 & 7);
  };
  const int z_from = 4 * (16 * (lane & 3) + (lane >> 2));
  const int y_lane = 8 * (lane & 31);
  if (tile_lo < tile_hi) {
    tile = load_tile(tile_lo); tile_1 = load_tile(tile_lo + stride); tile_2 = load_tile(tile_lo + 2 * stride);
  }
  for (int i = threadIdx.x * 2; i < (rows + 1) * width; i += blockDim.x * 2)
    *reinterpret_cast<double2*>(y_tile + i) = make_double2(0., 0.);
  if (ORDERED && threadIdx.x < (unsigned)(width / kPass)) turn[threadIdx.x] = 0;
  if (tile_lo < tile_hi) {
    e = load_entries(first_of(tile), shape_of(tile), steps_of(tile));
    e_1 = load_entries(first_of(tile_1), shape_of(tile_1), steps_of(tile_1));
    e.x = x_place(e.x);
    load_w(rel_of(tile), 0, 0, w[0]);
    if constexpr (kChunks > 1) load_w(rel_of(tile), 0, 1, w[1]);
    const int shape = shape_of(tile);
    load_next(shape);
  }
  __syncthreads();

  for (int t = tile_lo; t < tile_hi; t += stride) {
    // ---- gather: entry 0 of all pieces, entry 1, ..
    // (All that the last turn has loaded is waited for here, and what only some turns load is waited for where they do: past
    // that the compiler cannot count what is in flight, and would wait for the loads that are to stay there.)
    if constexpr (kChunks == 1) wait_for_loads();
    const int shape = shape_of(tile), n_1 = shape >> 3 & 7, n_2 = shape >> 6 & 7, n_3 = shape >> 9 & 7;
    int n_quads = shape & 7;
    const int rel = rel_of(tile), rel_next = rel_of(tile_1), shape_1 = shape_of(tile_1);
    const int first_2 = first_of(tile_2), shape_2 = shape_of(tile_2), steps_2 = steps_of(tile_2);
    int piece_rows[4];  // two each: of pieces 8 p + 4 (lane >> 5) ..
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) piece_rows[2 * p + i] = from_lane(4 * (4 + 4 * p + i) + 8 * (lane >> 5), tile);
    float z[4][kZ];
    undefined(z);
    sum_rows(integral_constant<int, 0>{}, xa, e, n_quads, z);
    if (n_1 > 0) {
      if constexpr (kTwoAhead) {
        load_rows(integral_constant<int, 2>{}, xa, e, n_2);
        sum_rows(integral_constant<int, 1>{}, xb, e, n_1, z);
        if (n_2 > 0) {
          load_rows(integral_constant<int, 3>{}, xb, e, n_3);
          sum_rows(integral_constant<int, 2>{}, xa, e, n_2, z);
          sum_rows(integral_constant<int, 3>{}, xb, e, n_3, z);
        }
      } else {
        float x[4][kZ];
        undefined(x);
        load_rows(integral_constant<int, 1>{}, x, e, n_1);
        sum_rows(integral_constant<int, 1>{}, x, e, n_1, z);
        if (n_2 > 0) {
          load_rows(integral_constant<int, 2>{}, x, e, n_2);
          sum_rows(integral_constant<int, 2>{}, x, e, n_2, z);
          load_rows(integral_constant<int, 3>{}, x, e, n_3);
          sum_rows(integral_constant<int, 3>{}, x, e, n_3, z);
        }
      }
    }
    if (const int joined = (unsigned)shape >> 28; joined != 0) {  // (four quads)
      const bool all = joined == 2;
#pragma unroll
      for (int k = 0; k < kZ; ++k) {
        z[0][k] += z[1][k];
        z[1][k] = z[2][k] + z[3][k];
      }
      if (all)
#pragma unroll
        for (int k = 0; k < kZ; ++k) z[0][k] += z[1][k];
      n_quads = all ? 1 : 2;
    }
    for_steps<4>([&](auto q) {  // to the places of the product
      constexpr int Q = decltype(q)::value;
      if (Q < n_quads) {
#pragma unroll
        for (int k = 0; k < kZ; ++k) z[Q][k] = __int_as_float(from_lane(z_from, __float_as_int(z[Q][k])));
      }
    });
    // ---- what the next tiles need
    if constexpr (kChunks == 1) wait_for_loads();
    e = make_int2(x_place(moved(e_1.x)), moved(e_1.y));
    e_1 = load_entries(first_2, shape_2, steps_2);
    tile = moved(tile_1); tile_1 = moved(tile_2);
    tile_2 = load_tile(t + 3 * stride);
    if constexpr (kChunks == 1) load_next(shape_1);
    // ---- multiply: quads Q0 .. Q0 + NQ - 1 and the pass at c0, to d
    auto products = [&](auto q0, auto nq, auto is_last, int c0, floatx4* d) {
      constexpr int Q0 = decltype(q0)::value, NQ = decltype(nq)::value;
      constexpr bool kLast = decltype(is_last)::value;
#pragma unroll
      for (int q = 0; q < (NQ + 1) / 2 * 2; ++q) d[q] = floatx4{0.f, 0.f, 0.f, 0.f};
      for_steps<kChunks>([&](auto chunk) {
        constexpr int C = decltype(chunk)::value;
        // (as late as leaves two chunks of W to load behind them, since those are waited for in order)
        if constexpr (kLast && kChunks > 1 && C == kChunks - 2) load_next(shape_1);
        for_steps<kChunk>([&](auto step) {
          constexpr int I = decltype(step)::value, J = C * kChunk + I;
          constexpr int R = VW * (J / kHalf) + J % VW, S = J % kHalf / VW;  // the feature's register, and the block that holds it
          for_steps<NQ>([&](auto q) {
            constexpr int Q = decltype(q)::value;
            d[Q] = __builtin_amdgcn_mfma_f32_4x4x1f32(z[Q0 + Q][R], w[C & 1][I], d[Q], 3, S, 0);
          });
        });
        if constexpr (kChunks > 1) {
          if constexpr (C + 2 < kChunks) load_w(rel, c0, C + 2, w[C & 1]);
          else load_w(kLast ? rel_next : rel, kLast ? 0 : c0 + kPass, C & 1, w[C & 1]);
        }
      });
    };
    // ---- two quads' sums: the halves meet, and row i of d is then that of piece 4 (lane >> 5) + i of them
    auto meet = [&](const floatx4* d, int i) {
      const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[0][i]), __float_as_uint(d[1][i]), false, false);
      return __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
    };
    auto add = [&](auto&& sum, int rows_01, int rows_23, int c0) {  // sum(i)
      for_steps<4>([&](auto row) {
        constexpr int i = decltype(row)::value;
        const float s = sum(i);
        const unsigned at = place_of_row(i < 2 ? rows_01 : rows_23, row, y_lane + 8 * c0);
        atomicAdd(reinterpret_cast<double*>(reinterpret_cast<char*>(y_tile) + at), (double)s);
      });
    };
    auto wait_for_turn = [&](int c0) {
      if constexpr (ORDERED) {
        // tile t adds after tile t - 1, which an earlier turn of this loop or another wavefront of this workgroup
        // is on its way to: the wait ends
        while (__hip_atomic_load(turn + c0 / kPass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != t)
          __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      }
    };
    auto pass = [&](auto is_last, int c0) {
      using C0 = integral_constant<int, 0>;
      using C1 = integral_constant<int, 1>;
      using C2 = integral_constant<int, 2>;
      if constexpr (kChunks == 1) {
        // (All of W is there: two quads at a time take fewer registers.  ORDERED: both are formed before the wait for the turn, with four
        // floats each until then.  Before, the others waited for the second product as well: 27,163 rows, 46 relations, 145 K entries, 32 x 32
        // features 28.1 -> 22.9 us, with the load of W below.)
        floatx4 d[2];
        float first[4], last[4];
        auto keep = [&](float (&sum)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[i] = meet(d, i);
        };
        if (n_quads > 2) {
          products(C0{}, C2{}, is_last, c0, d);
          keep(first);
          if constexpr (!ORDERED) add([&](int i) { return first[i]; }, piece_rows[0], piece_rows[1], c0);
          if (n_quads > 3) products(C2{}, C2{}, is_last, c0, d);
          else products(C2{}, C1{}, is_last, c0, d);
        } else if (n_quads > 1) {
          products(C0{}, C2{}, is_last, c0, d);
        } else {
          products(C0{}, C1{}, is_last, c0, d);
        }
        keep(last);
        // (W[r] that is multiplied next, on its way while the sums are added; asked for after them, every pass waited for it.  Held twice
        // and asked for before the products it takes 16 registers, a wavefront per SIMD: graphs of full tiles 3 to 10 % slower.)
        if constexpr (!decltype(is_last)::value) load_w(rel, c0 + kPass, 0, w[0]);
        else if (rel_next != rel || cols > kPass) load_w(rel_next, 0, 0, w[0]);
        wait_for_turn(c0);
        if (n_quads > 2) {
          if constexpr (ORDERED) add([&](int i) { return first[i]; }, piece_rows[0], piece_rows[1], c0);
          add([&](int i) { return last[i]; }, piece_rows[2], piece_rows[3], c0);
        } else {
          add([&](int i) { return last[i]; }, piece_rows[0], piece_rows[1], c0);
        }
      } else {
        auto quads = [&](auto nq) {
          floatx4 d[(decltype(nq)::value + 1) / 2 * 2];
          products(C0{}, nq, is_last, c0, d);
          wait_for_turn(c0);
          add([&](int i) { return meet(d, i); }, piece_rows[0], piece_rows[1], c0);
          if constexpr (decltype(nq)::value > 2) add([&](int i) { return meet(d + 2, i); }, piece_rows[2], piece_rows[3], c0);
        };
        if (n_quads == 4) quads(integral_constant<int, 4>{});
        else if (n_quads == 3) quads(integral_constant<int, 3>{});
        else if (n_quads == 2) quads(C2{});
        else quads(C1{});
      }
      if constexpr (ORDERED) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");  // (LDS only: the prefetches stay in flight)
        if (lane == 0)
          __hip_atomic_store(turn + c0 / kPass, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    };
    int c0 = 0;
#pragma unroll 1
    for (; c0 + kPass < cols; c0 += kPass) {
      pass(std::false_type{}, c0);
      if constexpr (kChunks == 1) wait_for_loads();
    }
    pass(std::true_type{}, c0);
  }
  __syncthreads();

  // ---- what is left (in a scope of its own: anything kept since the loop above costs registers in it)
  {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    // ---- the block's rows
    const int row0 = item.block * rows;
    const int rows_here = min(rows, a.n_rows - row0);
    const int quads = cols / 4;
    const int n_quads = rows_here * quads;
    const int shift = (quads & (quads - 1)) == 0 ? 31 - __builtin_clz((unsigned)quads) : -1;
    for (int i = tid; i < n_quads; i += (int)blockDim.x) {
      const int row = shift >= 0 ? i >> shift : i / quads, c = (i - row * quads) * 4;
      float y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = (float)y_tile[row * width + c + k];
      if (item.part < 0) {
        store_unaligned<4>(a.Y + (size_t)(row0 + row) * a.d_out + n0 + c, y);
      } else if constexpr (ORDERED) {
        store_vec<4>(a.partial + ((size_t)item.part * rows + row) * a.d_out + n0 + c, y);
      } else {
        float* p = a.Y + (size_t)(row0 + row) * a.d_out + n0 + c;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (y[k] != 0.f) atomicAdd(p + k, y[k]);
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_zero(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0.f;
}

// The rows of a divided block: cleared before its items add to them, or, with a workspace, the sum of its items' parts
// in their order.  divided[b] = {block, first part, parts}.
__global__ __launch_bounds__(256) void k_rgms_divided(const int4* __restrict__ divided, int32_t n_rows,
                                                      int32_t block_rows, int32_t d_out,
                                                      const float* __restrict__ partial, float* Y) {
  const int4 d = divided[blockIdx.x];
  const int row0 = d.x * block_rows, rows = min(block_rows, n_rows - row0);
  for (int i = blockIdx.y * blockDim.x + threadIdx.x; i < rows * d_out; i += gridDim.y * blockDim.x) {
    float sum = 0.f;
    if (partial)
      for (int p = 0; p < d.z; ++p) sum += partial[(size_t)(d.y + p) * block_rows * d_out + i];
    Y[(size_t)row0 * d_out + i] = sum;
  }
}

// ------------------------------------------------------------------- build
// cells are (block, relation), block-major; one wavefront each
struct CellArgs {
  const int32_t* indptr;
  int64_t n_cells;
  int32_t n_rel, n_rows, block_rows, k;
};
constexpr int kCountSlots = 64, kCountStride = 8;

// The pieces of a cell in the order of its tiles: longest first, in quads of four and tiles of four quads.
// at_least[L]: quads with a piece of at least L entries, which therefore have so many steps.
struct CellShape {
  int count[kPieceEntries + 1];      // pieces of L entries
  int at_least[kPieceEntries + 1];
  __device__ __forceinline__ int tiles() const { return (at_least[1] + 3) >> 2; }
  __device__ __forceinline__ int steps_of(int quad) const {
    int n = 0;
#pragma unroll
    for (int len = 1; len <= kPieceEntries; ++len) n += at_least[len] > quad;
    return n;
  }
  __device__ __forceinline__ int steps_before(int quad) const {
    int n = 0;
#pragma unroll
    for (int len = 1; len <= kPieceEntries; ++len) n += min(at_least[len], quad);
    return n;
  }
};

// (one wavefront; the result in all lanes)  row(n): what else there is to do for a row of n entries
template <typename F>
__device__ __forceinline__ CellShape cell_shape(const int32_t* __restrict__ ptr, int rows, int lane, F&& row) {
  CellShape c;
#pragma unroll
  for (int len = 0; len <= kPieceEntries; ++len) c.count[len] = c.at_least[len] = 0;
  int full = 0;
  for (int i0 = 0; i0 < rows; i0 += 64) {
    const int i = i0 + lane;
    const int n = i < rows ? ptr[i + 1] - ptr[i] : 0;
    row(n);
    full += n / kPieceEntries;
#pragma unroll
    for (int len = 1; len < kPieceEntries; ++len) c.count[len] += __popcll(__ballot(n % kPieceEntries == len));
  }
  for (int d = 32; d > 0; d >>= 1) full += __shfl_xor(full, d, 64);
  c.count[kPieceEntries] = full;
  int pieces = 0;
#pragma unroll
  for (int len = kPieceEntries; len >= 1; --len) {
    pieces += c.count[len];
    c.at_least[len] = (pieces + 3) >> 2;
  }
  return c;
}

// tiles and steps of every cell; counts[slot][0] += pairs with entries, [1] += slots of padding that hyb(1, k) has for them
__global__ __launch_bounds__(256) void k_cell_tiles(CellArgs a, int32_t* cell_tiles, int32_t* cell_steps,
                                                    unsigned long long* counts) {
  const int lane = threadIdx.x & 63;
  const int64_t cell = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cell >= a.n_cells) return;
  const int64_t block = cell / a.n_rel, rel = cell - block * a.n_rel;
  const int64_t row0 = block * a.block_rows;
  const int rows = (int)min((int64_t)a.block_rows, (int64_t)a.n_rows - row0);
  const int32_t* ptr = a.indptr + rel * a.n_rows + row0;
  int pairs = 0, pads = 0;
  const CellShape c = cell_shape(ptr, rows, lane, [&](int len) {
    pairs += len > 0;
    if (len > 1) {
      const int log2w = 32 - __clz(len - 1);
      if (log2w <= a.k) pads += (1 << log2w) - len;
    }
  });
  for (int d = 32; d > 0; d >>= 1) {
    pairs += __shfl_down(pairs, d, 64);
    pads += __shfl_down(pads, d, 64);
  }
  if (lane == 0) {
    cell_tiles[cell] = c.tiles();
    cell_steps[cell] = c.steps_before(c.at_least[1]);
    unsigned long long* to = counts + (blockIdx.x & (kCountSlots - 1)) * kCountStride;
    if (pairs) atomicAdd(&to[0], (unsigned long long)pairs);
    if (pads) atomicAdd(&to[1], (unsigned long long)pads);
  }
}

// block_tile[b] = first tile of block b (b = n_blocks: their number), block_step[b] = first step
__global__ void k_block_tiles(int32_t n_blocks, int32_t n_rel, const int32_t* __restrict__ cell_tile0,
                              const int32_t* __restrict__ n_tiles, const int32_t* __restrict__ cell_step0,
                              const int32_t* __restrict__ n_steps, int32_t* block_tile, int32_t* block_step) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > n_blocks) return;
  block_tile[b] = b < n_blocks ? cell_tile0[(int64_t)b * n_rel] : *n_tiles;
  block_step[b] = b < n_blocks ? cell_step0[(int64_t)b * n_rel] : *n_steps;
}

// the tiles of every cell and their entries
__global__ __launch_bounds__(256) void k_fill_tiles(CellArgs a, const int32_t* __restrict__ indices,
                                                    const float* __restrict__ values, const int32_t* __restrict__ cell_tile0,
                                                    const int32_t* __restrict__ cell_step0, RgmsTile* tiles, int2* entries) {
  const int lane = threadIdx.x & 63;
  const int64_t cell = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cell >= a.n_cells) return;
  const int64_t block = cell / a.n_rel, rel = cell - block * a.n_rel;
  const int64_t row0 = block * a.block_rows;
  const int rows = (int)min((int64_t)a.block_rows, (int64_t)a.n_rows - row0);
  const int32_t* ptr = a.indptr + rel * a.n_rows + row0;
  if (ptr[rows] == ptr[0]) return;
  // the rows with entries, so that the lanes below have one each
  __shared__ uint16_t filled[4][1 << kMaxLog2Block];
  uint16_t* rows_of = filled[threadIdx.x >> 6];
  int n_filled = 0, row = 0;
  int fours = 0, twos = 0;  // see below
  const CellShape c = cell_shape(ptr, rows, lane, [&](int n) {
    fours += n / (4 * kPieceEntries);
    twos += __popcll(__ballot((n / kPieceEntries & 2) != 0));
    const unsigned long long some = __ballot(n > 0);
    if (n > 0) rows_of[n_filled + __popcll(some & (((unsigned long long)1 << lane) - 1))] = (uint16_t)(row + lane);
    n_filled += __popcll(some);
    row += 64;
  });
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int tile0 = cell_tile0[cell], step0 = cell_step0[cell];
  const int n_tiles = c.tiles();
  int n_pieces = 0;
#pragma unroll
  for (int len = 1; len <= kPieceEntries; ++len) n_pieces += c.count[len];

  // The full pieces of a row are taken by fours, what is left by twos, what is left of that singly.  Fours fill tiles, a piece in the same place of
  // each of the tile's quads; then twos, in the same place of quads 0 and 1 or 2 and 3.  Fours that fill no tile are twos, and twos that fill
  // none are single pieces: there are as many tiles and steps as without, and a row's entries are multiplied by W[r] sixteen or eight at a
  // time.
  for (int d = 32; d > 0; d >>= 1) fours += __shfl_xor(fours, d, 64);
  const int tiles_of_fours = fours / 4;
  const int twos_of_fours = fours % 4 * 2;  // (the first twos)
  twos += twos_of_fours;
  const int tiles_of_twos = twos / 8, joined_tiles = tiles_of_fours + tiles_of_twos;
  const int singles_of_twos = twos % 8 * 2;

  // what a tile is, and the rows of pieces that are none
  auto quads_with = [&](int quad0, int e) { return min(max(c.at_least[e + 1] - quad0, 0), 4); };
  for (int t = lane; t < n_tiles; t += 64) {
    RgmsTile* to = tiles + tile0 + t;
    uint32_t shape = 0;
    int steps = 0;
#pragma unroll
    for (int e = 0; e < kPieceEntries; ++e) {
      const int n = quads_with(4 * t, e);
      shape |= (uint32_t)n << (3 * e) | (uint32_t)(steps & 15) << (12 + 4 * e);
      steps += n;
    }
    to->first = step0 + c.steps_before(4 * t);
    to->rel = (int)rel;
    const int joined = t < tiles_of_fours ? 2 : t < joined_tiles ? 1 : 0;
    to->shape = shape | (uint32_t)joined << 28;
    to->n_steps = steps;
    const int n_rows_of = min(kTileRows >> joined, n_pieces - kTileRows * t);
    for (int i = 0; i < kTileRows; ++i)
      if (i >= n_rows_of) to->rows[i] = (uint16_t)a.block_rows;
  }

  // piece number `place`: `len` entries from `from` on, of row `row`, which is number `slot` of its tile's rows (negative: another piece says so)
  auto put = [&](int place, int slot, int row, int from, int len) {
    const int quad = place >> 2, quad0 = quad & ~3;
    if (slot >= 0) tiles[tile0 + (place >> 4)].rows[slot] = (uint16_t)row;
    const int steps = c.steps_of(quad);
    const int i_end = place == n_pieces - 1 ? 4 : (place & 3) + 1;  // (the last piece fills its quad)
    int64_t step = step0 + c.steps_before(quad0) + (quad & 3);
#pragma unroll
    for (int e = 0; e < kPieceEntries; ++e) {
      if (e >= steps) break;
      const int at = from + e;
      int2* to = entries + step * 4 + (place & 3);
      *to = e < len ? make_int2(indices[at], __float_as_int(values[at])) : make_int2(kPad, 0);
      for (int i = (place & 3) + 1; i < i_end; ++i) *++to = make_int2(kPad, 0);
      step += quads_with(quad0, e);
    }
  };
  // full piece k of a row with `full` of them, before which there are so many fours, twos and single pieces
  auto put_full = [&](int k, int full, int before_4, int before_2, int before_1, int row, int from) {
    const int in_fours = full & ~3, in_twos = full & ~1;
    int place, slot;
    int two = -1, part = k & 1;  // the two that the piece belongs to, and which half of it
    if (k < in_fours) {
      const int four = before_4 + (k >> 2);
      if (four < 4 * tiles_of_fours) {
        place = (four & ~3) * 4 + (k & 3) * 4 + (four & 3);
        slot = (k & 3) == 0 ? four & 3 : -1;
      } else {
        two = (four - 4 * tiles_of_fours) * 2 + (k >> 1 & 1);
      }
    } else if (k < in_twos) {
      two = twos_of_fours + before_2;
    } else {
      place = joined_tiles * kTileRows + singles_of_twos + before_1;
      slot = place & 15;
    }
    if (two >= 8 * tiles_of_twos) {
      place = joined_tiles * kTileRows + (two - 8 * tiles_of_twos) * 2 + part;
      slot = place & 15;
    } else if (two >= 0) {
      place = (tiles_of_fours + (two >> 3)) * kTileRows + (two & 4) * 2 + part * 4 + (two & 3);
      slot = part == 0 ? two & 7 : -1;
    }
    put(place, slot, row, from + k * kPieceEntries, kPieceEntries);
  };
  int place_of[kPieceEntries];  // of the next piece of every smaller length
#pragma unroll
  for (int len = kPieceEntries - 1; len >= 1; --len)
    place_of[len] = len == kPieceEntries - 1 ? c.count[kPieceEntries] : place_of[len + 1] + c.count[len + 1];
  int done_4 = 0, done_2 = 0, done_1 = 0;
  for (int i0 = 0; i0 < n_filled; i0 += 64) {
    int i = 0, from = 0, n = 0;
    if (i0 + lane < n_filled) { i = rows_of[i0 + lane]; from = ptr[i]; n = ptr[i + 1] - from; }
    const int full = n / kPieceEntries, rest = n % kPieceEntries;
    int place = 0;
#pragma unroll
    for (int len = 1; len < kPieceEntries; ++len) {
      const unsigned long long same = __ballot(rest == len);
      if (rest == len) place = place_of[len] + __popcll(same & (((unsigned long long)1 << lane) - 1));
      place_of[len] += __popcll(same);
    }
    if (rest > 0) put(place, place & 15, i, from + n - rest, rest);
    if (c.count[kPieceEntries] == 0) continue;
    // full pieces, a lane each
    const unsigned long long before = ((unsigned long long)1 << lane) - 1;
    const unsigned long long with_two = __ballot((full & 2) != 0), with_one = __ballot((full & 1) != 0);
    const int upto = wave_inclusive_scan(full, lane), upto_4 = wave_inclusive_scan(full >> 2, lane);
    const int before_4 = done_4 + upto_4 - (full >> 2);
    const int before_2 = done_2 + __popcll(with_two & before), before_1 = done_1 + __popcll(with_one & before);
    const int packed = i | before_2 << 10 | before_1 << 20;  // (at most 512 rows)
    const int total = __shfl(upto, 63, 64);
    for (int k0 = 0; k0 < total; k0 += 64) {
      int src = 0;  // the row whose piece it is: the first with more pieces up to it
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (__shfl(upto, src + step - 1, 64) <= k0 + lane) src += step;
      const int m = __shfl(full, src, 64), f = __shfl(from, src, 64), b4 = __shfl(before_4, src, 64);
      const int first = __shfl(upto - full, src, 64), rest_of = __shfl(packed, src, 64);
      if (k0 + lane < total)
        put_full(k0 + lane - first, m, b4, rest_of >> 10 & 1023, rest_of >> 20, rest_of & 1023, f);
    }
    done_4 += __shfl(upto_4, 63, 64);
    done_2 += __popcll(with_two);
    done_1 += __popcll(with_one);
  }
}

template <int TIN, bool ORDERED, bool WIDE_X>
void launch_rgms(dim3 grid, dim3 block, size_t lds, hipStream_t stream, const RgmsArgs& a) {
  auto* kernel = &k_rgms<TIN, ORDERED, WIDE_X>;
  static OncePerDevice allowed;
  allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, allowed);
  hipLaunchKernelGGL(kernel, grid, block, lds, stream, a);
}

}  // namespace
}  // namespace sptir

// The handle behind sptir_rgms_t.
struct sptir_rgms_handle {
  int32_t n_rel, n_rows, n_cols, k;
  int64_t nnz, n_pairs, n_pads;
  int32_t block_rows;
  int64_t n_tiles;
  sptir::RgmsTile* tiles;
  int2* entries;          // [n_steps][4]
  sptir::RgmsItem* items;
  int32_t n_items;
  int4* divided;          // divided blocks: block, first part, parts
  int32_t n_divided, n_parts;
  int32_t workspace_d_out;
  float* partial;         // workspace: [n_parts][rows of a block][d_out]
  void* blob;             // one allocation holds all of them
  size_t device_bytes;
  sptir_alloc_fn alloc;
  sptir_free_fn free_;
  void* alloc_ctx;
};

using namespace sptir;

extern "C" sptir_status_t sptir_rgms_destroy(sptir_rgms_t* p) {
  if (!p) return SPTIR_OK;
  if (p->blob) p->free_(p->blob, p->alloc_ctx);
  delete p;
  return SPTIR_OK;
}

extern "C" sptir_status_t sptir_rgms_info(const sptir_rgms_t* p, sptir_rgms_info_t* out) {
  if (!p || !out) return SPTIR_ERR_INVALID_ARG;
  sptir_rgms_info_t o;
  o.n_relations = p->n_rel; o.n_rows = p->n_rows; o.n_cols = p->n_cols; o.max_bucket_log2 = p->k;
  o.nnz = p->nnz; o.n_stacked_rows_stored = p->n_pairs; o.n_pad_slots = p->n_pads;
  o.n_tiles = p->n_tiles; o.workspace_d_out = p->workspace_d_out; o.row_block = p->block_rows;
  o.device_bytes = (int64_t)p->device_bytes;
  *out = o;
  return SPTIR_OK;
}

extern "C" sptir_status_t sptir_rgms_build(const sptir_csr_t* stacked, int32_t n_relations, int32_t max_bucket_log2,
                                           int32_t workspace_d_out, void* stream_, sptir_rgms_t** out) {
  if (!stacked || !out || n_relations < 1) return SPTIR_ERR_INVALID_ARG;
  if (workspace_d_out < 0 || workspace_d_out % 32 != 0) return SPTIR_ERR_INVALID_ARG;
  if (stacked->n_rows < 0 || stacked->n_rows % n_relations != 0) return SPTIR_ERR_INVALID_ARG;
  const int32_t k = max_bucket_log2 < 0 ? 5 : max_bucket_log2;  // the paper decomposes every relation as hyb(1, 5)
  if (k > 5) return SPTIR_ERR_INVALID_ARG;
  const int64_t nnz = stacked->nnz;
  if (stacked->n_cols < 0 || nnz < 0) return SPTIR_ERR_INVALID_ARG;
  if (nnz >= ((int64_t)1 << 31)) return SPTIR_ERR_OVERFLOW;
  if (!stacked->indptr || (nnz > 0 && (!stacked->indices || !stacked->values))) return SPTIR_ERR_INVALID_ARG;
  if (nnz > 0 && (stacked->n_rows == 0 || stacked->n_cols == 0)) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;

  sptir_rgms_handle* p = new (std::nothrow) sptir_rgms_handle();
  if (!p) return SPTIR_ERR_ALLOC;
  memset(p, 0, sizeof(*p));
  current_allocator(&p->alloc, &p->free_, &p->alloc_ctx);
  p->n_rel = n_relations; p->n_rows = stacked->n_rows / n_relations; p->n_cols = stacked->n_cols; p->k = k;
  p->nnz = nnz; p->workspace_d_out = workspace_d_out;
  p->block_rows = rows_of_a_block(p->n_rows, n_relations, nnz, workspace_d_out > 0);
  const int32_t n_blocks = (int32_t)(((int64_t)p->n_rows + p->block_rows - 1) / p->block_rows);
  CellArgs ca;
  ca.indptr = stacked->indptr; ca.n_cells = (int64_t)n_blocks * n_relations; ca.n_rel = n_relations;
  ca.n_rows = p->n_rows; ca.block_rows = p->block_rows; ca.k = k;
  const int64_t cell_wgs = (ca.n_cells + 3) / 4;
  const int64_t n_seq = (int64_t)(scan_room(std::max<int64_t>(ca.n_cells, 1)) / kScanSeq);

  // temporaries: validation flags and counts, block starts (one copy brings them to the host), cells
  constexpr size_t kReport = (kValidationWords + kCountSlots * kCountStride) * sizeof(unsigned long long);
  size_t tmp_bytes = kReport;
  auto reserve = [](size_t* size, size_t bytes) { const size_t at = *size; *size = (at + bytes + 255) & ~(size_t)255; return at; };
  const size_t o_block_tile = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_blocks + 1));
  const size_t o_block_step = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_blocks + 1));
  const size_t report_bytes = o_block_step + sizeof(int32_t) * ((size_t)n_blocks + 1);
  const size_t o_cells = reserve(&tmp_bytes, sizeof(int32_t) * (size_t)n_seq * kScanSeq);
  const size_t o_cell_steps = reserve(&tmp_bytes, sizeof(int32_t) * (size_t)n_seq * kScanSeq);
  const size_t o_seq = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_seq + 1));
  const size_t o_step_seq = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_seq + 1));
  char* tmp = (char*)scratch_alloc(tmp_bytes, p->alloc, p->alloc_ctx, stream);
  PinnedBuf host = pinned_acquire(std::max(report_bytes, (size_t)16));
  std::vector<RgmsItem> items;
  std::vector<int4> divided;
  sptir_status_t st = SPTIR_OK;
#define RGMS_HIP(call)                                                 \
  do {                                                                 \
    hipError_t e_ = (call);                                            \
    if (e_ != hipSuccess) { st = note_hip_error(e_, #call); goto fail; } \
  } while (0)
  if (!tmp || !host.p) { st = SPTIR_ERR_ALLOC; goto fail; }
  {
    unsigned long long* d_flags = (unsigned long long*)tmp;
    unsigned long long* d_counts = d_flags + kValidationWords;
    int32_t* d_block_tile = (int32_t*)(tmp + o_block_tile);
    int32_t* d_block_step = (int32_t*)(tmp + o_block_step);
    int32_t* d_cells = (int32_t*)(tmp + o_cells);
    int32_t* d_cell_steps = (int32_t*)(tmp + o_cell_steps);
    int32_t* d_seq = (int32_t*)(tmp + o_seq);
    int32_t* d_step_seq = (int32_t*)(tmp + o_step_seq);
    if (cell_wgs > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
    RGMS_HIP(hipMemsetAsync(tmp, 0, kReport, stream));
    launch_validation(stacked, false, d_flags, stream);
    if (ca.n_cells > 0) {
      // (the numbers below mean something only if the verdict is good, and index nothing before it is known)
      hipLaunchKernelGGL(k_cell_tiles, dim3((unsigned)cell_wgs), dim3(256), 0, stream, ca, d_cells, d_cell_steps,
                         d_counts);
      RGMS_HIP(hipGetLastError());
      st = device_exclusive_scan(d_cells, ca.n_cells, d_seq, stream);
      if (st == SPTIR_OK) st = device_exclusive_scan(d_cell_steps, ca.n_cells, d_step_seq, stream);
      if (st != SPTIR_OK) goto fail;
      hipLaunchKernelGGL(k_block_tiles, dim3((unsigned)(n_blocks / 256 + 1)), dim3(256), 0, stream, n_blocks,
                         n_relations, d_cells, d_seq + n_seq, d_cell_steps, d_step_seq + n_seq, d_block_tile, d_block_step);
      RGMS_HIP(hipGetLastError());
    }
    RGMS_HIP(hipMemcpyAsync(host.p, tmp, report_bytes, hipMemcpyDeviceToHost, stream));
    int32_t first = 0;
    if (stacked->n_rows == 0)
      RGMS_HIP(hipMemcpyAsync(&first, stacked->indptr, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
    RGMS_HIP(hipStreamSynchronize(stream));
    if (stacked->n_rows == 0 && first != 0) { st = SPTIR_ERR_INVALID_ARG; goto fail; }
    st = validation_verdict((const unsigned long long*)host.p, nullptr);
    if (st != SPTIR_OK) goto fail;
    const unsigned long long* counts = (const unsigned long long*)host.p + kValidationWords;
    for (int s = 0; s < kCountSlots; ++s) {
      p->n_pairs += (int64_t)counts[s * kCountStride];
      p->n_pads += (int64_t)counts[s * kCountStride + 1];
    }
    const int32_t* block_tile = (const int32_t*)(host.p + o_block_tile);
    const int32_t* block_step = (const int32_t*)(host.p + o_block_step);
    p->n_tiles = n_blocks > 0 ? block_tile[n_blocks] : 0;
    const int64_t n_steps = n_blocks > 0 ? block_step[n_blocks] : 0;  // (at most nnz: a step has an entry)

    // ---- work items: a block each.  A block of more than twice the mean work is divided: 1775 drawn graphs and feature sizes of 30,000 to
    //      700,000 rows by popularity, without a workspace: at 1.6 times the mean 0.98 times as fast (0.75 to 1.26), at three times
    //      0.98 (0.67 to 1.55), at four 0.96 (0.53 to 1.58).  (564 with a workspace, which a divided block passes through: at three
    //      times 1.06 (0.75 to 1.51), at four 1.09, but 0.67 at worst.)
    //      Where there are few blocks, all are, into about 384 items: three for two CUs, so that some with less to do fill the gaps
    //      that others leave.  1169 drawn graphs of 1,500 to 18,000 rows, against 512 items: 1.07 times as fast (0.92 to 1.39); 256
    //      1.01 (0.55 to 1.83), 768 0.96, 1024 0.92.
    auto tiles_of = [&](int32_t b) { return block_tile[b + 1] - block_tile[b]; };
    auto cost_of = [&](int32_t b) { return (int64_t)tiles_of(b) + (block_step[b + 1] - block_step[b]) / 8; };
    const int64_t cost = p->n_tiles + n_steps / 8, mean = n_blocks > 0 ? cost / n_blocks : 0;
    // (an item's tiles lie within 4 GB)
    const int64_t most = std::min<int64_t>(n_blocks >= 160 ? std::max<int64_t>(64, 2 * mean) : std::max<int64_t>(8, cost / 384), 1 << 26);
    items.reserve((size_t)n_blocks + 16);
    for (int32_t b = 0; b < n_blocks; ++b) {  // divided blocks first: theirs are the longest items
      const int64_t c = cost_of(b);
      if (c <= most) continue;
      const int32_t t0 = block_tile[b], n = tiles_of(b);
      const int32_t parts = (int32_t)std::min<int64_t>(n, (c + most - 1) / most);
      divided.push_back(make_int4(b, p->n_parts, parts, 0));
      for (int32_t i = 0; i < parts; ++i) {
        const int32_t lo = (int32_t)((int64_t)n * i / parts), hi = (int32_t)((int64_t)n * (i + 1) / parts);
        items.push_back({b, t0 + lo, hi - lo, p->n_parts++});
      }
    }
    // Then the others, longest first (by 1024 classes of work), so that what the last workgroups leave idle is small: 93,773 rows, 51
    // relations, 4.76 M entries, 32 x 32, 1477 blocks of 52 to 204 tiles in two turns of the CUs: 104 -> 98 us.
    constexpr int kClasses = 1024;
    std::vector<int32_t> class_end(kClasses + 1, 0);
    auto class_of = [&](int64_t c) { return (int)((most - c) * (kClasses - 1) / most); };
    for (int32_t b = 0; b < n_blocks; ++b)
      if (cost_of(b) <= most) ++class_end[class_of(cost_of(b)) + 1];
    for (int i = 0; i < kClasses; ++i) class_end[i + 1] += class_end[i];
    const size_t n_before = items.size();
    items.resize(n_before + (size_t)class_end[kClasses]);
    for (int32_t b = 0; b < n_blocks; ++b)
      if (cost_of(b) <= most) items[n_before + (size_t)class_end[class_of(cost_of(b))]++] = {b, block_tile[b], tiles_of(b), -1};
    p->n_items = (int32_t)items.size();
    p->n_divided = (int32_t)divided.size();

    // ---- the handle's arrays
    size_t bytes = 0;
    const size_t o_tiles = reserve(&bytes, sizeof(RgmsTile) * (size_t)p->n_tiles);
    const size_t o_entries = reserve(&bytes, sizeof(int2) * 4 * (size_t)n_steps);
    const size_t o_items = reserve(&bytes, sizeof(RgmsItem) * items.size());
    const size_t o_divided = reserve(&bytes, sizeof(int4) * divided.size());
    const size_t o_partial = reserve(&bytes, sizeof(float) * ((size_t)p->n_parts * workspace_d_out * p->block_rows));
    bytes = std::max<size_t>(bytes, 256);
    p->blob = p->alloc(bytes, p->alloc_ctx, stream);
    if (!p->blob) { st = SPTIR_ERR_ALLOC; goto fail; }
    p->device_bytes = bytes;
    char* base = (char*)p->blob;
    p->tiles = (RgmsTile*)(base + o_tiles);
    p->entries = (int2*)(base + o_entries);
    p->items = (RgmsItem*)(base + o_items);
    p->divided = (int4*)(base + o_divided);
    p->partial = (float*)(base + o_partial);
    if (p->n_tiles > 0)
      hipLaunchKernelGGL(k_fill_tiles, dim3((unsigned)cell_wgs), dim3(256), 0, stream, ca, stacked->indices, stacked->values,
                         d_cells, d_cell_steps, p->tiles, p->entries);
    RGMS_HIP(hipGetLastError());
    if (!items.empty())
      RGMS_HIP(hipMemcpyAsync(p->items, items.data(), sizeof(RgmsItem) * items.size(), hipMemcpyHostToDevice, stream));
    if (!divided.empty())
      RGMS_HIP(hipMemcpyAsync(p->divided, divided.data(), sizeof(int4) * divided.size(), hipMemcpyHostToDevice, stream));
    RGMS_HIP(hipStreamSynchronize(stream));  // (also: the host vectors go out of scope)
  }
  scratch_free(tmp, p->free_, p->alloc_ctx);
  pinned_release(host);
  *out = p;
  return SPTIR_OK;

fail:
  (void)hipStreamSynchronize(stream);
  scratch_free(tmp, p->free_, p->alloc_ctx);
  pinned_release(host);
  sptir_rgms_destroy(p);
  return st;
#undef RGMS_HIP
}

extern "C" sptir_status_t sptir_rgms(const sptir_rgms_t* p, const float* X, const float* W, float* Y, int32_t d_in,
                                     int32_t d_out, void* stream_) {
  if (!p || d_in < 1 || d_out < 1) return SPTIR_ERR_INVALID_ARG;
  if (p->n_rows == 0) return SPTIR_OK;
  if (!Y || (p->nnz > 0 && (!X || !W))) return SPTIR_ERR_INVALID_ARG;
  if ((d_in != 32 && d_in != 64 && d_in != 128) || d_out % 32 != 0 || (((uintptr_t)X) & 15) != 0)
    return SPTIR_ERR_UNSUPPORTED;
  hipStream_t stream = (hipStream_t)stream_;
  RgmsArgs a;
  a.items = p->items; a.tiles = p->tiles; a.entries = p->entries;
  a.X = X; a.W = W; a.Y = Y; a.partial = p->partial;
  a.n_rows = p->n_rows; a.block_rows = p->block_rows; a.d_out = d_out;
  const bool large_block = is_large_block(p->block_rows);
  a.width = std::min<int32_t>(d_out, columns_beside(p->block_rows));
  const int64_t chunks = (d_out + a.width - 1) / a.width;
  if (chunks > 65535) return SPTIR_ERR_OVERFLOW;
  const bool ordered = d_out <= p->workspace_d_out;
  // Where the matrices W[r] are large (32 KB and up, more than L1 holds) the tiles are long, and a few hundred workgroups
  // leave the CUs unevenly filled: items are then shared by up to four, eight wavefronts each, whose sums meet in Y by
  // atomics.  An item takes about 0.12 us for 1000 elements of W that its tiles read; shared by s it takes an s-th of that, 8 us for the launch that
  // clears Y and 24 + 6 s us for a million elements of Y, cleared and added to: the s for which that is least.  98 drawn graphs: 1.09 times
  // as fast in the mean as with none shared (0.82 to 1.94), the best s for each 1.12.  (By the elements of W alone, two from 200,000 on and one more
  // for every further 250,000: 1.00 on 49 of them (0.50 to 1.53).  32,415 rows, 64 x 128, 471,000: 60 us alone, 119 by two; 7,119 rows, 128 x 128,
  // 2.7 million: 420 alone, 300 by two, 240 by four.)  Where there are fewer than 160 row blocks all are divided into items already; blocks of 512 rows have
  // 16 wavefronts as it is.
  const int64_t whole = (int64_t)p->n_items * chunks;
  const bool large_w = d_in * d_out >= 64 * 128;
  const int64_t tiles_each = p->n_tiles / std::max<int64_t>(p->n_items, 1), w_each = tiles_each * d_in * d_out;
  const bool undivided = ((int64_t)p->n_rows - 1) / p->block_rows >= 159 && !large_block;
  a.sharers = 1;
  if (!ordered && large_w && undivided && whole < 512) {
    const double alone = 0.12e-3 * (double)w_each, y = 1e-6 * (double)p->n_rows * d_out;
    double least = alone;
    for (int32_t n = 2; n <= 4; ++n) {
      const double shared = alone / n + 8. + (24. + 6. * n) * y;
      if (shared < least) { least = shared; a.sharers = n; }
    }
  }
  a.n_waves = wavefronts_per_workgroup(large_block, large_w, whole * a.sharers, tiles_each / a.sharers, ordered);
  const size_t lds = sizeof(double) * (size_t)a.width * ((size_t)p->block_rows + 1) + (ordered ? sizeof(int) * (a.width / 16) : 0);
  const dim3 grid((unsigned)(p->n_items * a.sharers), (unsigned)chunks), block(64 * a.n_waves);
  auto divided = [&](const float* partial) {
    if (p->n_divided > 0)
      hipLaunchKernelGGL(k_rgms_divided, dim3((unsigned)p->n_divided, 16), dim3(256), 0, stream, p->divided, p->n_rows,
                         p->block_rows, d_out, partial, Y);
  };
  if (a.sharers > 1) {
    const int64_t n = (int64_t)p->n_rows * d_out;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256), 0, stream, Y, n);
  } else if (!ordered) {
    divided(nullptr);
  }
  auto launch_for = [&](auto ord, auto wide) {
    constexpr bool kOrdered = decltype(ord)::value, kWide = decltype(wide)::value;
    if (d_in == 32) launch_rgms<1, kOrdered, kWide>(grid, block, lds, stream, a);
    else if (d_in == 64) launch_rgms<2, kOrdered, kWide>(grid, block, lds, stream, a);
    else launch_rgms<4, kOrdered, kWide>(grid, block, lds, stream, a);
  };
  // (a buffer has a 32-bit size)
  const uint64_t x_bytes = (uint64_t)p->n_cols * d_in * sizeof(float);
  const bool wide_x = x_bytes > 0xFFFFFFFFull;
  a.x_bytes = wide_x ? 0 : (uint32_t)x_bytes;
  if (ordered) wide_x ? launch_for(std::true_type{}, std::true_type{}) : launch_for(std::true_type{}, std::false_type{});
  else wide_x ? launch_for(std::false_type{}, std::true_type{}) : launch_for(std::false_type{}, std::false_type{});
  if (ordered) divided(p->partial);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}
