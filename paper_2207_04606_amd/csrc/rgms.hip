// Relational gather-matmul-scatter (RGMS, section 4.4 of arXiv 2207.04606):
//     Y[i,l] = sum_r sum_j sum_k A[r,i,j] * X[j,k] * W[r,k,l].
// The paper decomposes every relation's matrix into hyb(1, 5), gathers the
// rows of X, multiplies by W[r] on the matrix cores and scatters into Y, all in
// one kernel, so that T[r] = X W[r] never exists in memory.
//
// Here the kernel is stationary in Y instead of in r.  A arrives as one CSR
// over stacked rows r*n + i.  Rows of Y are cut into blocks of 2^s; a
// workgroup owns a block, keeps its rows of Y in LDS, walks the block's pairs
// (r, i) relation after relation and writes Y once.  The scatter of the
// relation-stationary order (a float atomic per element of every pair's product
// row, at L2) was what bound it.  32 x 32 features: 94 K rows, 51 relations, 4.76 M entries 0.257 -> 0.159 ms; 1.38 M rows, 25
// relations, 5.6 M entries 0.472 -> 0.294; 1.9 M rows, 96 relations, 5.7 M entries 0.560 -> 0.503, where a
// (relation, block) has few entries and what bounds the kernel is the trips to L2 for W[r].  Over 250 graphs and feature
// sizes it is 1.22 times as fast in the mean (1.5 to 2 with a workspace), but 58 of them lost: a tile reads all of W[r] however
// few pairs it holds, where the relation-stationary tiles held 32, so wide W[r] with few entries per (relation, block) take up
// to 2.3 times as long (1.7 M rows, 54 relations, 1.4 M entries, 128 x 128: 1.07 -> 2.43 ms; 9,788 rows, 52 relations, 30 K entries, 64 x 64:
// 19 -> 35 us).
//
// The entries of (relation, block) are consecutive in the stacked CSR, so the handle needs little more than a copy of the
// entries in their order.  A piece is the entries of one pair (longer pairs are several pieces of 8), a tile up to
// 16 consecutive pieces of one relation in one block.  A wavefront takes a tile:
//   gather    Z^T = X^T S on the matrix cores, four entries a step: S holds the value of an entry in the column of its
//             piece.  Lane (m, q) brings the features of entry q that are its row of X^T, so every load is whole rows of X
//             and nothing but rows that are needed: L1 returns 64 bytes a cycle, and loads laid out by piece, a
//             row per four lanes and most of them masked off, were what bound an earlier form (84 % of its
//             time).  Z comes out as the A operand of the next product;
//   multiply  Z W[r], v_mfma_f32_16x16x4_f32, float32 throughout, W[r] from L1 / L2, where the tiles of one relation
//             that a workgroup's wavefronts take together meet;
//   add       the 16 x 32 results to the block's rows in LDS, as float64 atomics: ds_add_f64 takes 21 cycles a
//             wavefront, ds_add_f32 193 (measured), and the sums lose nothing.
// Blocks are as large as gives (relation, block) a tile's worth of pieces, and small enough that there are workgroups
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

#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

constexpr int kTileRows = 16;      // pieces per tile: the rows of one matrix-core product
constexpr int kPieceEntries = 8;   // most entries per piece: at most two batches of 64 per tile
constexpr int kNoRow = 0xFFFF;
constexpr int kMinLog2Block = 5, kMaxLog2Block = 9;
constexpr int kYTileBytes = 64 * 1024;  // LDS for the rows of Y: two workgroups per CU; blocks of 2^kMaxLog2Block rows: twice that, one

struct RgmsItem {
  int32_t block;    // rows block << log2_block .. of Y
  int32_t tile0;
  int32_t n_tiles;
  int32_t part;     // -1: the whole block; otherwise number of this item among the items of divided blocks
};

struct RgmsTile {
  int32_t first, end;  // its entries
  int32_t rel;
  int32_t pad_;
};

struct RgmsArgs {
  const RgmsItem* items;
  const RgmsTile* tiles;
  const ushort4* tile_rows;  // [n_tiles][4]: the row in the block of each of the tile's 16 pieces, kNoRow: none
  const int2* entries;       // column, value bits
  const uint8_t* entry_piece;  // which of its tile's pieces an entry belongs to
  const float* X;
  const float* W;
  float* Y;
  float* partial;           // ORDERED: sums of the items of divided blocks
  int32_t n_rows;
  int32_t log2_block;
  int32_t d_out;
  int32_t width;            // columns of Y per workgroup, a multiple of 32
  int32_t n_waves;          // per workgroup
  int32_t sharers;          // workgroups per item
  uint32_t x_bytes;
};

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Place in the LDS tile: an instruction adds to 16 columns of any four rows; every other row has its halves of 32 columns
// swapped, so that the four are spread over all banks.
__device__ __forceinline__ int y_index(int row, int col, int width) { return row * width + (col ^ ((row & 1) << 4)); }

// f(0), f(1), .. f(N - 1) with the number as a type
template <int N, typename F, int I = 0>
__device__ __forceinline__ void for_steps(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    for_steps<N, F, I + 1>(std::forward<F>(f));
  }
}

// An entry of a tile as lane (m, q) holds it: number 4 m + q of a batch of 64.
struct Entry {
  int col;
  float val;
  int piece;  // (past the end of the tile: a piece that is none of the 16)
};

// lane S of every 16
template <int S>
__device__ __forceinline__ int bcast16(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + S, 0xF, 0xF, true);  // row_newbcast:S
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

constexpr int kPass = 32;       // columns of Y per pass: two products side by side

// TIN: d_in / 32.  Lane (m, q) = 16 q + m of a 16x16x4 product holds row m of A and column m of B at k = q, and rows
// 4 q .. + 3 of column m of the result.  The features are dealt to the rows of X^T so that a lane's are consecutive:
// row m of product (g, l) is feature 16 VW g + VW m + l.  Column m of product j of a pass over Y stands for the pass's
// column 4 (m & 7) + 2 (m >> 3) + j: that is what the lanes hold after a load of 16 consecutive bytes each (see
// load_w).  In the LDS tile the columns lie in the order of the products.
// WIDE_X: X has 4 GB or more.
template <int TIN, bool ORDERED, bool WIDE_X>
__global__ __launch_bounds__(1024) void k_rgms(RgmsArgs a) {
  constexpr int VW = TIN == 1 ? 2 : 4;              // floats per lane and load of a row of X
  constexpr int kLoads = 2 * TIN / VW;              // loads per row
  constexpr int kZ = 2 * TIN;                       // 16-feature products per step
  constexpr int kAhead = TIN <= 2 ? 8 : 4;                        // steps of four entries whose rows are in flight together
  constexpr int kDin = 32 * TIN, kRowBytes = 4 * kDin;
  extern __shared__ __align__(16) double y_tile[];  // [rows][width], then ORDERED: turn[width / kPass]
  RgmsItem item = a.items[blockIdx.x / (unsigned)a.sharers];
  if (a.sharers > 1) {
    const int part = (int)(blockIdx.x % (unsigned)a.sharers), n = item.n_tiles;
    const int lo = (int)((int64_t)n * part / a.sharers);
    item.n_tiles = (int)((int64_t)n * (part + 1) / a.sharers) - lo;
    item.tile0 += lo;
    item.part = 0;  // (its sums are added to Y)
  }
  const int rows = 1 << a.log2_block, width = a.width;
  const int n0 = blockIdx.y * width;
  const int cols = min(width, a.d_out - n0);
  int* turn = reinterpret_cast<int*>(y_tile + rows * width);
  for (int i = threadIdx.x * 2; i < rows * width; i += blockDim.x * 2)
    *reinterpret_cast<double2*>(y_tile + i) = make_double2(0., 0.);
  if (ORDERED && threadIdx.x < (unsigned)(width / kPass)) turn[threadIdx.x] = 0;
  __syncthreads();

  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), n_waves = a.n_waves;

  // A tile's loads depend on each other (the tile, its entries, the rows those name), each a trip past L2, so they run
  // ahead by three tiles, two and one: what is issued while tile t is multiplied has arrived when t + 1 begins.
  auto tile_number = [&](int t) { return item.tile0 + (t < item.n_tiles ? t : 0); };
  auto load_tile = [&](int t) -> RgmsTile { return a.tiles[tile_number(t)]; };
  auto load_rows = [&](int t) -> ushort4 { return a.tile_rows[(size_t)tile_number(t) * 4 + q]; };
  auto load_entry = [&](const RgmsTile& t, int batch) -> Entry {
    const int i = t.first + 64 * batch + 4 * m + q, at = min(i, t.end - 1);
    const int2 e = a.entries[at];
    const int p = a.entry_piece[at];
    return Entry{e.x, __int_as_float(e.y), i < t.end ? p : kNoRow};
  };
  const __amdgpu_buffer_rsrc_t x_buf = buffer_of(a.X, a.x_bytes);
  auto load_x = [&](int col, float (&x)[kLoads][VW]) {
    typedef float vec __attribute__((ext_vector_type(VW)));
#pragma unroll
    for (int g = 0; g < kLoads; ++g) {
      vec v;
      if constexpr (WIDE_X) v = *reinterpret_cast<const vec*>(a.X + (size_t)col * kDin + VW * m + 16 * VW * g);
      else if constexpr (VW == 2)
        v = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(x_buf, (int)((unsigned)col * kRowBytes + 8u * m), 128 * g, 0));
      else
        v = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(x_buf, (int)((unsigned)col * kRowBytes + 16u * m), 256 * g, 0));
#pragma unroll
      for (int l = 0; l < VW; ++l) x[g][l] = v[l];
    }
  };
  // the rows of X of steps S0 .. S0 + kAhead - 1 of a batch with n entries left (steps past them: nothing)
  float x[kAhead][kLoads][VW];
  auto load_steps = [&](auto s0, const Entry& e, int n) {
    for_steps<kAhead>([&](auto i) {
      constexpr int S = decltype(s0)::value + decltype(i)::value;
      if (4 * S < n) load_x(bcast16<S>(e.col), x[decltype(i)::value]);
    });
  };
  floatx4 z[kLoads][VW];
  auto sum_steps = [&](auto s0, const Entry& e, int n) {
    for_steps<kAhead>([&](auto i) {
      constexpr int S = decltype(s0)::value + decltype(i)::value;
      if (4 * S < n) {
        const float v = __int_as_float(bcast16<S>(__float_as_int(e.val)));
        const float b = bcast16<S>(e.piece) == m ? v : 0.f;
#pragma unroll
        for (int g = 0; g < kLoads; ++g)
#pragma unroll
          for (int l = 0; l < VW; ++l)
            z[g][l] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[decltype(i)::value][g][l], b, z[g][l], 0, 0, 0);
      }
    });
  };
  auto sum_rest = [&](const Entry& e, int n) {  // the steps of a batch that were not loaded ahead
    for_steps<16 / kAhead - 1>([&](auto c) {
      constexpr int S0 = (decltype(c)::value + 1) * kAhead;
      if (4 * S0 < n) {
        load_steps(std::integral_constant<int, S0>{}, e, n);
        sum_steps(std::integral_constant<int, S0>{}, e, n);
      }
    });
  };
  // W[r], part (g, l): the rows k = 16 VW g + VW (4 q + i) + l, i = 0 .. 3, that meet z[g][l][i].  Parts l and l + 1
  // are loaded together, a pair of rows (k, k + 1) at a time: lanes m < 8 take row k, the others k + 1, eight lanes to 128
  // consecutive bytes; take_w then trades halves between lanes m and m ^ 8, so that every lane holds two columns
  // of both rows.  (A lane loading its own two columns of one row costs L1 twice the cycles.)
  const bool upper = (m & 8) != 0;
  const int w_lane = 4 * ((4 * VW * q + (m >> 3)) * a.d_out + 4 * (m & 7));
  auto load_w = [&](int rel, int c0, int part, float4 (&wb)[4]) {  // part: number of a pair of parts
    const int g = part / (VW / 2), l = part % (VW / 2) * 2;
    const __amdgpu_buffer_rsrc_t w_buf = buffer_of(a.W + (size_t)rel * kDin * (size_t)a.d_out, (uint32_t)(kRowBytes * a.d_out));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      wb[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(
                                             w_buf, w_lane, 4 * ((16 * VW * g + VW * i + l) * a.d_out + n0 + c0), 0));
  };
  auto take_w = [&](const float4 w, float2& even, float2& odd) {
    auto pick = [&](float when_upper, float otherwise) { return upper ? when_upper : otherwise; };
    auto other_half = [&](float v) {  // lane m ^ 8's: row_ror:8
      return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, true));
    };
    const float here_x = other_half(pick(w.x, w.z)), here_y = other_half(pick(w.y, w.w));
    even = make_float2(pick(here_x, w.x), pick(here_y, w.y));
    odd = make_float2(pick(w.z, here_x), pick(w.w, here_y));
  };
  constexpr int kParts = kZ / 2, kHeld = kParts < 2 ? kParts : 2;  // pairs of parts of W, and how many are held at a time

  using std::integral_constant;
  if (wave < item.n_tiles) {
    RgmsTile tile = load_tile(wave), tile_1 = load_tile(wave + n_waves), tile_2 = load_tile(wave + 2 * n_waves);
    Entry e = load_entry(tile, 0), e_1 = load_entry(tile_1, 0);
    ushort4 rows_now = load_rows(wave), rows_next;
    float4 w[kHeld][4];  // a part is loaded anew as soon as it is used
    load_steps(integral_constant<int, 0>{}, e, tile.end - tile.first);
#pragma unroll
    for (int p = 0; p < kHeld; ++p) load_w(tile.rel, 0, p, w[p]);
    for (int t = wave; t < item.n_tiles; t += n_waves) {
      // ---- gather
#pragma unroll
      for (int g = 0; g < kLoads; ++g)
#pragma unroll
        for (int l = 0; l < VW; ++l) z[g][l] = floatx4{0.f, 0.f, 0.f, 0.f};
      const int n = tile.end - tile.first;
      sum_steps(integral_constant<int, 0>{}, e, n);
      sum_rest(e, n);
#pragma unroll 1
      for (int batch = 1; 64 * batch < n; ++batch) {
        const Entry more = load_entry(tile, batch);
        load_steps(integral_constant<int, 0>{}, more, n - 64 * batch);
        sum_steps(integral_constant<int, 0>{}, more, n - 64 * batch);
        sum_rest(more, n - 64 * batch);
      }
      // ---- what the next tiles need
      load_steps(integral_constant<int, 0>{}, e_1, tile_1.end - tile_1.first);
      e = e_1;
      e_1 = load_entry(tile_2, 0);
      rows_next = load_rows(t + n_waves);
      const int rel = tile.rel, rel_next = tile_1.rel;
      tile = tile_1; tile_1 = tile_2;
      tile_2 = load_tile(t + 3 * n_waves);
      const int y_row[4] = {rows_now.x, rows_now.y, rows_now.z, rows_now.w};
      // ---- multiply, a pass at a time
#pragma unroll 1
      for (int c0 = 0; c0 < cols; c0 += kPass) {
        const bool last = c0 + kPass >= cols;
        const int rel_then = last ? rel_next : rel, c_then = last ? 0 : c0 + kPass;
        floatx4 d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
          constexpr int kPairs = VW / 2;
          const int g = p / kPairs, l = p % kPairs * 2;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float2 even, odd;
            take_w(w[p % kHeld][i], even, odd);
            d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(z[g][l][i], even.x, d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(z[g][l][i], even.y, d1, 0, 0, 0);
            d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(z[g][l + 1][i], odd.x, d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(z[g][l + 1][i], odd.y, d1, 0, 0, 0);
          }
          if (p + kHeld < kParts) load_w(rel, c0, p + kHeld, w[p % kHeld]);
          else load_w(rel_then, c_then, p + kHeld - kParts, w[p % kHeld]);
        }
        // ---- add: d[v] belongs to piece 4q + v
        if constexpr (ORDERED) {
          // tile t adds after tile t - 1, which an earlier turn of this loop or another wavefront of this workgroup
          // is on its way to: the wait ends
          while (__hip_atomic_load(turn + c0 / kPass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != t)
            __builtin_amdgcn_s_sleep(1);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (y_row[v] != kNoRow) {
            double* y = y_tile + y_row[v] * width + c0 + m;
            const int half = (y_row[v] & 1) << 4;
            atomicAdd(y + half, (double)d0[v]);
            atomicAdd(y + (half ^ 16), (double)d1[v]);
          }
        if constexpr (ORDERED) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");  // (LDS only: the prefetches stay in flight)
          if (lane == 0)
            __hip_atomic_store(turn + c0 / kPass, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
      rows_now = rows_next;
    }
  }
  __syncthreads();

  // ---- what is left (in a scope of its own: anything kept since the loop above costs registers in it)
  {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    // The gather multiplies an entry's row of X with the value 0 for the pieces it does not belong to, and a lane past the end
    // of a tile does so with the tile's last row: a NaN or an infinity in a row of X has reached every pair of the tile.  Sums
    // that are not finite are therefore formed again before they are written, from their own row's entries only; the
    // wavefront takes a row of the block at a time.  y[0 .. 3] of a lane: columns n0 + c .. + 3 of row `row`.  (Testing every
    // tile's sums in front of its product instead: 0.505 -> 0.542 ms on 1.9 M rows; here the test does not show.)
    auto sum_again = [&](int row, int c, bool not_finite, float (&y)[4]) {
      unsigned long long todo = __ballot(not_finite);
      while (todo) {
        const int r = __builtin_amdgcn_readlane(row, __builtin_ctzll(todo));
        const bool here = not_finite && row == r;
        todo &= ~__ballot(here);
        double sum[4] = {0., 0., 0., 0.};
        for (int t0 = 0; t0 < item.n_tiles; t0 += 64) {
          bool has = false;  // a piece of row r in tile t0 + lane
          if (t0 + lane < item.n_tiles)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const ushort4 of = a.tile_rows[(size_t)(item.tile0 + t0 + lane) * 4 + i];
              has |= of.x == r || of.y == r || of.z == r || of.w == r;
            }
          for (unsigned long long tiles = __ballot(has); tiles; tiles &= tiles - 1) {
            const int t = item.tile0 + t0 + __builtin_ctzll(tiles);
            const RgmsTile tile = a.tiles[t];
            const int of_slot = reinterpret_cast<const uint16_t*>(a.tile_rows + (size_t)t * 4)[lane & 15];
            const unsigned slots = (unsigned)__ballot(of_slot == r) & 0xFFFFu;
            constexpr int kPerLane = (kDin + 63) / 64;
            float sums[kPerLane];  // features lane, lane + 64
#pragma unroll
            for (int i = 0; i < kPerLane; ++i) sums[i] = 0.f;
            for (int first = tile.first; first < tile.end; first += 64) {
              const int at = min(first + lane, tile.end - 1);
              const int2 e = a.entries[at];
              const bool take = first + lane < tile.end && (slots >> a.entry_piece[at] & 1u) != 0;
              for (unsigned long long left = __ballot(take); left; left &= left - 1) {
                const int from = __builtin_ctzll(left);
                const float* x_row = a.X + (size_t)__builtin_amdgcn_readlane(e.x, from) * kDin;
                const float v = __int_as_float(__builtin_amdgcn_readlane(e.y, from));
#pragma unroll
                for (int i = 0; i < kPerLane; ++i) sums[i] = fmaf(v, x_row[(64 * i + lane) % kDin], sums[i]);
              }
            }
            const float* w = a.W + (size_t)tile.rel * kDin * (size_t)a.d_out + n0 + c;
            float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kPerLane; ++i)
#pragma unroll 4
              for (int k = 0; k < (kDin < 64 ? kDin : 64); ++k) {
                const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sums[i]), k));
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = fmaf(s, w[(size_t)(64 * i + k) * a.d_out + j], d[j]);
              }
#pragma unroll
            for (int j = 0; j < 4; ++j) sum[j] += d[j];
          }
        }
        if (here) {
#pragma unroll
          for (int j = 0; j < 4; ++j) y[j] = (float)sum[j];
        }
      }
    };

    // ---- the block's rows
    const int row0 = item.block << a.log2_block;
    const int rows_here = min(rows, a.n_rows - row0);
    const int quads = cols / 4;
    const int n_quads = rows_here * quads;
    // (whole wavefronts: sum_again needs all lanes)
    for (int i0 = __builtin_amdgcn_readfirstlane(tid); i0 < n_quads; i0 += (int)blockDim.x) {
      const int i = min(i0 + lane, n_quads - 1);
      const int row = i / quads, c = (i - row * quads) * 4;
      float y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int p = (c + k) % kPass;
        y[k] = (float)y_tile[y_index(row, c + k - p + 16 * (p & 1) + 8 * ((p >> 1) & 1) + (p >> 2), width)];
      }
      const bool not_finite = fmaf(y[0], 0.f, fmaf(y[1], 0.f, fmaf(y[2], 0.f, y[3] * 0.f))) != 0.f;
      if (__any(not_finite)) sum_again(row, c, not_finite, y);
      if (i0 + lane >= n_quads) continue;
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
                                                      int32_t log2_block, int32_t d_out,
                                                      const float* __restrict__ partial, float* Y) {
  const int4 d = divided[blockIdx.x];
  const int row0 = d.x << log2_block, rows = min(1 << log2_block, n_rows - row0);
  for (int i = threadIdx.x; i < rows * d_out; i += blockDim.x) {
    float sum = 0.f;
    if (partial)
      for (int p = 0; p < d.z; ++p) sum += partial[(((size_t)(d.y + p)) << log2_block) * d_out + i];
    Y[(size_t)row0 * d_out + i] = sum;
  }
}

// ------------------------------------------------------------------- build
// cells are (block, relation), block-major; one wavefront each
struct CellArgs {
  const int32_t* indptr;
  int64_t n_cells;
  int32_t n_rel, n_rows, log2_block, k;
};
constexpr int kCountSlots = 64, kCountStride = 8;

// tiles of every cell, entries of every block (zeroed before); counts[slot][0] += pairs with entries, [1] += slots of padding that hyb(1, k) has for them
__global__ __launch_bounds__(256) void k_cell_tiles(CellArgs a, int32_t* cell_tiles, int32_t* block_entries,
                                                    unsigned long long* counts) {
  const int lane = threadIdx.x & 63;
  const int64_t cell = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cell >= a.n_cells) return;
  const int64_t block = cell / a.n_rel, rel = cell - block * a.n_rel;
  const int64_t row0 = block << a.log2_block;
  const int rows = (int)min((int64_t)1 << a.log2_block, (int64_t)a.n_rows - row0);
  const int32_t* ptr = a.indptr + rel * a.n_rows + row0;
  int pieces = 0, pairs = 0, pads = 0;
  for (int i = lane; i < rows; i += 64) {
    const int len = ptr[i + 1] - ptr[i];
    pieces += (len + kPieceEntries - 1) / kPieceEntries;
    pairs += len > 0;
    if (len > 1) {
      const int log2w = 32 - __clz(len - 1);
      if (log2w <= a.k) pads += (1 << log2w) - len;
    }
  }
  for (int d = 32; d > 0; d >>= 1) {
    pieces += __shfl_down(pieces, d, 64);
    pairs += __shfl_down(pairs, d, 64);
    pads += __shfl_down(pads, d, 64);
  }
  if (lane == 0) {
    cell_tiles[cell] = (pieces + kTileRows - 1) / kTileRows;
    const int entries = ptr[rows] - ptr[0];
    if (entries > 0) atomicAdd(&block_entries[block], entries);
    unsigned long long* c = counts + (blockIdx.x & (kCountSlots - 1)) * kCountStride;
    if (pairs) atomicAdd(&c[0], (unsigned long long)pairs);
    if (pads) atomicAdd(&c[1], (unsigned long long)pads);
  }
}

// block_tile[b] = first tile of block b (b = n_blocks: their number)
__global__ void k_block_tiles(int32_t n_blocks, int32_t n_rel, const int32_t* __restrict__ cell_tile0,
                              const int32_t* __restrict__ total, int32_t* block_tile) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b <= n_blocks) block_tile[b] = b < n_blocks ? cell_tile0[(int64_t)b * n_rel] : *total;
}

// the tiles of every cell: pieces in row order
__global__ __launch_bounds__(256) void k_fill_tiles(CellArgs a, const int32_t* __restrict__ cell_tile0,
                                                    const int32_t* __restrict__ total, RgmsTile* tiles,
                                                    uint16_t* tile_rows, uint8_t* entry_piece) {
  const int lane = threadIdx.x & 63;
  const int64_t cell = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cell >= a.n_cells) return;
  const int64_t block = cell / a.n_rel, rel = cell - block * a.n_rel;
  const int tile0 = cell_tile0[cell], tile_end = cell + 1 < a.n_cells ? cell_tile0[cell + 1] : *total;
  if (tile0 == tile_end) return;
  const int64_t row0 = block << a.log2_block;
  const int rows = (int)min((int64_t)1 << a.log2_block, (int64_t)a.n_rows - row0);
  const int32_t* ptr = a.indptr + rel * a.n_rows + row0;
  const int cell_end = ptr[rows];
  uint16_t* out = tile_rows + (size_t)tile0 * kTileRows;
  for (int t = tile0 + lane; t < tile_end; t += 64) tiles[t].rel = (int)rel;
  int done = 0;
  for (int i0 = 0; i0 < rows; i0 += 64) {
    const int i = i0 + lane;
    int first = 0, len = 0;
    if (i < rows) { first = ptr[i]; len = ptr[i + 1] - first; }
    const int n = (len + kPieceEntries - 1) / kPieceEntries;
    const int incl = wave_inclusive_scan(n, lane);
    const int slot0 = done + incl - n;
    for (int p = 0; p < n; ++p) {
      const int slot = slot0 + p, at = first + p * kPieceEntries, end = min(at + kPieceEntries, first + len);
      out[slot] = (uint16_t)i;
      RgmsTile* t = tiles + tile0 + slot / kTileRows;
      if (slot % kTileRows == 0) t->first = at;
      if (slot % kTileRows == kTileRows - 1 || end == cell_end) t->end = end;
    }
    // an entry's piece, 64 entries of a row at a time (short rows: a lane each)
    if (len <= 8)
      for (int k = 0; k < len; ++k) entry_piece[first + k] = (uint8_t)(slot0 % kTileRows);
    unsigned long long longer = __ballot(len > 8);
    while (longer) {
      const int src = __builtin_ctzll(longer);
      longer &= longer - 1;
      const int f = __shfl(first, src, 64), l = __shfl(len, src, 64), s0 = __shfl(slot0, src, 64);
      for (int k = lane; k < l; k += 64) entry_piece[f + k] = (uint8_t)((s0 + k / kPieceEntries) % kTileRows);
    }
    done += __shfl(incl, 63, 64);
  }
  for (int i = done + lane; i < (tile_end - tile0) * kTileRows; i += 64) out[i] = kNoRow;
}

__global__ __launch_bounds__(256) void k_pair_entries(int64_t nnz, const int32_t* __restrict__ cols,
                                                      const float* __restrict__ vals, int2* entries) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nnz) entries[i] = make_int2(cols[i], __float_as_int(vals[i]));
}

// Rows per block: 32 entries for every (relation, block), so that tiles fill (16: 4 to 14 % slower, 64: the same), as long
// as that leaves 160 blocks, about what keeps the matrix cores of 256 CUs busy with 16 wavefronts each.  (60 graphs, 32 x 32: the
// best block for each is 2.7 % faster in the mean, 20 % at most; any one size for all 16 to 34 % slower.)  Fewer,
// larger blocks divided into items were tried and lose more in global atomics than fuller tiles gain (27,163 rows,
// 64 x 64: 0.042 -> 0.093 ms).
// Blocks of 512 rows take the LDS of a CU and 16 wavefronts; what they win is W[r] read for half as many tiles.  They need two
// workgroups' worth of them per CU (158,566 rows: 0.81 times as fast as with 256), no workspace, whose tiles take turns (0.79 to
// 1.08), and fewer than 40 entries for every (relation, block) even so.  78 graphs and feature sizes, against 256 rows: up to 24 entries
// 1.10 times as fast (0.97 to 1.21), to 40 1.03 (0.94 to 1.10; 32 x 32 features 0.98), to 64 0.98 (0.87 to 1.05).  1.9 M rows, 96
// relations, 5.7 M entries, 32 x 32, 16 entries: 0.527 -> 0.458 ms.
int log2_block_rows(int64_t n_rows, int64_t n_rel, int64_t nnz, bool workspace) {
  int s = kMinLog2Block;
  while (((int64_t)1 << s) * nnz < 32 * n_rows * n_rel && s < kMaxLog2Block - 1 && (n_rows >> (s + 1)) >= 160) ++s;
  const bool large = s == kMaxLog2Block - 1 && !workspace && (n_rows >> kMaxLog2Block) >= 512 &&
                     ((int64_t)1 << kMaxLog2Block) * nnz < 40 * n_rows * n_rel;
  return large ? kMaxLog2Block : s;
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
  int32_t log2_block;
  int64_t n_tiles;
  sptir::RgmsTile* tiles;
  uint16_t* tile_rows;    // [n_tiles][16]
  int2* entries;          // [nnz]
  uint8_t* entry_piece;   // [nnz]
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
  o.n_tiles = p->n_tiles; o.workspace_d_out = p->workspace_d_out; o.row_block = 1 << p->log2_block;
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
  p->log2_block = log2_block_rows(p->n_rows, n_relations, nnz, workspace_d_out > 0);
  const int32_t n_blocks = (int32_t)(((int64_t)p->n_rows + (1 << p->log2_block) - 1) >> p->log2_block);
  CellArgs ca;
  ca.indptr = stacked->indptr; ca.n_cells = (int64_t)n_blocks * n_relations; ca.n_rel = n_relations;
  ca.n_rows = p->n_rows; ca.log2_block = p->log2_block; ca.k = k;
  const int64_t cell_wgs = (ca.n_cells + 3) / 4;
  const int64_t n_seq = (int64_t)(scan_room(std::max<int64_t>(ca.n_cells, 1)) / kScanSeq);

  // temporaries: validation flags and counts (one copy brings both to the host), cells, block starts
  constexpr size_t kReport = (kValidationWords + kCountSlots * kCountStride) * sizeof(unsigned long long);
  const size_t cleared = kReport + sizeof(int32_t) * (size_t)n_blocks;
  size_t tmp_bytes = cleared;
  auto reserve = [](size_t* size, size_t bytes) { const size_t at = *size; *size = (at + bytes + 255) & ~(size_t)255; return at; };
  const size_t o_block_tile = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_blocks + 1));
  const size_t report_bytes = o_block_tile + sizeof(int32_t) * ((size_t)n_blocks + 1);
  const size_t o_cells = reserve(&tmp_bytes, sizeof(int32_t) * (size_t)n_seq * kScanSeq);
  const size_t o_seq = reserve(&tmp_bytes, sizeof(int32_t) * ((size_t)n_seq + 1));
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
    int32_t* d_cells = (int32_t*)(tmp + o_cells);
    int32_t* d_seq = (int32_t*)(tmp + o_seq);
    if (cell_wgs > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
    RGMS_HIP(hipMemsetAsync(tmp, 0, cleared, stream));
    launch_validation(stacked, false, d_flags, stream);
    if (ca.n_cells > 0) {
      // (the numbers below mean something only if the verdict is good, and index nothing before it is known)
      hipLaunchKernelGGL(k_cell_tiles, dim3((unsigned)cell_wgs), dim3(256), 0, stream, ca, d_cells,
                         (int32_t*)(tmp + kReport), d_counts);
      RGMS_HIP(hipGetLastError());
      st = device_exclusive_scan(d_cells, ca.n_cells, d_seq, stream);
      if (st != SPTIR_OK) goto fail;
      hipLaunchKernelGGL(k_block_tiles, dim3((unsigned)(n_blocks / 256 + 1)), dim3(256), 0, stream, n_blocks,
                         n_relations, d_cells, d_seq + n_seq, d_block_tile);
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
    p->n_tiles = n_blocks > 0 ? block_tile[n_blocks] : 0;

    // ---- work items: a block each.  A block of more than twice the mean work is divided; where there are few blocks,
    //      all are, into about 512 items.
    const int32_t* block_entries = (const int32_t*)(host.p + kReport);
    auto tiles_of = [&](int32_t b) { return block_tile[b + 1] - block_tile[b]; };
    auto cost_of = [&](int32_t b) { return (int64_t)tiles_of(b) + block_entries[b] / 32; };  // (measured: 32 entries cost about what a tile does)
    const int64_t cost = p->n_tiles + nnz / 32, mean = n_blocks > 0 ? cost / n_blocks : 0;
    const int64_t most = n_blocks >= 160 ? std::max<int64_t>(64, 2 * mean) : std::max<int64_t>(8, cost / 512);
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
    for (int32_t b = 0; b < n_blocks; ++b)
      if (cost_of(b) <= most) items.push_back({b, block_tile[b], tiles_of(b), -1});
    p->n_items = (int32_t)items.size();
    p->n_divided = (int32_t)divided.size();

    // ---- the handle's arrays
    size_t bytes = 0;
    const size_t o_tiles = reserve(&bytes, sizeof(RgmsTile) * (size_t)p->n_tiles);
    const size_t o_rows = reserve(&bytes, sizeof(uint16_t) * (size_t)p->n_tiles * kTileRows);
    const size_t o_entries = reserve(&bytes, sizeof(int2) * (size_t)nnz);
    const size_t o_piece = reserve(&bytes, (size_t)nnz);
    const size_t o_items = reserve(&bytes, sizeof(RgmsItem) * items.size());
    const size_t o_divided = reserve(&bytes, sizeof(int4) * divided.size());
    const size_t o_partial = reserve(&bytes, sizeof(float) * (((size_t)p->n_parts * workspace_d_out) << p->log2_block));
    bytes = std::max<size_t>(bytes, 256);
    p->blob = p->alloc(bytes, p->alloc_ctx, stream);
    if (!p->blob) { st = SPTIR_ERR_ALLOC; goto fail; }
    p->device_bytes = bytes;
    char* base = (char*)p->blob;
    p->tiles = (RgmsTile*)(base + o_tiles);
    p->tile_rows = (uint16_t*)(base + o_rows);
    p->entries = (int2*)(base + o_entries);
    p->entry_piece = (uint8_t*)(base + o_piece);
    p->items = (RgmsItem*)(base + o_items);
    p->divided = (int4*)(base + o_divided);
    p->partial = (float*)(base + o_partial);
    if (p->n_tiles > 0)
      hipLaunchKernelGGL(k_fill_tiles, dim3((unsigned)cell_wgs), dim3(256), 0, stream, ca, d_cells, d_seq + n_seq,
                         p->tiles, p->tile_rows, p->entry_piece);
    if (nnz > 0)
      hipLaunchKernelGGL(k_pair_entries, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, stream, nnz,
                         stacked->indices, stacked->values, p->entries);
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
  a.items = p->items; a.tiles = p->tiles; a.tile_rows = (const ushort4*)p->tile_rows;
  a.entries = p->entries; a.entry_piece = p->entry_piece;
  a.X = X; a.W = W; a.Y = Y; a.partial = p->partial;
  a.n_rows = p->n_rows; a.log2_block = p->log2_block; a.d_out = d_out;
  const bool large_block = p->log2_block == kMaxLog2Block;
  a.width = std::min<int32_t>(d_out, ((large_block ? 2 : 1) * kYTileBytes / 8 >> p->log2_block) / 32 * 32);
  const int64_t chunks = (d_out + a.width - 1) / a.width;
  if (chunks > 65535) return SPTIR_ERR_OVERFLOW;
  const bool ordered = d_out <= p->workspace_d_out;
  // Where the matrices W[r] are large (32 KB and up, more than L1 holds) the tiles are long, and a few hundred workgroups
  // leave the CUs unevenly filled: items are then shared by several, eight wavefronts each, whose sums meet in Y by
  // atomics, until there are 512 (8,370 rows, 128 x 128, 262 items: 0.215 -> 0.168 ms).  Clearing Y and the atomics have to be
  // worth it, so an item needs 200,000 elements of W to read for two sharers and 250,000 more for each further one (27,608
  // rows, 64 x 128, 188,000: 35 us alone, 80 shared by two; 6,903 rows, 128 x 128, 328,000: 75 alone, 62 by two, 72 by three;
  // 6,110 rows, 983,000: 144 alone, 120 by two, 117 by three).  Where there are fewer than 160 row blocks all are
  // divided into items already (26 graphs, shared until there were 512 workgroups: 12 % slower in the mean, up to 1.7 times).
  const int64_t whole = (int64_t)p->n_items * chunks;
  const bool large_w = d_in * d_out >= 64 * 128;
  const int64_t tiles_each = p->n_tiles / std::max<int64_t>(p->n_items, 1), w_each = tiles_each * d_in * d_out;
  const bool undivided = ((int64_t)p->n_rows - 1) >> p->log2_block >= 159;
  a.sharers = 1;
  if (!ordered && large_w && undivided && whole < 512 && w_each >= 200000)
    a.sharers = (int32_t)std::min<int64_t>(std::max<int64_t>(2, w_each / 250000), std::min<int64_t>(8, (512 + whole - 1) / whole));
  // wavefronts per workgroup: 4, unless a workgroup has tiles for more; 16 where one workgroup per CU has to do.  (230 graphs
  // and feature sizes: against 8 everywhere it is alike in the mean, 0.83 to 1.2; 4 everywhere 8 % slower, 16 everywhere 7 %.)
  a.n_waves = large_block ? 16 : large_w ? 8 : whole <= 320 && tiles_each >= 16 ? 16 : tiles_each >= 24 ? 8 : 4;
  const size_t lds = sizeof(double) * ((size_t)a.width << p->log2_block) + (ordered ? sizeof(int) * (a.width / 16) : 0);
  const dim3 grid((unsigned)(p->n_items * a.sharers), (unsigned)chunks), block(64 * a.n_waves);
  auto divided = [&](const float* partial) {
    if (p->n_divided > 0)
      hipLaunchKernelGGL(k_rgms_divided, dim3((unsigned)p->n_divided), dim3(256), 0, stream, p->divided, p->n_rows,
                         p->log2_block, d_out, partial, Y);
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
