// RGMS: rows of Y per block, and how many of its columns fit beside them in LDS.  Plain arithmetic, of the host alone.
#ifndef SPTIR_RGMS_BLOCKS_H_
#define SPTIR_RGMS_BLOCKS_H_

#include <stdint.h>

#include <algorithm>

namespace sptir {
namespace {

constexpr int kMinLog2Block = 5, kMaxLog2Block = 9;
constexpr int kYTileBytes = 64 * 1024;  // LDS for the rows of Y: two workgroups per CU; blocks of 2^kMaxLog2Block rows: twice that, one
constexpr int kHalfLds = 80 * 1024;     // what each of two workgroups can have

inline bool is_large_block(int32_t rows) { return rows > 1 << (kMaxLog2Block - 1); }

// Columns of Y beside so many rows (a multiple of 32): what a pass over X takes.  Rows that are up to a quarter more than a power of two have the columns of that
// power.  (At a quarter, all of these leave a CU one workgroup: more than kHalfLds.)
inline int64_t y_tile_bytes(int32_t rows, int32_t columns) { return (int64_t)sizeof(double) * columns * (rows + 1); }
inline int32_t columns_beside(int32_t rows) {
  int32_t power = 1;
  while (2 * power <= rows) power *= 2;
  const int32_t cols = (is_large_block(rows) ? 2 : 1) * kYTileBytes / 8 / rows / 32 * 32, of_power = kYTileBytes / 8 / power;
  return of_power > cols && 4 * rows <= 5 * power ? of_power : cols;
}

// Rows per block: 32 entries for every (relation, block), so that tiles fill, as long as that leaves 160 blocks, about what keeps
// 256 CUs busy with 16 wavefronts each.  557 pairs of blocks of 32 to 256 rows, the larger against the smaller: with 16 to 24 entries in the
// smaller 1.05 times as fast, with 24 to 32 1.01, with 32 to 48 1.01, with 48 to 64 0.98 (0.74 to 1.45: what decides is whether the last
// turn of workgroups is nearly empty).  16 entries with a workspace: a tile's turn comes sooner where a block has fewer of them.  553 pairs: with
// less than 16 entries in the smaller 0.97, with 16 to 32 0.94 (0.58 to 1.47), with 32 to 64 0.90.
// Fewer, larger blocks divided into items lose more in global atomics than fuller tiles gain (27,163 rows, 64 x 64: blocks of 256 rows 83 us,
// of 128 30).
// Blocks of 512 rows take the LDS of a CU and 16 wavefronts; what they win is W[r] read for half as many tiles, if that is for few entries, and
// twice as many pieces to fill a tile with.  Against 256 rows, without a workspace, 142 graphs and feature sizes of 160 blocks of 512 and more: up
// to 24 entries for every (relation, block) 1.15 times as fast (0.90 to 1.39), however many the blocks; up to 40 entries 1.04 from 384 blocks on
// (0.97 to 1.22), where the last turn of workgroups weighs less, 1.01 below (0.88 to 1.24); up to 64 1.03 (0.88 to 1.34), beyond 1.01 (0.93 to
// 1.27), some of it lost to CUs without work.  Below 160 blocks, where all are divided, 0.39.  117,840 rows, 74 relations,
// 900 K entries, 64 x 64: 131 -> 114 us; 1.9 M rows, 96 relations, 5.7 M entries, 32 x 32, 16 entries: 394 -> 344.  With a workspace tiles take
// turns, and larger blocks lose sooner.
inline int log2_block_rows(int64_t n_rows, int64_t n_rel, int64_t nnz, bool workspace) {
  int s = kMinLog2Block;
  const int64_t enough = workspace ? 16 : 32;
  while (((int64_t)1 << s) * nnz < enough * n_rows * n_rel && s < kMaxLog2Block - 1 && (n_rows >> (s + 1)) >= 160) ++s;
  const int64_t entries = nnz << kMaxLog2Block, blocks = n_rows >> kMaxLog2Block;
  const bool large = s == kMaxLog2Block - 1 && !workspace &&
                     ((blocks >= 160 && entries < 24 * n_rows * n_rel) || (blocks >= 384 && entries < 40 * n_rows * n_rel));
  return large ? kMaxLog2Block : s;
}

// Where that is a few blocks for every CU, as many rows as make it whole turns of the 256 CUs.  Never so many that fewer columns of Y fit beside them than
// beside the power of two: every pass over X that this adds costs as much as the first (64 x 128 features, 522 blocks of 128 rows, 282,624 entries:
// 67 us, 76 by 512 blocks of 131 rows with 32 columns each, 63 with 64).  All against blocks of a power of two rows, without a workspace, by d_in x d_out
// (32 x 32; d_in of 64 and 128 with d_out up to 64; d_out of 128), 430 graphs of 1 to 70 relations:
//   192 to 255 blocks    256              1.02, 1.02, 1.03 times as fast (0.81 to 1.23; what loses has as many tiles in the smaller blocks); 256 of 384 to 510
//                                         rows instead of as many of 512, 60 graphs: 1.05, 1.04, 1.05 (0.96 to 1.14)
//   257 to 320           256              1.14 (0.93 to 1.55; 250 graphs, 1.20 with fewer than 13 entries for every (relation, block); 512 1.07, 0.74 to 1.39)
//   321 to 512           512              1.04, 1.07, 1.06 (0.83 to 1.34)
//   513 to 576           512              1.04, 1.04, 1.03 (0.94 to 1.22)
//   577 to 768           768              1.04, 1.02, 0.99 (0.92 to 1.14)
//   769 to 1300          the nearest of 768 and 1024, up to 948 and from 1025 on, for blocks of fewer than 300 entries, which end as soon as they have begun:
//                                         1.02, 1.02, 1.02 (0.92 to 1.27)
// Blocks of more entries beyond 768 keep the power of two: 768 instead of 769 to 948 of them are 1.04 times as fast with 32 features of X, of which a turn has
// three workgroups of eight wavefronts for every CU, but 0.97 (0.90 to 1.03) with more, where it has two; 1024 are 0.96 to 1.01 with either, also for few entries
// where they stand for fewer.  Below 192 blocks
// tiles lose a quarter of what they hold and more; blocks of 32 rows are as fast or slower by 256 (1.02, 0.82 to 1.16), and 512 instead of 316 to 477 of 256 rows
// 0.94 to 1.20; 1.9 M rows, 3682 blocks of 512 rows 341 us, 3840 of 491 351.  With a workspace one turn only: tiles take their turns longer in larger blocks.
// 27,163 rows, 46 relations, 64 x 64, 213 blocks of 128 rows 28.8 us, 256 of 107 28.1.
constexpr int64_t kMostForOneTurn = 320, kMostForTwoTurns = 576, kMostForAll = 768, kFewEntries = 300;
inline int32_t rows_of_a_block(int64_t n_rows, int64_t n_rel, int64_t nnz, bool workspace) {
  const int s = log2_block_rows(n_rows, n_rel, nnz, workspace);
  const int32_t power = 1 << s;
  const int64_t blocks = (n_rows + power - 1) >> s;
  const bool several = !workspace && s < kMaxLog2Block - 1;
  auto rows_of = [&](int64_t turns) {
    const int32_t rows = (int32_t)((n_rows + 256 * turns - 1) / (256 * turns));
    const int32_t cols = columns_beside(rows);
    const bool two_a_cu = turns == 1 || y_tile_bytes(rows, cols) <= kHalfLds;
    return cols < columns_beside(power) || !two_a_cu || (rows > 128 && power == 128 && turns > 2) ? power : rows;
  };
  if (blocks < 192 || blocks > 1300) return power;
  if (blocks <= 256) return s > kMinLog2Block ? rows_of(1) : power;
  if (!several) return power;
  if (blocks <= kMostForOneTurn) return rows_of(1);
  if (blocks <= kMostForTwoTurns) return rows_of(2);
  if (blocks > kMostForAll && nnz >= kFewEntries * blocks) return power;
  return blocks <= 948 ? rows_of(3) : blocks > 1024 ? rows_of(4) : power;
}

// Where matrices W[r] are large 8, else 4, unless a workgroup has tiles for more; 16 where one workgroup per CU has to do.  (230 graphs and feature sizes: against 8 everywhere it is alike in the
// mean, 0.83 to 1.2; 4 everywhere 8 % slower, 16 everywhere 7 %.)  Fewer tiles than 24 are for 8 wavefronts as well while workgroups are few: a launch is then
// as long as one of them takes (60 drawn graphs of 12,000 rows and more: those of 320 to 1024 workgroups 1.05 to 1.38 times as fast with 8, those of more 0.88 to
// 1.00).  12 tiles and more are for 16, since blocks that make one whole turn have down to three quarters of the tiles of a power of two (see
// rows_of_a_block()): from 16 on, 13,500 rows of 8 relations, 71,720 entries, 64 x 64, took 15.4 us where the power of two took 13.2, now 13.1; 60 graphs with
// d_out up to 64 and 192 to 255 blocks 1.01 times as fast, 60 of fewer 1.00 (0.98 to 1.13).  Where tiles add in their order they wait longer for 16: from 16 on
// (18,484 rows, 9 relations, 59,392 entries, 64 x 64: 18.1 us, 19.7 from 12 on).  The same for large W[r], which had 8 always and one workgroup of them a CU where one
// pass takes all columns: 120 graphs and feature sizes of 165 to 320 blocks 1.06 times as fast (0.96 to 1.40), 16,443 rows, 9 relations, 84,842 entries, 128 x 128
// 45.3 -> 39.4 us.  (workgroups, tiles_each: with the sharers of an item.)
inline int32_t wavefronts_per_workgroup(bool large_block, bool large_w, int64_t workgroups, int64_t tiles_each, bool ordered) {
  if (large_block) return 16;
  if (workgroups <= 320 && tiles_each >= (ordered ? 16 : 12)) return 16;
  if (large_w) return 8;
  return tiles_each >= (workgroups <= 1024 ? 8 : 24) ? 8 : 4;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_RGMS_BLOCKS_H_
