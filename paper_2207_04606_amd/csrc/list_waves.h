// How many wavefronts, each with a chunk list of its own, a workgroup of the SpMM kernels has.  Plain arithmetic, of the host alone.
#ifndef SPTIR_LIST_WAVES_H_
#define SPTIR_LIST_WAVES_H_

#include <stdint.h>

#include <algorithm>

namespace sptir {
namespace {

// the chunk lists of a call
struct ListLaunches {
  bool rounds;
  int32_t n_launches, parts_per_launch;  // of the column partitions
  int64_t n_cols, n_lists;
  int64_t entries, chunks, longest;      // in the lists; the longest list in chunks
  int32_t feat, tile_floats, n_tiles;
};

// Four where the lists of a launch go through slices of X nearly in step, as neighbours then walk the same ones: in rounds (232,965 rows, 114.6 M entries:
// 1791 us, one 1815), and in a single launch over several partitions where the columns of X that a feature tile reads are beyond an L2, there are several tiles,
// and lists are long, or even and not short.  Else one, whose place on the CU is free when it ends (132,534 rows, 39.6 M entries in eight launches: 997 -> 980 us;
// 17,000 rows, 59,069 entries, 117 features 24.3 -> 15.8).
// 217 graphs in a single launch over several partitions, one against four: 74 of at least 300 entries a list, even or 1280 of them, 0.95 times as fast with one
// (0.69 to 1.02; the 41 of them with fewer than 1280 entries 0.976, 0.87 to 1.02), the others 1.02 (0.95 to 1.18; with one feature tile up to 1.18, whatever the
// lists).  What loses below 600 entries with one has tiles of 64 floats; with tiles of 32, 300 to 599 entries take as long with either where columns are alike
// (0.96 to 1.04), and less with one where some are hot (transposed power-law graphs, 35 of them: 1.01, 0.995 to 1.026; from 600 on the same 1.00 to 1.02, columns
// alike 0.91 to 1.0).  From 1280 entries on alone, as this rule began: 126,254 rows, 2.4 M entries, 223 features, 1223 a list, 446 us where four take 365.
constexpr int64_t kBeyondL2 = (int64_t)8 << 20, kLongList = 1280, kEvenList = 600, kEvenListOfHalfRows = 300;
inline int32_t list_waves(const ListLaunches& l) {
  if (l.rounds) return 4;
  const int64_t tile_bytes = (int64_t)sizeof(float) * std::min(l.feat, l.tile_floats) * l.n_cols;
  if (l.n_launches != 1 || l.parts_per_launch < 2 || l.n_tiles < 2 || tile_bytes < kBeyondL2) return 1;
  const bool even = l.longest * l.n_lists <= 2 * l.chunks;
  const int64_t least = !even ? kLongList : l.tile_floats >= 64 ? kEvenListOfHalfRows : kEvenList;
  return l.entries >= least * l.n_lists ? 4 : 1;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_LIST_WAVES_H_
