// Column slices of an SDDMM plan: their width, their layout in LDS, and which kernel takes a call.  No device code, so
// that the choice can be checked for every pair of feature sizes without a GPU.
#ifndef SPTIR_SDDMM_SLICE_SHAPE_H_
#define SPTIR_SDDMM_SLICE_SHAPE_H_

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace sptir {

constexpr int kSliceBytes = 155 * 1024;  // of Yt in LDS; one workgroup a CU (two of 64 KB: 6 % slower, pieces half as long)
constexpr int kColumnBits = 13;          // of a column inside its slice (4 floats: 8192 columns)
constexpr int kLdsMostFeat = 256;        // floats of a row that the eight lanes of a group hold in eight float4 each

// Row to row in LDS, in float4: where all rows would begin in the same half of the 64 banks, half a row of banks more, or the
// lane groups meet in it (random 512-byte rows: 77 TB/s, 85 if half of them begin in the other half).
constexpr int slice_stride(int quads) { return quads % 16 == 0 ? quads + 8 : quads; }

// Columns per slice of a plan made for `feat` features; 0: no slices.
constexpr int32_t slice_width(int64_t feat) {
  if (feat > kLdsMostFeat) return 0;
  const int32_t fit = (int32_t)(kSliceBytes / (16 * slice_stride((int)(feat + 3) / 4))), most = 1 << kColumnBits;
  return fit < most ? fit : most;
}

// Float4 per lane of the kernel that takes a call from LDS, or 0: from memory (k_sddmm_segments), where a row has fewer than
// four floats, or more than a lane group holds, or the plan's slices have no room for it.
constexpr int slice_lane_quads(int32_t width, int32_t feat) {
  if (feat < 4 || feat > kLdsMostFeat) return 0;
  if ((int64_t)width * slice_stride((feat + 3) / 4) * 16 > kSliceBytes) return 0;
  return (feat + 31) / 32;
}

// Entries that long rows must have together for slices to pay: up to 32 features nothing is won (the reduction over the lanes costs
// what LDS saves); the loads of the slices, and the last wave of workgroups, want half a gigabyte of gathered rows, and 2 GB where a
// lane has two float4 or rows are cut inside one.  Drawn graphs: 96 features, 1.4 M entries 32 -> 22 us; 64, 2.0 M 40 -> 46;
// 64, 10.8 M 221 -> 197; 32, 6.3 M 59 -> 76; 67, 3.0 M 69 -> 98.
constexpr int64_t slice_min_entries(int64_t feat) {
  if (feat <= 32) return INT64_MAX;
  return (feat <= 64 || feat % 4 ? (int64_t)1 << 29 : (int64_t)1 << 27) / feat;
}

// Do slices pay for n_long rows with that many entries together?  Where Yt comes close to fitting an XCD's 4 MB of L2 the lists
// gather it at 17 to 20 TB/s, and slices, whose segments each ask for a row of X, are no faster; unless there are so few long rows
// that X stays near as well (40 dense matrices: within 512 KB 1.3 times as fast, 0.92 to 2.2; more 0.99, 0.35 to 2.2).
constexpr bool few_long_rows(int64_t feat, int64_t n_long) { return n_long * feat <= (int64_t)1 << 17; }
constexpr bool slices_pay(int64_t n_cols, int64_t feat, int64_t n_long, int64_t long_nnz) {
  if (long_nnz < slice_min_entries(feat)) return false;
  return few_long_rows(feat, n_long) || n_cols * feat >= (int64_t)7 << 18;  // (floats: 7 MB of Yt)
}

// And once the segments have been counted?  `units` are the pairs of a slice and a part of the rows that have any.  Below 10 MB of Yt
// a plan without slices keeps CSR order, which finds columns that many entries name in the caches too: where half of the segments lie
// in less than 42 % of the slices, slices pay from 10 MB on.  Where columns are even and a lane's last float4 is partly used, short
// segments pay from 12 MB on.  Never fewer units than leave two CUs in five idle.  500 graphs of 7 to 15 MB, 48 to 256 features,
// columns uniform, skewed, hot in a range, in communities and in a band, slices against lists: uneven ones up to 10 MB 0.90 times as
// fast (0.44 to 1.8), beyond 1.67 (1.1 to 5.4); even ones 1.22 (0.6 to 2.5), short segments up to 12 MB 0.92 (0.5 to 1.2).
constexpr bool slices_pay_as_counted(int64_t n_cols, int64_t feat, int64_t n_long, int64_t long_nnz, int64_t units, int64_t n_segs,
                                     int32_t n_slices, int32_t half_in) {
  if (!slices_pay(n_cols, feat, n_long, long_nnz)) return false;
  if (few_long_rows(feat, n_long)) return true;
  const bool uneven = 50 * (int64_t)half_in < 21 * (int64_t)n_slices, is_short = feat % 32 != 0 && 10 * long_nnz < 47 * n_segs;
  return units >= 160 && n_cols * feat >= (int64_t)(uneven ? 10 : is_short ? 12 : 7) << 18;
}

// The fewest slices that have half of the segments.  begin: see slice_units().
inline int32_t slices_of_half(const std::vector<int32_t>& begin, int32_t n_slices, int64_t parts) {
  std::vector<int64_t> segs((size_t)n_slices, 0);
  for (int64_t part = 0; part < parts; ++part)
    for (int32_t s = 0; s < n_slices; ++s) segs[(size_t)s] += begin[(size_t)(part * n_slices + s + 1)] - begin[(size_t)(part * n_slices + s)];
  std::sort(segs.begin(), segs.end(), [](int64_t x, int64_t y) { return x > y; });
  int64_t sum = 0;
  int32_t n = 0;
  while (n < n_slices && 2 * sum < begin.back() - begin.front()) sum += segs[(size_t)n++];
  return n;
}

// Is a row that begins and ends there long?  One that is not inside the entries is none: nothing is read for it here, and the
// general path treats it as it treats every other row.
constexpr bool is_long_row(int64_t begin, int64_t end, int64_t nnz, int64_t min_deg) {
  return begin >= 0 && end <= nnz && end - begin >= min_deg;
}

// A workgroup's work: segments begin .. end - 1, all of one slice.
struct SliceUnit {
  int32_t slice, begin, end, reserved;
};

// Units in the order of their workgroup ids, which go round the 8 XCDs.  begin[part * n_slices + slice]: the first segment of that
// part of the rows in that slice, one after the other, and the end of the last.  Each XCD has a range of slices of its own: what they
// share of a line of values and results (neighbouring pieces of a row) then meets in one L2.  What has more than `most` segments, a
// range of columns that many entries are in, is cut and dealt to the XCDs that have least.
inline std::vector<SliceUnit> slice_units(const std::vector<int32_t>& begin, int32_t n_slices, int64_t parts, int64_t most) {
  constexpr int kXcds = 8;
  const int32_t per_xcd = (n_slices + kXcds - 1) / kXcds;
  std::vector<SliceUnit> units, of_xcd[kXcds];
  int64_t load[kXcds] = {0};
  for (int64_t part = 0; part < parts; ++part) {
    const int32_t* at = begin.data() + part * n_slices;
    for (int32_t s = 0; s < n_slices; ++s)
      if (at[s + 1] - at[s] <= most) {
        of_xcd[s / per_xcd].push_back({s, at[s], at[s + 1], 0});
        load[s / per_xcd] += at[s + 1] - at[s];
      }
    for (int32_t s = 0; s < n_slices; ++s) {
      const int64_t n = at[s + 1] - at[s], pieces = (n + most - 1) / most;
      for (int64_t i = 0; n > most && i < pieces; ++i) {
        const int x = (int)(std::min_element(load, load + kXcds) - load);
        const int32_t lo = (int32_t)(n * i / pieces), hi = (int32_t)(n * (i + 1) / pieces);
        of_xcd[x].push_back({s, at[s] + lo, at[s] + hi, 0});
        load[x] += hi - lo;
      }
    }
    size_t longest = 0;
    for (const auto& list : of_xcd) longest = std::max(longest, list.size());
    for (size_t i = 0; i < longest; ++i)
      for (const auto& list : of_xcd) units.push_back(i < list.size() ? list[i] : SliceUnit{0, 0, 0, 0});
    for (auto& list : of_xcd) list.clear();
  }
  return units;
}

}  // namespace sptir

#endif  // SPTIR_SDDMM_SLICE_SHAPE_H_
