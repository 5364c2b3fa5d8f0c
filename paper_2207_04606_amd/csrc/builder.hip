// CSR -> hyb(c,k) format decomposition on the GPU (bucketing rule of section
// 4.2.1 of arXiv 2207.04606; the index inference that section 3.2.1 leaves to
// host pre-processing is done here by histogram -> scan -> stable scatter).
//
// Work unit: one thread per (row r, column partition p) pair, a workgroup per
// 256 consecutive rows of one partition.  A pair's row piece is the run of the
// row's (ascending) columns that fall in [p*w, (p+1)*w); its length l selects
// bin i = ceil(log2 l) (ELL bucket of width 2^i) or, for i > k, the remainder.
// Rows must appear in a bucket in ascending order, so placement is a stable
// multi-split: per-workgroup bin counts, an exclusive scan over workgroups per
// (partition, bin), and an in-workgroup rank from ballots.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_sort.h"

namespace sptir {
namespace {

constexpr int kMaxBins = 32;  // k <= 30 -> bins 0..k plus the remainder bin k+1

struct BuildShape {
  int32_t n_rows, n_cols, c, k, w;
  int32_t nb;  // bins per partition = k + 2
  int32_t NB;  // row blocks = ceil(n_rows / 256)
};

// bound[(p - 1) * n_rows + r] = first position of row r whose column is >= p * w, for p = 1 .. c-1.  A workgroup
// takes kBoundRows rows x up to kBoundParts partitions with the partition index running fastest over the lanes, so
// that the searches of a wavefront probe the entries of a few rows only (they are in cache after the first
// probes), and writes its results through an LDS tile, so that consecutive lanes write consecutive rows.
constexpr int kBoundRows = 64, kBoundParts = 64;

__device__ __forceinline__ void piece_bounds_workgroup(const BuildShape& s, int32_t nnz, unsigned wg,
                                                       const int32_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ indices,
                                                       int32_t* __restrict__ bound) {
  __shared__ int32_t tile[kBoundParts][kBoundRows + 1];
  const int n_pc = (s.c - 1 + kBoundParts - 1) / kBoundParts;
  const int rb = (int)wg / n_pc, pc = (int)wg % n_pc;
  const int r0 = rb * kBoundRows, p0 = 1 + pc * kBoundParts;
  const int np = s.c - p0 < kBoundParts ? s.c - p0 : kBoundParts;
  const int nr = s.n_rows - r0 < kBoundRows ? s.n_rows - r0 : kBoundRows;
  for (int idx = threadIdx.x; idx < nr * np; idx += blockDim.x) {
    const int rl = idx / np, pl = idx - rl * np;
    // (this runs before the host has seen the verdict on indptr: whatever it holds, no read leaves `indices`)
    int a = indptr[r0 + rl], b = indptr[r0 + rl + 1];
    a = a < 0 ? 0 : (a > nnz ? nnz : a);
    b = b < a ? a : (b > nnz ? nnz : b);
    tile[pl][rl] = lower_bound_col(indices, a, b, (int64_t)(p0 + pl) * s.w);
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < nr * np; idx += blockDim.x) {
    const int pl = idx / nr, rl = idx - pl * nr;
    bound[(int64_t)(p0 + pl - 1) * s.n_rows + r0 + rl] = tile[pl][rl];
  }
}

// start and length of row r's piece in partition p
__device__ __forceinline__ void row_piece(const BuildShape& s, const int32_t* __restrict__ indptr,
                                          const int32_t* __restrict__ bound, int r, int p, int* lo, int* len) {
  const int first = (p == 0) ? indptr[r] : bound[(int64_t)(p - 1) * s.n_rows + r];
  const int last = (p == s.c - 1) ? indptr[r + 1] : bound[(int64_t)p * s.n_rows + r];
  *lo = first;
  *len = last - first;
}

// bin of a piece of length l >= 1: smallest i with l <= 2^i, capped at k+1 (remainder)
__device__ __forceinline__ int bin_of_length(int l, int k) {
  int i = (l <= 1) ? 0 : 32 - __clz(l - 1);
  return i > k ? k + 1 : i;
}

// ---------------------------------------------------------------- validation
// flags[0]: indptr is not a non-decreasing prefix from 0 to nnz
// flags[1]: a column id outside [0, n_cols)
// flags[2]: number of positions q >= 1 with indices[q] <= indices[q-1]
// flags[3]: number of non-empty rows whose first column does not exceed the
//           column stored just before it (descents that are legal)
// Columns ascend strictly inside every row iff flags[2] == flags[3].
// flags[4]: number of positions q >= 1 whose value differs (as a bit pattern) from the one stored before it
// flags[6]: entries of the longest row
// flags[7]: rows of min_deg entries and more (bits 32 ..), and their entries
// flags[5]: number of non-empty rows whose first value differs from the value stored just before it
// Every row has one value for all of its entries iff flags[4] == flags[5] (only counted when `values` is given).
// The counters exist kFlagSlots times, 64 bytes apart, and a wavefront adds to the copy its workgroup id picks:
// tens of thousands of atomic adds to one address would take longer than reading the matrix.  The host adds up.
constexpr int kFlagSlots = 64, kFlagStride = 8;
static_assert(kFlagSlots * kFlagStride == kValidationWords, "the words a caller provides");
__device__ __forceinline__ unsigned long long* flag_slot(unsigned long long* flags) {
  return flags + (blockIdx.x & (kFlagSlots - 1)) * kFlagStride;
}
__device__ __forceinline__ void validate_rows(int n_wg, int wg, int32_t n_rows, int64_t nnz,
                                              const int32_t* __restrict__ indptr,
                                              const int32_t* __restrict__ indices,
                                              const int32_t* __restrict__ values, int32_t min_deg, unsigned long long* flags) {
  const int64_t stride = (int64_t)n_wg * blockDim.x;
  unsigned long long of_long = 0;
  unsigned int legal_descents = 0, legal_changes = 0, longest = 0;
  bool bad = false;
  for (int64_t r = (int64_t)wg * blockDim.x + threadIdx.x; r < n_rows; r += stride) {
    int64_t a = indptr[r], b = indptr[r + 1];
    const bool bad_here = (a < 0) || (b > nnz) || (a > b) || (r == 0 && a != 0) || (r == n_rows - 1 && b != nnz);
    bad |= bad_here;
    if (!bad_here) longest = max(longest, (unsigned int)(b - a));
    if (!bad_here && b - a >= min_deg) of_long += (1ull << 32) + (unsigned long long)(b - a);
    legal_descents += !bad_here && a < b && a > 0 && indices[a] <= indices[a - 1];
    if (values) legal_changes += !bad_here && a < b && a > 0 && values[a] != values[a - 1];
  }
  // a grid-wide count through one address: one atomic per wavefront, a few thousand in all
  for (int d = 32; d > 0; d >>= 1) {
    legal_descents += __shfl_down(legal_descents, d, 64);
    legal_changes += __shfl_down(legal_changes, d, 64);
    longest = max(longest, (unsigned int)__shfl_down((int)longest, d, 64));
    of_long += __shfl_down(of_long, d, 64);
  }
  const unsigned long long any_bad = __ballot(bad);
  flags = flag_slot(flags);
  if ((threadIdx.x & 63) == 0) {
    if (legal_changes) atomicAdd(&flags[5], (unsigned long long)legal_changes);
    if (legal_descents) atomicAdd(&flags[3], (unsigned long long)legal_descents);
    if (any_bad) flags[0] = 1;
    if (longest) atomicMax(&flags[6], (unsigned long long)longest);
    if (of_long) atomicAdd(&flags[7], of_long);
  }
}

// One thread checks 8 consecutive positions per step (two 16-byte loads per array when `vec` says that the arrays
// are 16-byte aligned, 4-byte loads otherwise; all loads of a step are issued before any is used); position q is
// compared with position q - 1, which the lane below holds (the first lane of a wavefront loads it).
__device__ __forceinline__ int4 load4(const int32_t* __restrict__ p, int vec) {
  if (vec) return *reinterpret_cast<const int4*>(p);
  return make_int4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ int ascents_not(int prev, const int4& a, const int4& b, bool has_prev) {
  return (has_prev && a.x <= prev) + (a.y <= a.x) + (a.z <= a.y) + (a.w <= a.z) + (b.x <= a.w) + (b.y <= b.x) +
         (b.z <= b.y) + (b.w <= b.z);
}
__device__ __forceinline__ int changes_of(int prev, const int4& a, const int4& b, bool has_prev) {
  return (has_prev && a.x != prev) + (a.y != a.x) + (a.z != a.y) + (a.w != a.z) + (b.x != a.w) + (b.y != b.x) +
         (b.z != b.y) + (b.w != b.z);
}

__device__ __forceinline__ void validate_elems(int n_wg, int wg, int64_t nnz, int32_t n_cols, int vec,
                                               const int32_t* __restrict__ indices,
                                               const int32_t* __restrict__ values, unsigned long long* flags) {
  constexpr int kPer = 8;
  const int64_t stride = (int64_t)n_wg * blockDim.x * kPer;
  const int lane = threadIdx.x & 63;
  const bool with_values = values != nullptr;
  unsigned int descents = 0, changes = 0;
  bool range = false;
  int64_t q = ((int64_t)wg * blockDim.x + threadIdx.x) * kPer;
  for (; q + kPer <= nnz; q += stride) {  // whole groups
    const int64_t q_prev = q > 0 ? q - 1 : 0;
    const int4 c0 = load4(indices + q, vec), c1 = load4(indices + q + 4, vec);
    int4 v0 = make_int4(0, 0, 0, 0), v1 = v0;
    if (with_values) { v0 = load4(values + q, vec); v1 = load4(values + q + 4, vec); }
    int first_c = 0, first_v = 0;
    if (lane == 0) {
      first_c = indices[q_prev];
      if (with_values) first_v = values[q_prev];
    }
    int prev_c = __shfl_up(c1.w, 1, 64), prev_v = __shfl_up(v1.w, 1, 64);
    if (lane == 0) { prev_c = first_c; prev_v = first_v; }
    const unsigned n = (unsigned)n_cols;
    range |= ((unsigned)c0.x >= n) | ((unsigned)c0.y >= n) | ((unsigned)c0.z >= n) | ((unsigned)c0.w >= n) |
             ((unsigned)c1.x >= n) | ((unsigned)c1.y >= n) | ((unsigned)c1.z >= n) | ((unsigned)c1.w >= n);
    descents += ascents_not(prev_c, c0, c1, q > 0);
    if (with_values) changes += changes_of(prev_v, v0, v1, q > 0);
  }
  for (int i = 0; i < kPer && q + i < nnz; ++i) {  // the thread that holds the last, partial group
    const int32_t col = indices[q + i];
    range |= (unsigned)col >= (unsigned)n_cols;
    descents += (q + i > 0) && col <= indices[q + i > 0 ? q + i - 1 : 0];
    if (with_values) changes += (q + i > 0) && values[q + i] != values[q + i > 0 ? q + i - 1 : 0];
  }
  // a grid-wide count through one address: one atomic per wavefront, a few thousand in all
  for (int d = 32; d > 0; d >>= 1) {
    descents += __shfl_down(descents, d, 64);
    changes += __shfl_down(changes, d, 64);
  }
  unsigned long long any_range = __ballot(range);
  flags = flag_slot(flags);
  if ((threadIdx.x & 63) == 0) {
    if (changes) atomicAdd(&flags[4], (unsigned long long)changes);
    if (descents) atomicAdd(&flags[2], (unsigned long long)descents);
    if (any_range) flags[1] = 1;
  }
}

// Both checks in one launch: the first row_wgs workgroups take the rows, the others the entries.
__global__ __launch_bounds__(256) void k_validate(int row_wgs, int32_t n_rows, int64_t nnz, int32_t n_cols, int vec,
                                                  const int32_t* __restrict__ indptr,
                                                  const int32_t* __restrict__ indices,
                                                  const int32_t* __restrict__ values, int32_t min_deg,
                                                  unsigned long long* flags) {
  const int wg = (int)blockIdx.x;
  if (wg < row_wgs) validate_rows(row_wgs, wg, n_rows, nnz, indptr, indices, values, min_deg, flags);
  else validate_elems((int)gridDim.x - row_wgs, wg - row_wgs, nnz, n_cols, vec, indices, values, flags);
}

// Both, and next to them the piece boundaries, which wait for nothing either: the first n_bound workgroups
__global__ __launch_bounds__(256) void k_first_pass(unsigned n_bound, int row_wgs, BuildShape s, int64_t nnz, int vec,
                                                    const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                    const int32_t* __restrict__ values, int32_t min_deg,
                                                    unsigned long long* flags, int32_t* __restrict__ bound) {
  if (blockIdx.x < n_bound) {
    piece_bounds_workgroup(s, (int32_t)nnz, blockIdx.x, indptr, indices, bound);
    return;
  }
  const int wg = (int)(blockIdx.x - n_bound);
  if (wg < row_wgs) validate_rows(row_wgs, wg, s.n_rows, nnz, indptr, indices, values, min_deg, flags);
  else validate_elems((int)(gridDim.x - n_bound) - row_wgs, wg - row_wgs, nnz, s.n_cols, vec, indices, values, flags);
}

// row_val[r] = the value of row r's first entry (0 for an empty row)
__global__ void k_row_values(int32_t n_rows, const int32_t* __restrict__ indptr, const float* __restrict__ values,
                             float* row_val) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_rows) row_val[r] = indptr[r + 1] > indptr[r] ? values[indptr[r]] : 0.f;
}

// --------------------------------------------------------------------- count
// counts   [c][nb][NB] int32 : pieces of each bin per row block
// rem_nnz  [c][NB]     int64 : non-zeros sent to the remainder per row block
__global__ __launch_bounds__(kBuildBlock) void k_count(BuildShape s, const int32_t* __restrict__ indptr,
                                                       const int32_t* __restrict__ bound, int32_t* counts,
                                                       int64_t* rem_nnz) {
  __shared__ int hist[kMaxBins];
  __shared__ unsigned long long sum_nnz;
  int tid = threadIdx.x;
  int p = blockIdx.x / s.NB, rb = blockIdx.x % s.NB;
  if (tid < kMaxBins) hist[tid] = 0;
  if (tid == 0) sum_nnz = 0;
  __syncthreads();
  int r = rb * kBuildBlock + tid;
  if (r < s.n_rows) {
    int lo, l;
    row_piece(s, indptr, bound, r, p, &lo, &l);
    if (l > 0) {
      int bin = bin_of_length(l, s.k);
      atomicAdd(&hist[bin], 1);
      if (bin == s.k + 1) atomicAdd(&sum_nnz, (unsigned long long)l);
    }
  }
  __syncthreads();
  if (tid < s.nb) counts[((int64_t)p * s.nb + tid) * s.NB + rb] = hist[tid];
  if (tid == 0) rem_nnz[(int64_t)p * s.NB + rb] = (int64_t)sum_nnz;
}

// The counts become positions, a workgroup per sequence; their totals and (the last workgroup) the verdict's words go to
// the host's memory, where it reads them once the stream has drained.
struct FirstReport {
  unsigned long long* flags;  // [kValidationWords]
  int64_t* rem_nnz;           // [c]
  int32_t* bins;              // [c][nb]
};
__global__ __launch_bounds__(kBuildBlock) void k_first_totals(BuildShape s, int32_t* counts, int64_t* rem_nnz,
                                                              const unsigned long long* __restrict__ flags,
                                                              FirstReport report) {
  __shared__ int bin_sums[kWaves];
  __shared__ long long nnz_sums[kWaves];
  const int n_bins = s.c * s.nb, seq = (int)blockIdx.x;
  if (seq < n_bins) {
    const int total = scan_sequence(counts + (int64_t)seq * s.NB, s.NB, bin_sums);
    if (threadIdx.x == 0) report.bins[seq] = total;
  } else if (seq < n_bins + s.c) {
    const long long total = scan_sequence((long long*)rem_nnz + (int64_t)(seq - n_bins) * s.NB, s.NB, nnz_sums);
    if (threadIdx.x == 0) report.rem_nnz[seq - n_bins] = total;
  } else {
    for (int i = threadIdx.x; i < kValidationWords; i += kBuildBlock) report.flags[i] = flags[i];
  }
}

// --------------------------------------------------------------------- place
struct PlaceArgs {
  const int32_t* indptr;
  const int32_t* bound;        // piece boundaries (k_piece_bounds)
  const int32_t* counts;       // scanned: rank of the block's first piece of each bin
  const int64_t* rem_nnz;      // scanned
  const int64_t* bucket_row_ptr;
  const int32_t* rem_part_ptr;
  const int64_t* rem_nnz_base;   // [c] first remainder nnz of each partition
  int32_t* row_ids;
  int64_t* rem_ptr;
  int32_t* row_len;  // [R+M] real (unpadded) length of every ELL row and remainder piece
  int32_t* piece_of; // [c][n_rows] position in row_ids of the piece of (row, partition), -1 where the piece is empty
  int64_t R, M, T;
  int32_t min_deg;   // rows of so many entries are long: their pieces are in no list (negative row_len)
};

// Every piece finds its position in row_ids; the entries follow in k_copy, once the lists of the SpMM are known.
__global__ __launch_bounds__(kBuildBlock) void k_place(BuildShape s, PlaceArgs a) {
  __shared__ int wave_cnt[kWaves][kMaxBins];
  __shared__ long long wave_sums[kWaves];
  int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int p = blockIdx.x / s.NB, rb = blockIdx.x % s.NB;
  if (tid < kWaves * kMaxBins) (&wave_cnt[0][0])[tid] = 0;
  if (blockIdx.x == 0 && tid == 0) a.rem_ptr[a.M] = a.T;
  if (blockIdx.x == 0 && tid < kChunkSlots) a.row_ids[a.R + a.M + tid] = 0;  // the spare entries past the end
  __syncthreads();

  int r = rb * kBuildBlock + tid;
  int lo = 0, l = 0, bin = -1;
  if (r < s.n_rows) {
    row_piece(s, a.indptr, a.bound, r, p, &lo, &l);
    if (l > 0) bin = bin_of_length(l, s.k);
  }
  // rank among the lanes of this wave that hold the same bin (stable: lower lanes first)
  int code = bin < 0 ? 63 : bin;
  unsigned long long peers = ~0ull;
#pragma unroll
  for (int bit = 0; bit < 6; ++bit) {
    bool mine = (code >> bit) & 1;
    unsigned long long b = __ballot(mine);
    peers &= mine ? b : ~b;
  }
  int rank_in_wave = __popcll(peers & ((1ull << lane) - 1ull));
  if (bin >= 0 && rank_in_wave == 0) wave_cnt[wave][bin] = __popcll(peers);

  // remainder pieces also need the running sum of their lengths
  bool is_rem = (bin == s.k + 1);
  long long my_nnz = is_rem ? l : 0;
  long long tot;
  long long nnz_before = block_exclusive_scan<long long>(my_nnz, wave_sums, &tot);
  // (block_exclusive_scan synchronises the workgroup, so wave_cnt is complete here)
  if (r >= s.n_rows) return;
  int32_t where = -1;  // position of this piece in row_ids
  if (bin >= 0) {
    int before = 0;
    for (int wv = 0; wv < wave; ++wv) before += wave_cnt[wv][bin];
    int64_t q = (int64_t)a.counts[((int64_t)p * s.nb + bin) * s.NB + rb] + before + rank_in_wave;
    if (!is_rem) {
      where = (int32_t)(a.bucket_row_ptr[(int64_t)p * (s.k + 1) + bin] + q);
    } else {
      int64_t m = (int64_t)a.rem_part_ptr[p] + q;
      where = (int32_t)(a.R + m);
      a.rem_ptr[m] = a.rem_nnz_base[p] + a.rem_nnz[(int64_t)p * s.NB + rb] + nnz_before;
    }
    a.row_ids[where] = r;
    a.row_len[where] = a.indptr[r + 1] - a.indptr[r] >= a.min_deg ? -l : l;
  }
  a.piece_of[(int64_t)p * s.n_rows + r] = where;
}

// ------------------------------------------------------- SpMM work-item list
// The SpMM kernel keeps the Y rows of one row block (row_block consecutive
// rows) in LDS and walks the real entries of the block's row pieces in chunks
// of kChunkSlots; a chunk never crosses a row-block boundary.  Rows ascend
// inside every bucket and inside every partition's remainder, hence the rows
// of a bin that fall into row block j are one contiguous run of row_ids; a
// "cell" holds the chunks that one (phase, row block, partition) contributes
// from one bin, or from its queues.  The cells of a (phase, row block) group
// are numbered partition by partition (see cells_per_group below) and their
// chunks are laid out in that order, so the chunks of a group are contiguous
// and sweep the column partitions in ascending order.
struct CellShape {
  int32_t c, k, nb;
  int32_t log2_rb, n_rb, ppg, n_phases;
  int32_t long_len;  // pieces with more real entries are not in the lists (heavy pieces)
  int32_t wide_margin;  // see below
  bool cut_queues = false;  // see there too
  int64_t R;
};

// bin_rb_ptr[(p*nb + bin)*(n_rb+1) + j] = first position in row_ids of bin
// (p, bin) whose row id is >= j * row_block (absolute index into row_ids)
__device__ __forceinline__ void cell_bounds_workgroup(const CellShape& cs, unsigned wg, const int64_t* __restrict__ bucket_row_ptr,
                                                      const int32_t* __restrict__ rem_part_ptr,
                                                      const int32_t* __restrict__ row_ids, int32_t* bin_rb_ptr) {
  int64_t t = (int64_t)wg * blockDim.x + threadIdx.x;
  int64_t per_bin = (int64_t)cs.n_rb + 1;
  if (t >= (int64_t)cs.c * cs.nb * per_bin) return;
  int j = (int)(t % per_bin);
  int pb = (int)(t / per_bin);
  int p = pb / cs.nb, bin = pb % cs.nb;
  int64_t lo, hi;
  if (bin <= cs.k) {
    int64_t b = (int64_t)p * (cs.k + 1) + bin;
    lo = bucket_row_ptr[b]; hi = bucket_row_ptr[b + 1];
  } else {
    lo = cs.R + rem_part_ptr[p]; hi = cs.R + rem_part_ptr[p + 1];
  }
  int64_t bound = (int64_t)j << cs.log2_rb;
  while (lo < hi) {
    int64_t mid = lo + ((hi - lo) >> 1);
    if ((int64_t)row_ids[mid] < bound) lo = mid + 1; else hi = mid;
  }
  bin_rb_ptr[t] = (int32_t)lo;
}

// Cells of one (phase, row block) group, in chunk order: for every partition of the phase its nb bin cells
// (the chunks of that bin's rows that are cut wide) and one queue cell, then one pad cell that rounds the
// group's chunk count up to a multiple of kChunksPerQuad (the SpMM kernel fetches chunks four at a time).
//
// How the row pieces of a (group, partition) become chunks (pieces of at most long_len entries; bucket
// rows and remainder pieces alike, each with its real entries only):
//  * a piece is dealt whole to one of eight queues, one per lane group of the SpMM kernel, where its entries
//    follow those of the piece before it without a gap; chunk t of the queue cell holds entries 8t .. 8t+7 of
//    every queue, and the last entry of a piece carries a flag.  A lane group then walks whole rows alone,
//    keeps the running sum in registers, hands it over at a flag and needs no cross-lane reduction; no pad of
//    a bucket row is ever walked.  A piece goes to the queue that is shortest so far (buckets are visited
//    widest first, so this is the longest-first rule up to a factor of two);
//  * unless that would leave the queues uneven: a piece that is longer than a chunk and than an even share of what is
//    still to be dealt, or a shorter one that would reach wide_margin entries beyond the level at which all queues
//    would end, is cut "wide" instead, into chunks of 64 entries that all eight lane groups share, in its bin's cell.
//    (A piece of 60 entries among rows of four makes its queue, and with it the list, 60 entries long: 14,964 rows,
//    156,998 entries in 16 partitions 59 -> 33 us.  Two chunks of margin, as the wide chunk costs one; in rounds, whose
//    lists are long enough to be even, four.)
// Where that takes a chunk more than the entries need, the queues may be cut instead (cut_queues): the pieces follow each other
// through all eight queues, each as long as the entries need, and a piece that does not fit the end of a queue has its first entries
// at the start of the next, flagged at both ends.  A dozen or two of long rows do not divide by eight: rows of 37 +- 12 entries in
// blocks of 32 walk 9 % more slots than there are entries when dealt whole, 3 % when cut (132,534 rows of 37 in each of eight
// partitions, 128 features: 1048 -> 997 us; cut only where two chunks are saved 0.96 times as fast as that, where four 0.94).
// The first entries and not the last: so all queues begin at the first columns of the partition and sweep X together at first, as they
// do where rows are dealt whole.  With queues that began in the middle of a row, 34 drawn graphs whose rows of X are no whole lines (100 and 200
// features, a partition's X beyond L2) took 1.02 times as long (up to 1.06) as with rows dealt whole, now 0.98 (up to 1.01).
// The rows of one partition are distinct, and a piece that is cut is a chunk shorter than a queue, so that its ends lie in
// different chunks: two queues never hand over the same row of Y in one instruction.
__device__ __forceinline__ int cells_per_part(const CellShape& cs) { return cs.nb + 1; }
__device__ __forceinline__ int cells_per_group(const CellShape& cs) { return cs.ppg * (cs.nb + 1) + 1; }

__device__ __forceinline__ int chunks_of_length(int len) { return (len + kChunkSlots - 1) / kChunkSlots; }
inline int64_t chunks_of_slots(int64_t slots) { return (slots + kChunkSlots - 1) / kChunkSlots; }

// What becomes of a piece of at most long_len entries, one word per piece (in the order of row_ids):
//   queued    its first entry's position in the queue (bits 0..27; 0..26 where queues may be cut) and the queue (28..30)
//   cut       bit 27: the position (bits 0..14), the chunks of the queue (15..26) and the queue: the last entries, to the end of the
//             queue; those before are at the start of the next
//   cut wide  bit 31 and the chunks of the pieces before it in its bin's cell
constexpr uint32_t kWidePiece = 0x80000000u, kCutPiece = 1u << 27;
constexpr int kCutPosBits = 15, kCutQueueMax = 1 << kCutPosBits;  // entries of a queue that may be cut: fewer than this

__device__ __forceinline__ unsigned min_of_8(unsigned v) {  // over the eight lanes of a lane group
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1 0 3 2
  v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2 3 0 1
  return min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
}

// Eight lanes per (group, partition of its phase), one per queue.  The lengths are fetched side by side into LDS first;
// what remains serial, a piece after the other to the shortest queue, runs on registers.  (A thread per partition that
// read a length at a time, once to count and once more to fill, took 35 + 93 us on 169,343 rows; this takes 15.)
// Writes the chunk counts of the partition's cells, a word per piece (see above) and the entries of every queue.
constexpr int kDealParts = 8;  // partitions per workgroup, a wavefront
template <bool MAY_CUT>
__global__ __launch_bounds__(8 * kDealParts) void k_deal(CellShape cs, int64_t n_parts, const int32_t* __restrict__ bin_rb_ptr,
                                              const int32_t* __restrict__ row_len, long long* __restrict__ cell_chunks,
                                              uint32_t* __restrict__ dealt, int32_t* __restrict__ queue_len) {
  extern __shared__ int piece_len[];                 // [kDealParts][rows of a row block]: lengths (then words), then positions
  __shared__ int before[kDealParts][kMaxBins + 1];   // pieces before a bin, widest bin first
  __shared__ int first[kDealParts][kMaxBins];        // first piece of a bin
  __shared__ int wide[kDealParts][kMaxBins];         // chunks cut wide so far
  const int l = threadIdx.x & 7, part = threadIdx.x >> 3;
  const int64_t t = (int64_t)blockIdx.x * kDealParts + part;
  const int64_t grp = t / cs.ppg;
  const int p_local = (int)(t % cs.ppg);
  const int rb = (int)(grp % cs.n_rb), phase = (int)(grp / cs.n_rb);
  const int p = phase * cs.ppg + p_local;
  const bool real = t < n_parts && p < cs.c;  // (the last phase may have fewer partitions)
  int* len_of = piece_len + (part << cs.log2_rb);
  int* piece_at = len_of + (kDealParts << cs.log2_rb);

  int count[kMaxBins / 8], mine = 0;
#pragma unroll
  for (int i = 0; i < kMaxBins / 8; ++i) {
    const int at = l * (kMaxBins / 8) + i, bin = cs.nb - 1 - at;
    count[i] = 0;
    if (real && bin >= 0) {
      const int32_t* ptr = bin_rb_ptr + ((int64_t)p * cs.nb + bin) * ((int64_t)cs.n_rb + 1) + rb;
      first[part][at] = ptr[0];
      count[i] = ptr[1] - ptr[0];
    }
    mine += count[i];
    wide[part][at] = 0;
  }
  int sum = mine;
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    const int o = __shfl_up(sum, d, 8);
    if (l >= d) sum += o;
  }
  int at0 = sum - mine;
#pragma unroll
  for (int i = 0; i < kMaxBins / 8; ++i) {
    before[part][l * (kMaxBins / 8) + i] = at0;
    at0 += count[i];
  }
  if (l == 7) before[part][kMaxBins] = at0;
  __syncthreads();
  const int n = before[part][kMaxBins];
  auto piece = [&](int i) {  // position in row_ids of the i-th piece to deal
    int b = 0;  // the last bin that starts at or before i
#pragma unroll
    for (int step = kMaxBins / 2; step > 0; step >>= 1)
      if (before[part][b + step] <= i) b += step;
    return first[part][b] + (i - before[part][b]);
  };
  unsigned to_deal = 0;  // entries not dealt yet (fewer than 2^31)
  unsigned most = 0;     // of the longest piece
  for (int i = l; i < n; i += 8) {
    const int q = piece(i), len = max(row_len[q], 0);  // (of a long row: nothing to deal)
    len_of[i] = len;
    piece_at[i] = q;
    if (len <= cs.long_len) { to_deal += (unsigned)len; most = max(most, (unsigned)len); }
  }
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    to_deal += (unsigned)__shfl_xor((int)to_deal, d, 8);
    most = max(most, (unsigned)__shfl_xor((int)most, d, 8));
  }
  const unsigned total = to_deal;
  __syncthreads();

  unsigned load = 0;  // entries of queue l
  unsigned queued = 0;  // entries of all queues
  int len = n > 0 ? len_of[0] : 0;
  for (int i = 0; i < n; ++i) {
    const int next = len_of[i + 1 < n ? i + 1 : i];
    if (len <= cs.long_len) {
      const unsigned share = (to_deal + 7) >> 3, level = (queued + to_deal) >> 3;
      to_deal -= (unsigned)len;
      const unsigned best = min_of_8(load * 8 + l);  // of equally short queues the first
      uint32_t word;
      if ((len > kChunkSlots ? (unsigned)len > share : (best >> 3) + (unsigned)len > level + (unsigned)cs.wide_margin) ||
          (MAY_CUT && (best >> 3) + (unsigned)len >= kCutPiece)) {
        const int at = cs.nb - 1 - bin_of_length(len, cs.k);
        const int w = wide[part][at];
        if (l == 0) wide[part][at] = w + chunks_of_length(len);
        word = kWidePiece | (uint32_t)w;
      } else {
        word = (best >> 3) | ((best & 7u) << 28);
        if ((best & 7u) == (unsigned)l) load += (unsigned)len;
        queued += (unsigned)len;
      }
      if (l == 0) len_of[i] = (int)word;
    }
    len = next;
  }
  unsigned longest = load;
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) longest = max(longest, (unsigned)__shfl_xor((int)longest, d, 8));
  __syncthreads();
  bool cut = false;
  if constexpr (MAY_CUT) {
    unsigned n_wide = 0;
#pragma unroll
    for (int i = 0; i < kMaxBins / 8; ++i) n_wide += (unsigned)wide[part][l * (kMaxBins / 8) + i];
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) n_wide += (unsigned)__shfl_xor((int)n_wide, d, 8);
    const unsigned per_queue = (total + kChunkSlots - 1) / kChunkSlots * 8;
    cut = per_queue / 8 < ((longest + 7) >> 3) + n_wide && most + 8 <= per_queue && per_queue < (unsigned)kCutQueueMax;
    if (cut) {
      unsigned done = 0;  // entries of the pieces before
      for (int i0 = 0; i0 < n; i0 += 8) {
        const int i = i0 + l, own = i < n ? max(row_len[piece_at[i]], 0) : 0;
        const unsigned here = own <= cs.long_len ? (unsigned)own : 0u;
        unsigned upto = here;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
          const unsigned o = (unsigned)__shfl_up((int)upto, d, 8);
          if (l >= d) upto += o;
        }
        const unsigned at = done + upto - here, queue = at / per_queue, pos = at - queue * per_queue;
        if (i < n)
          len_of[i] = (int)((queue << 28) | pos | (pos + here > per_queue ? kCutPiece | (per_queue / 8 << kCutPosBits) : 0u));
        done += (unsigned)__shfl((int)upto, 7, 8);
      }
      const unsigned start = l * per_queue;
      load = total <= start ? 0u : min(total - start, per_queue);
      longest = per_queue;
    }
  }
  for (int i = l; i < n; i += 8) dealt[piece_at[i]] = (uint32_t)len_of[i];  // (a heavy piece's word is not looked at)
  if (t < n_parts) {
    long long* cell = cell_chunks + grp * cells_per_group(cs) + (int64_t)p_local * cells_per_part(cs);
    for (int bin = l; bin < cs.nb; bin += 8) cell[bin] = cut ? 0 : wide[part][cs.nb - 1 - bin];
    if (l == 0) cell[cs.nb] = (longest + 7) >> 3;
    queue_len[t * 8 + l] = (int32_t)load;
  }
}

// One wavefront per (phase, row block) group: its cells' counts become their exclusive prefix inside the group (the pad
// cell's is then the number of chunks before the padding), group_total[grp] the group's chunks, a multiple of
// kChunksPerQuad.
__global__ __launch_bounds__(256) void k_group_scan(CellShape cs, int64_t n_groups, long long* cell_chunks,
                                                    long long* group_total) {
  const int64_t grp = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (grp >= n_groups) return;
  const int lane = threadIdx.x & 63;
  const int cpg = cells_per_group(cs);
  long long* c = cell_chunks + grp * cpg;
  long long carry = 0;
  for (int i0 = 0; i0 < cpg - 1; i0 += 64) {
    const int i = i0 + lane;
    const long long n = i < cpg - 1 ? c[i] : 0;
    const long long incl = wave_inclusive_scan(n, lane);
    if (i < cpg - 1) c[i] = carry + incl - n;
    carry += __shfl(incl, 63, 64);
  }
  if (lane == 0) {
    c[cpg - 1] = carry;
    group_total[grp] = (carry + kChunksPerQuad - 1) / kChunksPerQuad * kChunksPerQuad;
  }
}

// ------------------------------------------------------------ chunk stream
// What the SpMM kernel actually reads: the chunks as fixed records, in list
// order, so that the address of every record follows from its list position
// alone (no dependent descriptor load inside the gather loop).  Four
// consecutive chunks form a quad, fetched with one 16-byte load per lane and
// array.  The 12-byte form (3 KB per quad):
//   quad[  0..255]  column ids, chunk i at 64*i  (slots past the last real one repeat a real column)
//   quad[256..511]  values                        (slots past the last real one hold +0.0f)
//   quad[512..767]  per slot: row relative to the first row of the row block in bits 0..15,
//                   the chunk's log2w in bits 16..21, the hand-over flag in bit 22 (the chunk's, or in a
//                   queue chunk the slot's: the last entry of a row piece), bit 23: the slot belongs to no
//                   row (past the end of a queue); slots of a wide chunk past its last entry hold -1
// The compact form (2 KB per quad; the kernel's time goes with the bytes it has
// to pull from beyond L2, and every feature tile re-reads the stream) folds the
// row word into the column word, see kCompactColBits:
//   quad[  0..255]  column - first column of the launch | row << 20 | real << 27 | log2w code << 28 | hand-over << 31
//   quad[256..511]  values
struct StreamShape {
  int32_t* stream;
  int32_t unit;   // 1: no values array (every row of A has one value, kept aside)
  int32_t compact;
  int32_t log2_rb;
  int32_t phase_width;  // columns a launch covers
};

__device__ __forceinline__ void put_slot(const StreamShape& ss, int64_t chunk, int slot, int32_t col_word,
                                         int32_t val_bits, int32_t row_word) {
  constexpr int kQuadSlots = kChunkSlots * kChunksPerQuad;
  const int n_arrays = (ss.compact ? 2 : 3) - (ss.unit ? 1 : 0);  // [cols][vals unless unit][row words unless compact]
  int32_t* quad = ss.stream + (chunk / kChunksPerQuad) * (n_arrays * kQuadSlots);
  const int at = (int)(chunk % kChunksPerQuad) * kChunkSlots + slot;
  quad[at] = col_word;
  if (!ss.unit) quad[kQuadSlots + at] = val_bits;
  if (!ss.compact) quad[(n_arrays - 1) * kQuadSlots + at] = row_word;
}

// One wavefront per (group, partition), a lane per slot of a chunk: the slots past the end of each queue; the first
// partition of a group also writes the chunks that round the group up to whole quads, and rb_chunk_ptr.
__device__ __forceinline__ void list_ends_workgroup(const CellShape& cs, const StreamShape& ss, int64_t n_parts, unsigned wg,
                                                    const long long* __restrict__ cell_first_chunk,
                                                    const long long* __restrict__ group_first_chunk,
                                                    const int32_t* __restrict__ queue_len, int64_t* rb_chunk_ptr,
                                                    int64_t n_chunks_total) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)wg * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (t >= n_parts) return;
  const int64_t grp = t / cs.ppg;
  const int p_local = (int)(t % cs.ppg);
  const long long* cells = cell_first_chunk + grp * cells_per_group(cs);
  const int64_t group_first = group_first_chunk[grp];
  const long long* queue_cell = cells + (int64_t)p_local * cells_per_part(cs) + cs.nb;
  const int from = queue_len[t * 8 + (lane >> 3)];
  const int64_t chunk0 = group_first + queue_cell[0];
  const int n_chunks = (int)(queue_cell[1] - queue_cell[0]);
  int shortest = from;
#pragma unroll
  for (int d = 8; d < 64; d <<= 1) shortest = min(shortest, __shfl_xor(shortest, d, 64));
  for (int ck = shortest >> 3; ck < n_chunks; ++ck)  // zeros that belong to no row
    if (ck * 8 + (lane & 7) >= from)
      put_slot(ss, chunk0 + ck, lane, ss.compact ? (int32_t)(3u << 28) : 0, 0, (3 << 16) | (1 << 23));
  if (p_local != 0) return;
  for (int64_t ck = cells[cells_per_group(cs) - 1]; ck % kChunksPerQuad != 0; ++ck)  // contribute nothing
    put_slot(ss, group_first + ck, lane, ss.compact ? (int32_t)0xF0000000u : 0, 0, -1);
  if (lane == 0) rb_chunk_ptr[grp] = group_first;
  if (lane == 0 && grp == 0) rb_chunk_ptr[n_parts / cs.ppg] = n_chunks_total;
}

// ------------------------------------------------------------ heavy pieces
// A piece of more than heavy_len real entries is "heavy".  The entries of all heavy pieces form one sequence, in
// the order of row_ids (buckets in bucket order, then the remainder: partition-major), which is cut into 64-slot
// chunks.  When heavy_len >= kChunkSlots the pieces follow each other without a gap (a chunk then holds the end
// of at most one piece, which is what the kernel can hand over per chunk); shorter heavy pieces each start a
// chunk of their own.
__device__ __forceinline__ int heavy_footprint(int len, int heavy_len) {
  return heavy_len >= kChunkSlots ? len : chunks_of_length(len) * kChunkSlots;
}

// Heavy pieces are numbered, and given their slots, by an exclusive scan over all pieces: sums over kHeavySpan pieces,
// their scan (k_totals), then the numbers of the heavy pieces themselves (k_heavy_units).
constexpr int kHeavyPerThread = 4, kHeavySpan = kBuildBlock * kHeavyPerThread;
struct HeavySums {  // one of each per kHeavySpan pieces
  long long *units, *slots, *entries;
  unsigned long long* not_taken;  // [2], or NULL: pieces and slots that would be heavy if their rows were not long
};

__device__ __forceinline__ void heavy_sums_workgroup(int64_t n_pieces, unsigned wg, const int32_t* __restrict__ row_len,
                                                     int32_t heavy_len, const HeavySums& sums) {
  __shared__ long long wave_sums[kWaves];
  long long units = 0, slots = 0, entries = 0, long_units = 0, long_slots = 0;
#pragma unroll
  for (int i = 0; i < kHeavyPerThread; ++i) {
    const int64_t q = (int64_t)wg * kHeavySpan + i * kBuildBlock + threadIdx.x;
    const int len = q < n_pieces ? row_len[q] : 0;
    if (len > heavy_len) { ++units; slots += heavy_footprint(len, heavy_len); entries += len; }
    if (-len > heavy_len) { ++long_units; long_slots += heavy_footprint(-len, heavy_len); }
  }
  long long tot[3];
  if (sums.not_taken) {
    long long t;
    block_exclusive_scan(long_units, wave_sums, &t);
    if (t > 0) {  // (the same in all threads)
      long long t_slots;
      block_exclusive_scan(long_slots, wave_sums, &t_slots);
      if (threadIdx.x == 0) {
        atomicAdd(&sums.not_taken[0], (unsigned long long)t);
        atomicAdd(&sums.not_taken[1], (unsigned long long)t_slots);
      }
    }
  }
  block_exclusive_scan(units, wave_sums, &tot[0]);
  block_exclusive_scan(slots, wave_sums, &tot[1]);
  block_exclusive_scan(entries, wave_sums, &tot[2]);
  if (threadIdx.x == 0) {
    sums.units[wg] = tot[0]; sums.slots[wg] = tot[1]; sums.entries[wg] = tot[2];
  }
}

// The sums, and next to them the bounds of the cells: the first n_sums workgroups
__global__ __launch_bounds__(kBuildBlock) void k_sums_and_cells(unsigned n_sums, int64_t n_pieces,
                                                                const int32_t* __restrict__ row_len, int32_t heavy_len,
                                                                HeavySums sums, CellShape cs,
                                                                const int64_t* __restrict__ bucket_row_ptr,
                                                                const int32_t* __restrict__ rem_part_ptr,
                                                                const int32_t* __restrict__ row_ids, int32_t* bin_rb_ptr) {
  if (blockIdx.x < n_sums) heavy_sums_workgroup(n_pieces, blockIdx.x, row_len, heavy_len, sums);
  else cell_bounds_workgroup(cs, blockIdx.x - n_sums, bucket_row_ptr, rem_part_ptr, row_ids, bin_rb_ptr);
}

// Exclusive scan of data[0 .. n) in place by one workgroup of kOneBlock threads (a run of elements each); *total and
// *most receive the sum and the largest element.
constexpr int kOneBlock = 1024;
__device__ __forceinline__ void scan_by_one_block(long long* data, int64_t n, long long* total, long long* most) {
  __shared__ long long wave_sum[kOneBlock / 64], wave_most[kOneBlock / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t per = (n + kOneBlock - 1) / kOneBlock;
  const int64_t i0 = threadIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
  long long mine = 0, largest = 0;
  for (int64_t i = i0; i < i1; ++i) { mine += data[i]; largest = max(largest, data[i]); }
  const long long incl = wave_inclusive_scan(mine, lane);
  for (int d = 32; d > 0; d >>= 1) largest = max(largest, __shfl_xor(largest, d, 64));
  __syncthreads();  // (the arrays may still be read from a previous call)
  if (lane == 63) wave_sum[wave] = incl;
  if (lane == 0) wave_most[wave] = largest;
  __syncthreads();
  long long before = incl - mine, all = 0;
  largest = 0;
  for (int w = 0; w < kOneBlock / 64; ++w) {
    if (w < wave) before += wave_sum[w];
    all += wave_sum[w];
    largest = max(largest, wave_most[w]);
  }
  for (int64_t i = i0; i < i1; ++i) {
    const long long v = data[i];
    data[i] = before;
    before += v;
  }
  *total = all;
  *most = largest;
}

// The last step of the scans over groups and over heavy pieces (a workgroup per array), and what the host needs to know
// before it can size the stream, written to its memory: report[0] = chunks of all lists, [1] = chunks of the longest
// list, [2] = heavy pieces, [3] = slots of the heavy sequence, [4] = entries of heavy pieces, [5] and [6] = what not_taken holds.
constexpr int kReport2 = 7;
__global__ __launch_bounds__(kOneBlock) void k_totals(int64_t n_groups, long long* group_chunks, int64_t n_spans,
                                                      HeavySums sums, long long* report) {
  const int which = blockIdx.x;
  long long* data = which == 0 ? group_chunks : which == 1 ? sums.units : which == 2 ? sums.slots : sums.entries;
  long long total, most;
  scan_by_one_block(data, which == 0 ? n_groups : n_spans, &total, &most);
  if (threadIdx.x != 0) return;
  if (which == 0) {
    if (n_groups > 0) group_chunks[n_groups] = total;  // (the end of the last list)
    report[0] = total; report[1] = most;
    report[5] = sums.not_taken ? (long long)sums.not_taken[0] : 0;
    report[6] = sums.not_taken ? (long long)sums.not_taken[1] : 0;
  } else {
    report[which + 1] = total;
  }
}

// Heavy list w covers the chunks [w*L, (w+1)*L) of the heavy sequence.  A wavefront writes a partial-sum row at
// every piece end and one more where its list ends, so its first write goes to row (pieces that end before
// chunk w*L) + w.
// A heavy piece q learns its number and its first slot (unit[q] = number << 32 | slot; the words of other pieces are not
// written), and the lists that start in it (in it: their first slot is one of its own) where their first write goes.
__device__ __forceinline__ void heavy_units_workgroup(int64_t n_pieces, unsigned wg, const int32_t* __restrict__ row_len,
                                                      int32_t heavy_len, const HeavySums& sums, int32_t list_chunks,
                                                      unsigned long long* __restrict__ unit,
                                                      int32_t* __restrict__ hlist_first_slot) {
  __shared__ unsigned long long wave_sums[kWaves];
  const int64_t q0 = (int64_t)wg * kHeavySpan + threadIdx.x * kHeavyPerThread;
  int len[kHeavyPerThread];
  unsigned long long mine = 0;
#pragma unroll
  for (int i = 0; i < kHeavyPerThread; ++i) {
    len[i] = q0 + i < n_pieces ? row_len[q0 + i] : 0;
    if (len[i] > heavy_len) mine += (1ull << 32) + (unsigned)heavy_footprint(len[i], heavy_len);
  }
  unsigned long long tot;
  unsigned long long at = block_exclusive_scan(mine, wave_sums, &tot) + ((unsigned long long)sums.units[wg] << 32) +
                          (unsigned long long)sums.slots[wg];
  const int per_list = list_chunks * kChunkSlots;
#pragma unroll
  for (int i = 0; i < kHeavyPerThread; ++i) {
    if (len[i] <= heavy_len) continue;
    unit[q0 + i] = at;
    const unsigned start = (unsigned)at, u = (unsigned)(at >> 32), end = start + (unsigned)len[i];
    for (unsigned w = (start + per_list - 1) / per_list; (unsigned long long)w * per_list < end; ++w)
      hlist_first_slot[w] = (int32_t)(u + w);
    at += (1ull << 32) + (unsigned)heavy_footprint(len[i], heavy_len);
  }
}

// What remains of the order of the row blocks by list length where one digit tells the lengths apart (order.hip): its three steps
// go with launches that are there anyway.
struct SortPass {
  SortInput in;
  int32_t n_rb, tiles, n_launches;
  int32_t* hist;
  int32_t* order;
};

__global__ __launch_bounds__(kBuildBlock) void k_units_and_hist(unsigned n_units, int64_t n_pieces,
                                                                const int32_t* __restrict__ row_len, int32_t heavy_len,
                                                                HeavySums sums, int32_t list_chunks,
                                                                unsigned long long* __restrict__ unit,
                                                                int32_t* __restrict__ hlist_first_slot, SortPass sort) {
  if (blockIdx.x < n_units)
    heavy_units_workgroup(n_pieces, blockIdx.x, row_len, heavy_len, sums, list_chunks, unit, hlist_first_slot);
  else
    sort_hist_workgroup(sort.in, sort.n_rb, sort.tiles, 0, blockIdx.x - n_units, sort.hist);
}

// The partial-sum rows of heavy piece number u whose real entries are the slots [e0, e1) of the heavy sequence:
// rows u + w for every heavy list w that holds one of them (see k_heavy_units).
__device__ __forceinline__ void piece_slots(int list_chunks, int u, int e0, int e1, int* first, int* count) {
  const int per_list = list_chunks * kChunkSlots;
  const int w0 = e0 / per_list, w1 = (e1 - 1) / per_list;
  *first = u + w0;
  *count = w1 - w0 + 1;
}

// The partial-sum rows of every row, partition by partition, and the rows that have any: counts per kBuildBlock rows
// (slots << 32 | rows), their scan, then the lists.
struct RowSlotArgs {
  int32_t n_rows, c, list_chunks, heavy_len;
  const int32_t *indptr, *piece_of, *row_len;
  const unsigned long long* unit;
  unsigned long long* sums;  // one per kBuildBlock rows
  int32_t *row_slot_ptr, *row_slots, *heavy_rows;
};

template <typename F>
__device__ __forceinline__ void for_row_slots(const RowSlotArgs& a, int r, F&& f) {
  if (r >= a.n_rows || a.indptr[r + 1] - a.indptr[r] <= a.heavy_len) return;
  for (int p = 0; p < a.c; ++p) {
    const int32_t q = a.piece_of[(int64_t)p * a.n_rows + r];
    if (q < 0) continue;
    const int len = a.row_len[q];
    if (len <= a.heavy_len) continue;
    const unsigned long long unit = a.unit[q];
    int first, count;
    piece_slots(a.list_chunks, (int)(unit >> 32), (int)(unsigned)unit, (int)(unsigned)unit + len, &first, &count);
    f(first, count);
  }
}

// The counts; the workgroups past n_sums scan the histograms of the sort
__global__ __launch_bounds__(kBuildBlock) void k_row_slot_sums(unsigned n_sums, RowSlotArgs a, SortPass sort) {
  __shared__ unsigned long long wave_sums[kWaves];
  __shared__ int32_t hist_sums[kWaves];
  if (blockIdx.x >= n_sums) {
    const int32_t len = kDigits * sort.tiles;
    (void)scan_sequence(sort.hist + (int64_t)(blockIdx.x - n_sums) * len, len, hist_sums);
    return;
  }
  unsigned long long n = 0, tot;
  for_row_slots(a, blockIdx.x * kBuildBlock + threadIdx.x, [&](int, int count) { n += count; });
  block_exclusive_scan((n << 32) + (n > 0), wave_sums, &tot);
  if (threadIdx.x == 0) a.sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kOneBlock) void k_row_slot_scan(unsigned long long* sums, int64_t n, int32_t* report) {
  long long total, unused;
  scan_by_one_block((long long*)sums, n, &total, &unused);
  if (threadIdx.x == 0) { report[0] = (int32_t)(total >> 32); report[1] = (int32_t)(uint32_t)total; }
}

__device__ __forceinline__ void row_slot_fill_workgroup(const RowSlotArgs& a, unsigned wg) {
  __shared__ unsigned long long wave_sums[kWaves];
  const int r = wg * kBuildBlock + threadIdx.x;
  unsigned long long n = 0, tot;
  for_row_slots(a, r, [&](int, int count) { n += count; });
  const unsigned long long at = a.sums[wg] + block_exclusive_scan((n << 32) + (n > 0), wave_sums, &tot);
  if (r >= a.n_rows) return;
  a.row_slot_ptr[r] = (int32_t)(at >> 32);
  if (r == a.n_rows - 1) a.row_slot_ptr[a.n_rows] = (int32_t)((at >> 32) + n);
  if (n == 0) return;
  a.heavy_rows[(uint32_t)at] = r;
  int32_t* out = a.row_slots + (at >> 32);
  for_row_slots(a, r, [&](int first, int count) {
    for (int i = 0; i < count; ++i) *out++ = first + i;
  });
}

// ---------------------------------------------------------------------- copy
// Every entry of A goes to its slot of the canonical arrays and of the stream in one pass over the CSR input.  A
// workgroup takes `per_wg` consecutive entries, whatever rows they belong to, so that the longest row costs no more than
// its share; it walks them by blocks of 2^log2_rows rows.  What is the same for all entries of a piece (where it goes) is
// put into LDS first, then a lane per entry finds its row by a search over the rows' starts and its partition from its
// column.  169,343 rows, 1.17 M entries in four partitions: 29 us with what goes along, most of it the chain of loads up to the pieces
// (three kernels with a wavefront per 64 pieces took 78 us, most of it in a few wavefronts with long pieces).
struct CopyArgs {
  const int32_t *indptr, *indices;
  const float* values;
  const int32_t *bound, *piece_of;
  const int64_t *bucket_row_ptr, *bucket_slot_ptr, *rem_ptr;
  int32_t* cols;
  float* vals;
  int64_t R, S, T;
  int64_t nnz;
  double inv_w;
  int32_t log2_rows, per_wg;
  // the stream (stream.stream NULL: canonical arrays only)
  const uint32_t* dealt;
  const unsigned long long* unit;
  const long long *cell_first_chunk, *group_first_chunk;
  int64_t heavy_chunk0, heavy_slots, n_heavy_chunks;
  int32_t min_deg;  // rows of so many entries are not in the stream
};
constexpr int kCopyPieces = 1024;  // most pieces a workgroup holds at a time
constexpr int kCopyWords = 6;      // LDS words per piece
constexpr int kCopyLog2Rows = 7;   // at most 128 rows a block

// What goes with the copy, in workgroups after its own: the ends of the lists, the partial-sum rows, the order of the row blocks.  (They take a
// third of the time that one of the copy's does, so they fill what those leave.  169,343 rows, 1.17 M entries: before them 33 us, after them 29, with the
// entries asked for before it is known where they go and no pieces looked up that have none of a workgroup's entries.)
struct CopyCompany {
  unsigned n_ends, n_slots, n_sort;  // workgroups of each
  unsigned n_copy;                   // the copy's
  int64_t n_parts;
  const int32_t* queue_len;
  int64_t* rb_chunk_ptr;
  int64_t n_chunks;
  RowSlotArgs slots;
  SortPass sort;
};

// (MAY_CUT costs a build of 169,343 rows and 1.17 M entries 1 of 217 us where no queue is cut)
template <bool MAY_CUT>
__global__ __launch_bounds__(256) void k_copy(BuildShape s, CellShape cs, StreamShape ss, CopyArgs a, int pieces_at_a_time,
                                              CopyCompany with) {
  extern __shared__ int lds[];
  if (blockIdx.x >= with.n_copy) {
    unsigned wg = blockIdx.x - with.n_copy;
    if (wg < with.n_slots) return row_slot_fill_workgroup(with.slots, wg);
    wg -= with.n_slots;
    if (wg < with.n_ends)
      return list_ends_workgroup(cs, ss, with.n_parts, wg, a.cell_first_chunk, a.group_first_chunk, with.queue_len,
                                 with.rb_chunk_ptr, with.n_chunks);
    wg -= with.n_ends;
    if (wg < with.n_sort)
      sort_scatter_workgroup(with.sort.in, with.sort.n_rb, with.sort.tiles, 0, wg, with.sort.hist, nullptr, with.sort.order);
    return;
  }
  const unsigned copy_wg = blockIdx.x, n_copy = with.n_copy;
  __shared__ int row_lo[(1 << kCopyLog2Rows) + 1];
  const int log2_rows = a.log2_rows, n_rows_here = 1 << log2_rows;
  int* piece_lo = lds;                                                 // first entry in the input
  int* piece_len = piece_lo + pieces_at_a_time;
  uint32_t* piece_dst = (uint32_t*)(piece_len + pieces_at_a_time);     // first slot in the canonical arrays
  uint32_t* piece_word = piece_dst + pieces_at_a_time;                 // see k_deal
  int* piece_chunk = (int*)(piece_word + pieces_at_a_time);            // first chunk of its cell; heavy: its first slot
  int* piece_last = piece_chunk + pieces_at_a_time;                    // last column
  const int tid = threadIdx.x;
  const bool with_stream = ss.stream != nullptr, gapless = cs.long_len >= kChunkSlots;
  if (copy_wg == 0 && tid < kChunkSlots) {  // the spare entries past the end of the arrays
    a.cols[a.S + a.T + tid] = 0;
    a.vals[a.S + a.T + tid] = 0.f;
  }
  const int parts_at_a_time = pieces_at_a_time >> log2_rows;
  const int row_mask = (1 << cs.log2_rb) - 1;

  int r0 = 0;
  // one slot of the stream: entry (or pad, real == false) number j of piece i
  auto put = [&](int i, int p, int rl, int j, int32_t col, float val, bool real) {
    const int len = piece_len[i], chunk_or_slot = piece_chunk[i];
    int64_t chunk;
    int slot, field, flag, code = 7;
    uint32_t col_field = (uint32_t)col;
    if (len > cs.long_len) {
      // all slots of a chunk name the slot at which a piece ends in it: this one, or (nothing lies between two pieces
      // unless each starts a chunk) the one before it
      const int64_t x = (int64_t)chunk_or_slot + j, e0 = x / kChunkSlots * kChunkSlots;
      const int64_t last = (int64_t)chunk_or_slot + len - 1 - e0;
      const bool ends = last >= 0 && last < kChunkSlots, before = !ends && gapless && chunk_or_slot > e0;
      chunk = a.heavy_chunk0 + x / kChunkSlots;
      slot = (int)(x - e0);
      flag = ends || before;
      field = ends ? (int)last : before ? (int)(chunk_or_slot - 1 - e0) : 0;
    } else {
      const uint32_t word = piece_word[i];
      field = (r0 + rl) & row_mask;
      col_field -= cs.n_phases == 1 ? 0u : (uint32_t)((int64_t)(p / cs.ppg) * ss.phase_width);
      if (word & kWidePiece) {
        chunk = (int64_t)chunk_or_slot + (word & ~kWidePiece) + j / kChunkSlots;
        slot = j % kChunkSlots;
        flag = j / kChunkSlots == (len - 1) / kChunkSlots;
      } else {
        int pos, queue = (int)(word >> 28);
        flag = j == len - 1;
        if (MAY_CUT && (word & kCutPiece)) {
          const int per_queue = (int)((word & (kCutPiece - 1)) >> kCutPosBits) * 8;
          pos = (int)(word & (kCutQueueMax - 1)) + j;
          const int in_next = pos - j + len - per_queue;  // the first so many entries are in the next queue
          flag |= j == in_next - 1;
          if (j < in_next) { pos = j; ++queue; } else { pos -= in_next; }
        } else {
          pos = (int)(word & 0x0FFFFFFFu) + j;
        }
        chunk = (int64_t)chunk_or_slot + (pos >> 3);
        slot = queue * 8 + (pos & 7);
        code = 3;
      }
    }
    if (ss.compact)
      put_slot(ss, chunk, slot,
               (int32_t)(col_field | ((uint32_t)field << kCompactColBits) | ((uint32_t)real << 27) | ((uint32_t)code << 28) |
                         ((uint32_t)flag << 31)),
               real ? __float_as_int(val) : 0, 0);
    else
      put_slot(ss, chunk, slot, col, real ? __float_as_int(val) : 0,
               real ? (field | ((code == 3 ? 3 : kRowLog2W) << 16) | (flag << 22)) : -1);
  };

  // Workgroup ids go round the 8 XCDs: ids b, b + 8, b + 16, .. take consecutive ranges, so that the lines two ranges
  // write parts of (pieces of neighbouring rows lie next to each other) meet in one L2.
  const int64_t per_xcd = ((int64_t)n_copy + 7) / 8;
  int64_t work = (int64_t)(copy_wg & 7) * per_xcd + (copy_wg >> 3);
  // (a grid that is no multiple of 8 leaves the last XCDs one workgroup short: numbers past the end wrap into the gaps)
  const int full = (int)(n_copy & 7);
  if (full != 0 && (int)(copy_wg & 7) >= full) work -= (int)(copy_wg & 7) - full;
  const int64_t first = work * a.per_wg;
  const int64_t last = first + a.per_wg < a.nnz ? first + a.per_wg : a.nnz;
  // A workgroup's first entries are on their way while it finds out where they go.
  constexpr int kUnroll = 4;
  int32_t col[kUnroll];
  float val[kUnroll];
  auto fetch = [&](unsigned e0) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const unsigned e = e0 + u * 256 + tid;
      col[u] = 0; val[u] = 0.f;
      if (e < (unsigned)last) { col[u] = a.indices[e]; val[u] = a.values[e]; }
    }
  };
  unsigned held = (unsigned)first;  // the entries that col and val hold: from here on
  fetch(held);
  for (int64_t at = first; at < last;) {
    r0 = row_of_entry(a.indptr, s.n_rows, at, tid & 63);
    __syncthreads();  // (the last block's rows are no longer read)
    for (int i = tid; i <= n_rows_here; i += 256) row_lo[i] = a.indptr[i < s.n_rows - r0 ? r0 + i : s.n_rows];
    __syncthreads();
    const unsigned e_begin = (unsigned)at;
    const unsigned e_end = row_lo[n_rows_here] < last ? (unsigned)row_lo[n_rows_here] : (unsigned)last;
    at = e_end;
    for (int p0 = 0; p0 < s.c; p0 += parts_at_a_time) {
      const int np = s.c - p0 < parts_at_a_time ? s.c - p0 : parts_at_a_time;
      if (p0 > 0) __syncthreads();  // (the pieces of the last turn are no longer read)
      for (int i = tid; i < np << log2_rows; i += 256) {
        const int p = p0 + (i >> log2_rows), rl = i & (n_rows_here - 1);
        if (rl >= s.n_rows - r0 || (unsigned)row_lo[rl] >= e_end) { piece_len[i] = 0; continue; }  // (none of its entries is here)
        const int r = r0 + rl;
        // (everything that the row alone decides is on its way before the piece's position is needed)
        const int32_t q = a.piece_of[(int64_t)p * s.n_rows + r];
        int lo, len;
        row_piece(s, a.indptr, a.bound, r, p, &lo, &len);
        int64_t group_first = 0;
        const long long* cell = nullptr;
        if (with_stream) {
          const int64_t grp = (int64_t)(p / cs.ppg) * cs.n_rb + (r >> cs.log2_rb);
          cell = a.cell_first_chunk + grp * cells_per_group(cs) + (int64_t)(p % cs.ppg) * cells_per_part(cs);
          group_first = a.group_first_chunk[grp];
        }
        piece_lo[i] = lo;
        piece_len[i] = len;
        if (len <= 0) continue;
        const int bin = bin_of_length(len, s.k);
        const int64_t b = (int64_t)p * (s.k + 1) + bin;
        piece_last[i] = a.indices[lo + len - 1];
        piece_dst[i] = bin <= s.k ? (uint32_t)(a.bucket_slot_ptr[b] + ((q - a.bucket_row_ptr[b]) << bin))
                                  : (uint32_t)(a.S + a.rem_ptr[q - a.R]);
        if (!with_stream) continue;
        if (row_lo[rl + 1] - row_lo[rl] >= a.min_deg) {
          piece_chunk[i] = -1;
        } else if (len > cs.long_len) {
          piece_word[i] = 0;
          piece_chunk[i] = (int)(uint32_t)a.unit[q];
        } else {
          const int64_t queue = cell[cs.nb], wide = cell[bin];
          const uint32_t word = a.dealt[q];
          piece_word[i] = word;
          piece_chunk[i] = (int)(group_first + ((word & kWidePiece) ? wide : queue));
        }
      }
      __syncthreads();
      for (unsigned e0 = (unsigned)first + (e_begin - (unsigned)first) / (256 * kUnroll) * (256 * kUnroll); e0 < e_end; e0 += 256 * kUnroll) {
        if (e0 != held) { held = e0; fetch(e0); }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const unsigned e = e0 + u * 256 + tid;
          if (e < e_begin || e >= e_end) continue;
          int rl = 0;  // the last row that starts at or before e
          for (int step = n_rows_here >> 1; step > 0; step >>= 1)
            if ((unsigned)row_lo[rl + step] <= e) rl += step;
          int p = (int)((double)col[u] * a.inv_w);  // off by one at most
          const int over = (int)((unsigned)col[u] - (unsigned)p * (unsigned)s.w);
          p += over >= s.w ? 1 : over < 0 ? -1 : 0;
          if (p < p0 || p >= p0 + np) continue;
          const int i = ((p - p0) << log2_rows) + rl;
          const int j = (int)(e - (unsigned)piece_lo[i]);
          const int len = piece_len[i];
          const uint32_t dst = piece_dst[i] + (uint32_t)j;
          a.cols[dst] = col[u];
          a.vals[dst] = val[u];
          // Pads: number j of a piece is written with its entry j (a bucket row is less than half pads).  Those of a bucket
          // row repeat the last column and hold +0.0f.
          const int bin = bin_of_length(len, s.k);
          if (bin <= s.k && j < (1 << bin) - len) {
            a.cols[dst + (uint32_t)len] = piece_last[i];
            a.vals[dst + (uint32_t)len] = 0.f;
          }
          if (!with_stream || piece_chunk[i] < 0) continue;
          put(i, p, rl, j, col[u], val[u], true);
          // In the stream the last chunk of a piece cut wide, and of a heavy piece that no other follows in its chunk, is
          // filled with marked slots that repeat the last column too; the last heavy piece also fills its quad.
          int pads = 0;
          if (len > cs.long_len) {
            const int64_t end = (int64_t)piece_chunk[i] + len;
            const int to_chunk = (int)((kChunkSlots - end % kChunkSlots) % kChunkSlots);
            const bool last_piece = end + (gapless ? 0 : to_chunk) == a.heavy_slots;
            if (!gapless || last_piece) pads = to_chunk;
            if (last_piece)
              for (int64_t x = end + to_chunk + j; x < a.n_heavy_chunks * kChunkSlots; x += len)
                put_slot(ss, a.heavy_chunk0 + x / kChunkSlots, (int)(x % kChunkSlots),
                         ss.compact ? (int32_t)0xF0000000u : 0, 0, -1);
          } else if (piece_word[i] & kWidePiece) {
            pads = (kChunkSlots - len % kChunkSlots) % kChunkSlots;
          }
          for (int k = j; k < pads; k += len) put(i, p, rl, len + k, piece_last[i], 0.f, false);
        }
      }
    }
  }
}

// --------------------------------------------------------------- host helpers
// Pinned host memory for the few small arrays a build exchanges with the device.  The blocks are kept for the life
// of the process (pinning memory costs more than a small build) and lent to one build at a time.
class PinnedPool {
 public:
  using Buf = PinnedBuf;
  Buf acquire(size_t bytes) {
    {
      std::lock_guard<std::mutex> g(m_);
      for (size_t i = 0; i < free_.size(); ++i)
        if (free_[i].size >= bytes) {
          Buf b = free_[i];
          free_.erase(free_.begin() + (long)i);
          return b;
        }
    }
    Buf b;
    b.size = std::max<size_t>(bytes, 64 * 1024);
    void* p = nullptr;
    if (hipHostMalloc(&p, b.size, hipHostMallocPortable) != hipSuccess) { (void)hipGetLastError(); b.size = 0; return b; }
    b.p = (char*)p;
    return b;
  }
  void release(Buf b) {
    if (!b.p) return;
    {
      std::lock_guard<std::mutex> g(m_);
      if (free_.size() < 8) { free_.push_back(b); return; }
    }
    (void)hipHostFree(b.p);
  }

 private:
  std::mutex m_;
  std::vector<Buf> free_;
};
PinnedPool& pinned_pool() {
  static PinnedPool* pool = new PinnedPool();  // never destroyed: no HIP call at process exit
  return *pool;
}

struct ValidationGrid {
  int row_wgs, elem_wgs, vec;
  explicit ValidationGrid(const sptir_csr_t* csr)
      : row_wgs((int)std::min<int64_t>(((int64_t)csr->n_rows + 255) / 256, 4096)),
        elem_wgs((int)std::min<int64_t>((csr->nnz + 2047) / 2048, 8192)),
        vec((((uintptr_t)csr->indices | (uintptr_t)csr->values) & 15) == 0) {}
};

struct Blob {  // bump allocator over one device allocation
  char* base = nullptr;
  size_t size = 0;
  size_t reserve(size_t bytes) {
    size_t off = size;
    size = (size + bytes + 255) & ~(size_t)255;
    return off;
  }
};

// data[i] += seq_base[i / kScanSeq]: the last step of the device-wide exclusive scan
__global__ void k_add_seq_base(int64_t n, int32_t* data, const int32_t* __restrict__ seq_base) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) data[i] += seq_base[i / kScanSeq];
}

// Exclusive scan of data[0 .. n) in place on `stream`; data must have room for n rounded up to whole sequences
// (the tail is zeroed here), seq_base for one int per sequence plus one.
}  // namespace
sptir_status_t device_exclusive_scan(int32_t* data, int64_t n, int32_t* seq_base, hipStream_t stream) {
  if (n <= 0) return SPTIR_OK;
  const int64_t n_seq = (n + kScanSeq - 1) / kScanSeq;
  if (n_seq * kScanSeq > n)
    SPTIR_HIP(hipMemsetAsync(data + n, 0, sizeof(int32_t) * (size_t)(n_seq * kScanSeq - n), stream));
  hipLaunchKernelGGL(k_scan_sequences<int32_t>, dim3((unsigned)n_seq), dim3(kBuildBlock), 0, stream, data,
                     (int32_t)kScanSeq, seq_base);
  hipLaunchKernelGGL(k_scan_sequences<int32_t>, dim3(1), dim3(kBuildBlock), 0, stream, seq_base, (int32_t)n_seq,
                     seq_base + n_seq);
  hipLaunchKernelGGL(k_add_seq_base, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, n, data, seq_base);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}
size_t scan_room(int64_t n) { return (size_t)((n + kScanSeq - 1) / kScanSeq) * kScanSeq; }

PinnedBuf pinned_acquire(size_t bytes) { return pinned_pool().acquire(bytes); }
void pinned_release(PinnedBuf b) { pinned_pool().release(b); }

void launch_validation(const sptir_csr_t* csr, bool with_values, unsigned long long* flags, hipStream_t stream,
                       int32_t min_deg) {
  const int32_t* value_bits = with_values ? (const int32_t*)csr->values : nullptr;
  const ValidationGrid v(csr);
  if (v.row_wgs + v.elem_wgs > 0)
    hipLaunchKernelGGL(k_validate, dim3((unsigned)(v.row_wgs + v.elem_wgs)), dim3(256), 0, stream, v.row_wgs, csr->n_rows,
                       csr->nnz, csr->n_cols, v.vec, csr->indptr, csr->indices, value_bits, min_deg, flags);
}

sptir_status_t validation_verdict(const unsigned long long* flag_slots, bool* one_value_per_row) {
  unsigned long long flags[6] = {0, 0, 0, 0, 0, 0};
  for (int slot = 0; slot < kFlagSlots; ++slot)
    for (int i = 0; i < 6; ++i) flags[i] += flag_slots[slot * kFlagStride + i];
  if (flags[0]) return SPTIR_ERR_INVALID_ARG;
  if (flags[1] || flags[2] != flags[3]) return SPTIR_ERR_UNSORTED;
  if (one_value_per_row) *one_value_per_row = flags[4] == flags[5];
  return SPTIR_OK;
}

namespace {

int log2_row_block_setting(int32_t n_rows, bool rounds, bool several_launches, bool full_rows,
                           const sptir_build_options_t& opt) {
  long v = opt.row_block;
  if ((v < 8 || v > 256 || (v & (v - 1))) && full_rows) {
    // 16 rows x 512 bytes: the same 8 KB of LDS per wavefront as 64 rows of a 128-byte tile
    v = 16;
    while (v > 8 && n_rows / v < 1024) v >>= 1;
  } else if (v < 8 || v > 256 || (v & (v - 1))) {
    // A wavefront walks the list of one row block alone and keeps the block's tile of Y in LDS:
    // 64 rows x 128 bytes = 8 KB next to its 4 KB (6 KB) chunk ring allow 12 wavefronts per CU.  Measured on
    // the two large graphs with a launch per partition: 32 rows cost 3 % (more lists, each rounded up to whole
    // chunks), 128 rows 12 - 25 % (fewer wavefronts per CU); the low-degree graphs do not care.  In rounds the
    // lists hold short pieces only and 128 rows win (fewer, longer lists: 6 % on the largest graph).  128 rows is
    // the most a compact record can address.
    v = rounds ? 128 : 64;
    // A launch has (row blocks x feature tiles) wavefronts.  With one or two tiles (feat <= 64) that is too few
    // to balance 3,000 wavefront slots, and smaller row blocks win (measured at feat = 32: 32 rows 21 % faster).
    const long tiles = opt.feat_hint > 0 ? (opt.feat_hint + 31) / 32 : 4;
    // A launch per group of partitions ends in a partly filled GPU that many times: three times the 3,300 wavefronts that
    // are resident at 64 rows keep that small (132,534 rows, 39.6 M entries, 8 launches, 32 rows instead of 64: 1.07 ->
    // 1.04 ms).  On 80 graphs in several launches the rule is 7 % faster than
    // 64 rows for all and level with 32 or 16 for all; the best size for each graph would be 5 % faster, 29 % at most.
    while (v > 16 && (n_rows / v) * tiles < (several_launches ? 10240 : 6144)) v >>= 1;
    // ... but keep at least ~1024 row blocks, or the 256 CUs do not fill
    while (v > 8 && n_rows / v < 1024) v >>= 1;
  }
  int l = 0;
  while ((1L << l) < v) ++l;
  return l;
}

// Do the X rows of a column partition have to be kept L2-resident while they are gathered (section 4.2.1's reason
// for column partitions)?  Only when rows are long: the gathers of a low-degree graph come from beyond L2 either
// way (measured: 8 slots per row and 4 partitions run 1.7x faster without any ordering by partition).  `fit`
// receives the partitions whose 128-byte-wide slices fit 2.5 MB of an XCD's 4 MB L2 together.
bool partitions_matter(int32_t c, int32_t w, int32_t n_rows, int64_t slots, long* fit_out) {
  const double slice_bytes = (double)w * 128.0;               // one 32-float tile of a partition's X rows
  long fit = (long)(2.5 * 1024 * 1024 / (slice_bytes > 1 ? slice_bytes : 1));
  if (fit < 1) fit = 1;
  *fit_out = fit;
  if (fit >= c) return false;
  const long phases = (c + fit - 1) / fit;
  const double slots_per_row = n_rows > 0 ? (double)slots / n_rows : 0.0;
  return slots_per_row >= 16.0 * (double)(phases - 1);
}

// A wavefront walks a chunk list alone, so the longest list bounds a launch from below, and the lists of a round
// run only as fast as the longest of them.  In rounds every piece longer than one chunk therefore leaves the lists: what
// stays is then so even that the wavefronts of a round sweep the column partitions nearly in step.  Otherwise long
// pieces leave when the longest row shows that lists are uneven; the launches that sum them cost some 8 microseconds:
//  * the longest row (its share of one launch, `longest`) is worth two average lists and 16 chunks or more (32 where there
//    are fewer than 2^19 entries and the whole takes about as long as those launches);
//  * or the graph is large enough for 8 microseconds not to matter;
//  * or it has so few lists that they leave most of the GPU idle.
// One launch of fewer than 1024 lists, no row of kHeavyLenMax entries: none, its lists are shared by the wavefronts of
// workgroups (shared_list_waves() in spmm.hip) and there is no second launch to wait for.  (55 graphs, 0.5 to 3.7 M entries, 16
// to 256 features: 1.01 to 1.59 times as fast in all of them, 1.23 in the mean; 3,265 rows, 666,264 entries, 64 features 18.8 ->
// 12.4 us.)
// An even matrix (no row four times the mean) keeps all of its pieces in the lists.  Pieces leave from one chunk on.
// Measured on 320 graphs with power-law degrees, 2,500 to 235,000 rows, 60,000 to 8 M entries, 32 to 128 features.  Where the
// rule takes pieces out, against the rule before it (nothing out below 2^19 entries, beyond that pieces of more than two
// average lists, 256 to 2048 entries): 1.78 times as fast below 2^19 entries, 1.35 up to 2^20, 1.46 up to 2^21, 1.60 up to
// 2^22, 1.42 beyond (single graphs 0.84 to 3.6); the third case alone 1.45.  160 to 256 features (200 graphs): 1.15, 1.10, 1.07,
// 1.20, 1.15 (0.70 to 2.6: the partial sums of wide rows cost more).  Where it leaves all in the lists, taking them out would be
// 1.13 times as fast in the mean, but 0.78 to 2.0.  From two chunks on instead of one: 8 % slower between 2^20 and 2^21; from four
// on: 12 % slower between 2^19 and 2^20, 9 % below.
int32_t heavy_len_setting(int64_t nnz, int32_t n_rows, int64_t n_row_blocks, int32_t n_phases, int64_t longest_row,
                          bool rounds, const sptir_build_options_t& opt) {
  if (opt.heavy_len >= 1) return opt.heavy_len;
  if (rounds) return kChunkSlots;
  const int64_t n_lists = n_row_blocks * n_phases, per_list = n_lists > 0 ? nnz / n_lists : 0;
  const int64_t longest = longest_row / std::max(1, n_phases);
  if (n_phases == 1 && n_row_blocks < 1024 && longest_row < kHeavyLenMax && nnz < (1 << 22)) return kHeavyLenMax;
  const bool small = nnz < (1 << 19);
  const bool uneven = longest_row * n_rows >= 4 * nnz;
  const bool worth = (longest >= (small ? 32 : 16) * kChunkSlots && longest >= 2 * per_list) || nnz >= (1 << 22) ||
                     (!small && n_row_blocks < 1024 && longest >= 12 * kChunkSlots);
  if (!uneven || !worth) return kHeavyLenMax;
  return kChunkSlots;
}

// Do the long rows leave lists and heavy pieces for column slices (spmm_slices.hip)?  Only where pieces leave the lists at all
// and the longest row has one that does, so that no handle without heavy pieces comes to own partial sums; and from so many
// entries on that a build and ONE product together win: slices cost a build some ten launches and a synchronisation, 50 to 150 us.
// 86 graphs of uniform columns, 16 to 256 features, against column_slices = 2: 4.2 to 12.6 M long entries, build and product 0.94
// times as fast in the mean (0.80 to 1.17; the product alone 1.20); to 16.8 M 1.05 (0.83 to 1.25; 1.45); beyond 1.24 (0.91 to 1.79;
// 1.97).  A caller who multiplies often with fewer asks for them (column_slices = 1).
constexpr int64_t kMinSliceNnz = (int64_t)3 << 22;
bool use_slices(const sptir_build_options_t& opt, int32_t heavy_len, int32_t c, int64_t longest_row, int64_t long_nnz) {
  if (opt.no_spmm_plan || opt.column_slices == 2 || opt.full_rows == 1 || long_nnz == 0) return false;
  if (opt.column_slices == 1) return true;
  return opt.heavy_len < 1 && heavy_len < kHeavyLenMax && longest_row > (int64_t)heavy_len * c && long_nnz >= kMinSliceNnz;
}

}  // namespace

sptir_build_options_t complete_options(const sptir_build_options_t* given) {
  sptir_build_options_t o;
  memset(&o, 0, sizeof(o));
  if (given) {
    size_t n = given->struct_size > 0 ? (size_t)given->struct_size : 0;
    if (n > sizeof(o)) n = sizeof(o);
    memcpy(&o, given, n);
  }
  o.struct_size = (int32_t)sizeof(o);
  return o;
}

LaunchShape decide_launch_shape(int32_t n_rows, int32_t n_cols, int32_t c, int32_t w, int64_t stored_slots,
                                const sptir_build_options_t& opt) {
  LaunchShape ls;
  long fit = 1;
  const bool matter = partitions_matter(c, w, n_rows, stored_slots, &fit);
  // rounds: every list sweeps all partitions, Y stays on chip and is written once; otherwise a launch per group
  // of partitions that reads back what the one before it wrote
  const bool parts_given = opt.parts_per_launch >= 1 && opt.parts_per_launch <= c;
  // (rounds pay when the pieces that stay in the lists are short: a read-modify-write of Y per partition then
  //  costs as much as the pieces themselves; with long pieces the wavefronts of a round, which nothing holds in
  //  step, lose more by drifting onto different partitions.  Measured: mean piece of 8 entries, 1.54 -> 1.04 ms;
  //  of 37 entries, 1.11 -> 1.39 ms.)
  const bool short_pieces = opt.light_piece_len == 0 || opt.light_piece_len < 16;
  ls.rounds = opt.rounds == 1 ? 1 : opt.rounds == 2 ? 0 : (matter && !parts_given && short_pieces ? 1 : 0);
  // Whole 512-byte runs of X per entry: only when asked for.  Measured at feat = 128 against the 128-byte tiles
  // bound to XCDs: 7 entries per row 0.108 -> 0.151 ms, 4.5 per row 0.037 -> 0.090 ms, 300 per row
  // 1.09 -> 1.66 ms: two lane groups instead of eight have a quarter of the rows in flight, and every XCD's L2 then sees
  // all of X instead of a quarter of it.
  ls.full_rows = opt.full_rows == 1 ? 1 : 0;
  if (ls.rounds) ls.parts_per_phase = c;
  else if (parts_given) ls.parts_per_phase = opt.parts_per_launch;
  else ls.parts_per_phase = matter ? (int32_t)fit : c;
  ls.log2_row_block = log2_row_block_setting(n_rows, ls.rounds != 0, ls.parts_per_phase < c, ls.full_rows != 0, opt);
  // a compact record holds a column in kCompactColBits bits and a row of the row block in 7
  const int64_t max_span = (int64_t)1 << kCompactColBits;
  ls.compact = (!opt.wide_stream && n_cols <= max_span && ls.log2_row_block <= kCompactMaxLog2RowBlock) ? 1 : 0;
  ls.n_phases = (c + ls.parts_per_phase - 1) / ls.parts_per_phase;
  return ls;
}

}  // namespace sptir

using namespace sptir;

extern "C" sptir_status_t sptir_hyb_build(const sptir_csr_t* csr, int32_t n_col_parts, int32_t max_bucket_log2,
                                          void* stream_, sptir_hyb_t** out) {
  return sptir::hyb_build_impl(csr, n_col_parts, max_bucket_log2, sptir::complete_options(nullptr), stream_, out);
}

extern "C" sptir_status_t sptir_hyb_build_ex(const sptir_csr_t* csr, int32_t n_col_parts, int32_t max_bucket_log2,
                                             const sptir_build_options_t* options, void* stream_, sptir_hyb_t** out) {
  const sptir_build_options_t opt = sptir::complete_options(options);
  if (opt.row_block != 0 && (opt.row_block < 8 || opt.row_block > 256 || (opt.row_block & (opt.row_block - 1))))
    return SPTIR_ERR_INVALID_ARG;
  if (opt.parts_per_launch < 0 || opt.rounds < 0 || opt.rounds > 2 || opt.heavy_len < 0 || opt.sweep_kb < 0 ||
      opt.feat_hint < 0 || opt.full_rows < 0 || opt.full_rows > 2 || opt.column_slices < 0 || opt.column_slices > 2)
    return SPTIR_ERR_INVALID_ARG;
  return sptir::hyb_build_impl(csr, n_col_parts, max_bucket_log2, opt, stream_, out);
}

sptir_status_t sptir::hyb_build_impl(const sptir_csr_t* csr, int32_t n_col_parts, int32_t max_bucket_log2,
                                     const sptir_build_options_t& opt, void* stream_, sptir_hyb_t** out) {
  const bool with_spmm_plan = !opt.no_spmm_plan;
  if (!csr || !out) return SPTIR_ERR_INVALID_ARG;
  if (csr->n_rows < 0 || csr->n_cols < 0 || csr->nnz < 0) return SPTIR_ERR_INVALID_ARG;
  if (n_col_parts < 1 || max_bucket_log2 < 0 || max_bucket_log2 > 30) return SPTIR_ERR_INVALID_ARG;
  if (csr->nnz >= ((int64_t)1 << 31)) return SPTIR_ERR_OVERFLOW;
  if (!csr->indptr || (csr->nnz > 0 && (!csr->indices || !csr->values))) return SPTIR_ERR_INVALID_ARG;
  if (csr->nnz > 0 && (csr->n_rows == 0 || csr->n_cols == 0)) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;

  BuildShape s;
  s.n_rows = csr->n_rows; s.n_cols = csr->n_cols; s.c = n_col_parts; s.k = max_bucket_log2;
  s.w = (int32_t)(((int64_t)csr->n_cols + n_col_parts - 1) / n_col_parts);
  s.nb = s.k + 2;
  s.NB = (s.n_rows + kBuildBlock - 1) / kBuildBlock;
  const int64_t n_pair_blocks = (int64_t)s.NB * s.c;
  if (n_pair_blocks > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  const int64_t B = (int64_t)s.c * (s.k + 1);
  if (B > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;

  sptir_alloc_fn alloc; sptir_free_fn free_; void* actx;
  current_allocator(&alloc, &free_, &actx);

  // ---- temporary storage: one device blob now, a second one once the cell count is known; one pinned host block
  // for everything that crosses to or from the host (pageable memory would make every small copy a blocking one)
  const size_t nbk = (size_t)(s.NB ? s.NB : 1);
  Blob tmp;
  const size_t o_flags = tmp.reserve((kValidationWords + 2) * sizeof(unsigned long long));  // (the last two: HeavySums::not_taken)
  const size_t o_counts = tmp.reserve(sizeof(int32_t) * (size_t)s.c * s.nb * nbk);
  const size_t o_rnnz = tmp.reserve(sizeof(int64_t) * (size_t)s.c * nbk);
  const size_t o_bound = tmp.reserve(sizeof(int32_t) * (size_t)(s.c - 1) * (size_t)(s.n_rows ? s.n_rows : 1) + 16);
  const int64_t n_bound_blocks =
      (((int64_t)s.n_rows + kBoundRows - 1) / kBoundRows) * (((int64_t)s.c - 1 + kBoundParts - 1) / kBoundParts);
  if (n_bound_blocks > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  Blob host;
  const size_t h_flags = host.reserve(kValidationWords * sizeof(unsigned long long));
  const size_t h_tot_rnnz = host.reserve(sizeof(int64_t) * (size_t)s.c);
  const size_t h_tot_bins = host.reserve(sizeof(int32_t) * (size_t)s.c * s.nb);
  // (these four reach the device in one copy, into the start of the handle's first allocation)
  Blob ba;
  const size_t a_row_ptr = ba.reserve(sizeof(int64_t) * (size_t)(B + 1));
  const size_t a_slot_ptr = ba.reserve(sizeof(int64_t) * (size_t)(B + 1));
  const size_t a_rem_part = ba.reserve(sizeof(int32_t) * (size_t)(s.c + 1));
  const size_t a_rnnz_base = ba.reserve(sizeof(int64_t) * (size_t)s.c);
  const size_t small_bytes = ba.size;
  const size_t h_small = host.reserve(small_bytes);
  const size_t h_report2 = host.reserve(sizeof(long long) * kReport2);
  const size_t h_report3 = host.reserve(sizeof(int32_t) * 2);
  const size_t h_misc = host.reserve(64);
  PinnedPool::Buf pinned = pinned_pool().acquire(host.size);
  if (!pinned.p) return SPTIR_ERR_ALLOC;
  host.base = pinned.p;
  tmp.base = (char*)scratch_alloc(tmp.size, alloc, actx, stream);
  if (!tmp.base) { pinned_pool().release(pinned); return SPTIR_ERR_ALLOC; }
  Blob tmp2;
  void* tmp_order = nullptr;
  SpmmSliceBuild slice_build;
  int32_t min_deg = INT32_MAX;

  sptir_hyb* h = new (std::nothrow) sptir_hyb();
  if (!h) { scratch_free(tmp.base, free_, actx); pinned_pool().release(pinned); return SPTIR_ERR_ALLOC; }
  h->alloc = alloc; h->free_ = free_; h->alloc_ctx = actx;
  h->n_rows = s.n_rows; h->n_cols = s.n_cols; h->c = s.c; h->k = s.k; h->w = s.w;
  h->nnz = csr->nnz; h->B = B;

  // every exit after this point goes through `fail`
  sptir_status_t st = SPTIR_OK;
#define BUILD_HIP(call)                                              \
  do {                                                               \
    hipError_t e_ = (call);                                          \
    if (e_ != hipSuccess) { st = note_hip_error(e_, #call); goto fail; } \
  } while (0)

  {
    unsigned long long* d_flags = (unsigned long long*)(tmp.base + o_flags);
    int32_t* d_counts = (int32_t*)(tmp.base + o_counts);
    int64_t* d_rnnz = (int64_t*)(tmp.base + o_rnnz);
    int32_t* d_bound = (int32_t*)(tmp.base + o_bound);

    // ---- validation of the CSR input, and with it (their results are only used if the input is valid, and they
    // read nothing at a position the input names without clamping it) the piece boundaries, histogram and scans
    const FirstReport report1{(unsigned long long*)(host.base + h_flags), (int64_t*)(host.base + h_tot_rnnz),
                              (int32_t*)(host.base + h_tot_bins)};
    bool one_value = false;
    const int64_t* tot_rnnz = report1.rem_nnz;
    const int32_t* tot_bins = report1.bins;
    // (values are only looked at when a value-less stream is an option)
    const int32_t* value_bits = (with_spmm_plan && !opt.keep_values) ? (const int32_t*)csr->values : nullptr;
    BUILD_HIP(hipMemsetAsync(d_flags, 0, (kValidationWords + 2) * sizeof(unsigned long long), stream));
    const bool want_slices = with_spmm_plan && opt.column_slices != 2 && opt.full_rows != 1;
    if (want_slices) min_deg = (int32_t)std::min<int64_t>(INT32_MAX, slice_min_degree(s.n_cols));
    {
      const ValidationGrid v(csr);
      const int64_t n_wg = n_bound_blocks + v.row_wgs + v.elem_wgs;
      if (n_wg > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
      if (n_wg > 0)
        hipLaunchKernelGGL(k_first_pass, dim3((unsigned)n_wg), dim3(256), 0, stream, (unsigned)n_bound_blocks, v.row_wgs, s, csr->nnz,
                           v.vec, csr->indptr, csr->indices, value_bits, min_deg, d_flags, d_bound);
    }
    if (s.NB > 0) {
      hipLaunchKernelGGL(k_count, dim3((unsigned)n_pair_blocks), dim3(kBuildBlock), 0, stream, s, csr->indptr,
                         d_bound, d_counts, d_rnnz);
    }
    hipLaunchKernelGGL(k_first_totals, dim3((unsigned)(s.c * s.nb + s.c + 1)), dim3(kBuildBlock), 0, stream, s, d_counts,
                       d_rnnz, d_flags, report1);
    BUILD_HIP(hipGetLastError());
    BUILD_HIP(hipStreamSynchronize(stream));
    if (s.n_rows == 0) {
      int32_t* first = (int32_t*)(host.base + h_misc);
      BUILD_HIP(hipMemcpyAsync(first, csr->indptr, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
      BUILD_HIP(hipStreamSynchronize(stream));
      if (*first != 0 || csr->nnz != 0) { st = SPTIR_ERR_INVALID_ARG; goto fail; }
    }
    st = validation_verdict(report1.flags, &one_value);
    if (st != SPTIR_OK) goto fail;

    // ---- sizes and the small prefix arrays (host)
    int64_t* row_ptr = (int64_t*)(host.base + h_small + a_row_ptr);
    int64_t* slot_ptr = (int64_t*)(host.base + h_small + a_slot_ptr);
    int32_t* rem_part_ptr = (int32_t*)(host.base + h_small + a_rem_part);
    int64_t* rnnz_base = (int64_t*)(host.base + h_small + a_rnnz_base);
    int64_t M = 0, T = 0;
    row_ptr[0] = 0; slot_ptr[0] = 0; rem_part_ptr[0] = 0;
    for (int32_t p = 0; p < s.c; ++p) {
      for (int32_t i = 0; i <= s.k; ++i) {
        int64_t b = (int64_t)p * (s.k + 1) + i;
        int64_t rows = tot_bins[(size_t)p * s.nb + i];
        row_ptr[b + 1] = row_ptr[b] + rows;
        slot_ptr[b + 1] = slot_ptr[b] + (rows << i);
      }
      rnnz_base[p] = T;
      M += tot_bins[(size_t)p * s.nb + s.k + 1];
      T += tot_rnnz[p];
      if (M > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
      rem_part_ptr[p + 1] = (int32_t)M;
    }
    h->R = row_ptr[B]; h->S = slot_ptr[B]; h->M = M; h->T = T;
    if (h->R + h->M > 0x7FFFFFFF || h->S + T >= 0xFFFFFFFFll) { st = SPTIR_ERR_OVERFLOW; goto fail; }

    // ---- launch shape of the SpMM: row blocks, lists, heavy pieces
    CellShape cs;
    cs.c = s.c; cs.k = s.k; cs.nb = s.nb; cs.R = h->R;
    // mean real length of the pieces of at most kChunkSlots entries, estimated from the bucket sizes
    // (bucket i holds lengths 2^(i-1)+1 .. 2^i)
    sptir_build_options_t opt_here = opt;
    if (opt_here.light_piece_len == 0) {
      double pieces = 0, entries = 0;
      for (int32_t p = 0; p < s.c; ++p)
        for (int32_t i = 0; i <= s.k && (1 << i) <= kChunkSlots; ++i) {
          const double n = tot_bins[(size_t)p * s.nb + i];
          pieces += n;
          entries += n * (i == 0 ? 1.0 : 0.5 * ((1 << (i - 1)) + 1 + (1 << i)));
        }
      opt_here.light_piece_len = pieces > 0 ? std::max(1, (int)(entries / pieces + 0.5)) : 0;
    }
    const LaunchShape ls = decide_launch_shape(s.n_rows, s.n_cols, s.c, s.w, h->S + h->T, opt_here);
    cs.ppg = ls.parts_per_phase; cs.log2_rb = ls.log2_row_block; cs.n_phases = ls.n_phases;
    h->compact_stream = ls.compact;
    h->rounds = ls.rounds;
    h->full_rows = ls.full_rows;
    // Every row has one value for all its entries (a row-normalised adjacency matrix, say): the stream
    // carries no values, the kernels sum rows of X and scale each row of Y once.
    const bool one_value_per_row = value_bits && csr->nnz > 0 && one_value;
    h->sweep_kb = opt.sweep_kb;  // (0: the defaults of the two sweep rules)
    cs.n_rb = (int32_t)(((int64_t)s.n_rows + (1 << cs.log2_rb) - 1) >> cs.log2_rb);
    int64_t longest_row = 0;
    for (int slot = 0; slot < kFlagSlots; ++slot)
      longest_row = std::max<int64_t>(longest_row, (int64_t)report1.flags[slot * kFlagStride + 6]);
    cs.wide_margin = ls.rounds ? 32 : 16;
    cs.long_len = heavy_len_setting(csr->nnz, s.n_rows, cs.n_rb, cs.n_phases, longest_row, ls.rounds != 0, opt);
    // Queues are cut where rows are long and all in the lists, in several launches: 85 drawn graphs, products 1.05 x (0.986 to 1.34), 27 more,
    // a build and one product 1.02 x (0.982 to 1.19).  In one launch, whose lists sweep X beyond L2, it lost (50,970 rows of 496: 0.89 x,
    // measured with queues that began in the middle of a row); with heavy pieces, or rows of fewer than 16, what is left to deal is short and
    // divides evenly (12 graphs: 1.00, builds 0.99).
    cs.cut_queues = cs.n_phases > 1 && longest_row <= cs.long_len && csr->nnz >= 16 * (int64_t)s.n_rows * s.c;
    if (opt.heavy_len < 1 && !ls.rounds && cs.long_len < kHeavyLenMax) {
      // sptir_spmm_noalloc has room for so many narrow partial-sum rows; bucket i > 6 holds the pieces of
      // 2^(i-1)+1 .. 2^i entries, and a heavy list takes at least the entries of 16 chunks once there are thousands
      const int64_t most = (int64_t)(SPTIR_NOALLOC_SCRATCH_BYTES / sizeof(float)) / (ls.full_rows ? kPartialFeat : kNarrowPartialFeat);
      auto partial_rows = [&](int32_t len) {
        int64_t n = std::max<int64_t>(csr->nnz / (kHeavyListChunks * kChunkSlots), 2 * 4096);
        for (int32_t p = 0; p < s.c; ++p)
          for (int32_t i = 0; i < s.nb; ++i)
            if (i == s.k + 1 || ((int64_t)1 << i) > len) n += tot_bins[(size_t)p * s.nb + i];
        return n;
      };
      while (cs.long_len < kHeavyLenMax && partial_rows(cs.long_len) > most) cs.long_len *= 2;
      h->lowered_heavy_len = 1;
    }
    h->heavy_len = cs.long_len;
    int64_t n_long = 0, long_nnz = 0;
    for (int slot = 0; slot < kFlagSlots; ++slot) {
      n_long += (int64_t)(report1.flags[slot * kFlagStride + 7] >> 32);
      long_nnz += (int64_t)(uint32_t)report1.flags[slot * kFlagStride + 7];
    }
    // Without slices after all: `st` says why, nothing that uses their memory is running.  No build ends here for their sake
    // unless the caller has asked for them.
    auto no_slices = [&]() {
      scratch_free(h->slices.blob, free_, actx);
      h->slices = SpmmSlices();
      spmm_slices_done(&slice_build, free_, actx);
      min_deg = INT32_MAX; n_long = 0;
      st = SPTIR_OK;
    };
    auto slices_or_none = [&]() {  // false: the build fails
      if (st == SPTIR_OK) return true;
      if (opt.column_slices == 1 || (st != SPTIR_ERR_ALLOC && st != SPTIR_ERR_OVERFLOW)) return false;
      no_slices();
      return true;
    };
    if (!use_slices(opt, cs.long_len, s.c, longest_row, long_nnz)) { min_deg = INT32_MAX; n_long = 0; }
    if (n_long > 0) {
      st = spmm_slices_count(&slice_build, csr, min_deg, (int32_t)n_long, longest_row, alloc, actx, stream);
      if (!slices_or_none()) goto fail;
    }
    if (!with_spmm_plan) cs.n_rb = 0;  // no row blocks, no cells, no chunks: only the canonical arrays are built
    h->spmm_plan = with_spmm_plan ? 1 : 0;
    h->log2_row_block = cs.log2_rb; h->n_row_blocks = cs.n_rb;
    h->parts_per_phase = cs.ppg; h->n_phases = cs.n_phases;
    const int64_t n_pieces = h->R + M;
    const int64_t n_groups = (int64_t)cs.n_phases * cs.n_rb;
    const int64_t n_cells = n_groups * ((int64_t)cs.ppg * (cs.nb + 1) + 1);
    const int64_t n_parts = n_groups * cs.ppg;
    const int64_t n_bounds = (int64_t)s.c * s.nb * ((int64_t)cs.n_rb + 1);
    if (n_cells > 0x7FFFFFFF || n_bounds > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
    const size_t o_bounds = tmp2.reserve(sizeof(int32_t) * (size_t)(n_bounds ? n_bounds : 1));
    const size_t o_cell_chunks = tmp2.reserve(sizeof(long long) * (size_t)(n_cells ? n_cells : 1));
    const size_t o_group_tot = tmp2.reserve(sizeof(long long) * (size_t)(n_groups + 1));
    const size_t o_queue_len = tmp2.reserve(sizeof(int32_t) * 8 * (size_t)(n_parts ? n_parts : 1));
    const size_t o_piece_of = tmp2.reserve(sizeof(int32_t) * (size_t)s.c * (size_t)(s.n_rows ? s.n_rows : 1));
    // per piece: what the lists do with it, or its number among the heavy pieces; the sums of the scans
    const bool want_heavy = with_spmm_plan && n_pieces > 0;
    const int64_t n_spans = want_heavy ? (n_pieces + kHeavySpan - 1) / kHeavySpan : 0;
    const size_t o_dealt = tmp2.reserve(sizeof(uint32_t) * (size_t)(want_heavy ? n_pieces : 1));
    const size_t o_unit = tmp2.reserve(sizeof(long long) * (size_t)(want_heavy ? n_pieces : 1));
    const size_t o_spans = tmp2.reserve(sizeof(long long) * 3 * (size_t)(n_spans ? n_spans : 1));
    const size_t o_row_sums = tmp2.reserve(sizeof(long long) * nbk);
    tmp2.base = (char*)scratch_alloc(tmp2.size, alloc, actx, stream);
    if (!tmp2.base) { st = SPTIR_ERR_ALLOC; goto fail; }
    int32_t* d_bounds = (int32_t*)(tmp2.base + o_bounds);
    long long* d_cell_chunks = (long long*)(tmp2.base + o_cell_chunks);
    long long* d_group_tot = (long long*)(tmp2.base + o_group_tot);
    int32_t* d_queue_len = (int32_t*)(tmp2.base + o_queue_len);
    int32_t* d_piece_of = (int32_t*)(tmp2.base + o_piece_of);
    uint32_t* d_dealt = (uint32_t*)(tmp2.base + o_dealt);
    unsigned long long* d_unit = (unsigned long long*)(tmp2.base + o_unit);
    HeavySums sums;
    sums.units = (long long*)(tmp2.base + o_spans); sums.slots = sums.units + n_spans; sums.entries = sums.slots + n_spans;

    // ---- the handle's device arrays whose sizes are known now: two allocations (cols and vals can be released
    // on their own); the arrays of the SpMM plan follow further down
    {
      Blob bb;
      const size_t a_rem_ptr = ba.reserve(sizeof(int64_t) * (size_t)(M + 1));
      // (row_ids, cols and vals end in kChunkSlots spare zero entries)
      const size_t a_row_ids = ba.reserve(sizeof(int32_t) * (size_t)(h->R + M + kChunkSlots));
      const size_t a_row_len = ba.reserve(sizeof(int32_t) * (size_t)(h->R + M + 1));
      const size_t a_rb_chunk = ba.reserve(sizeof(int64_t) * ((size_t)cs.n_phases * cs.n_rb + 1));
      const size_t a_row_val = ba.reserve(one_value_per_row ? sizeof(float) * (size_t)s.n_rows : 0);
      const size_t a_row_slot = ba.reserve(want_heavy ? sizeof(int32_t) * ((size_t)s.n_rows + 1) : 0);
      const size_t b_cols = bb.reserve(sizeof(int32_t) * (size_t)(h->S + T + kChunkSlots));
      const size_t b_vals = bb.reserve(sizeof(float) * (size_t)(h->S + T + kChunkSlots));
      size_t index_bytes = 0;
      h->blobs[0] = scratch_alloc(ba.size, alloc, actx, stream, &index_bytes);
      h->blobs[1] = scratch_alloc(bb.size, alloc, actx, stream, &h->canonical_bytes);
      if (!h->blobs[0] || !h->blobs[1]) { st = SPTIR_ERR_ALLOC; goto fail; }
      h->device_bytes += index_bytes + h->canonical_bytes;
      char* a0 = (char*)h->blobs[0];
      char* b0 = (char*)h->blobs[1];
      h->bucket_row_ptr = (int64_t*)(a0 + a_row_ptr); h->bucket_slot_ptr = (int64_t*)(a0 + a_slot_ptr);
      h->rem_part_ptr = (int32_t*)(a0 + a_rem_part); h->rem_ptr = (int64_t*)(a0 + a_rem_ptr);
      h->row_ids = (int32_t*)(a0 + a_row_ids); h->row_len = (int32_t*)(a0 + a_row_len);
      h->rb_chunk_ptr = (int64_t*)(a0 + a_rb_chunk);
      if (one_value_per_row) h->row_val = (float*)(a0 + a_row_val);
      if (want_heavy) h->row_slot_ptr = (int32_t*)(a0 + a_row_slot);
      h->cols = (int32_t*)(b0 + b_cols); h->vals = (float*)(b0 + b_vals);
    }
    if (one_value_per_row) {
      hipLaunchKernelGGL(k_row_values, dim3((unsigned)((s.n_rows + 255) / 256)), dim3(256), 0, stream, s.n_rows,
                         csr->indptr, csr->values, h->row_val);
      BUILD_HIP(hipGetLastError());
    }
    BUILD_HIP(hipMemcpyAsync(h->blobs[0], host.base + h_small, small_bytes, hipMemcpyHostToDevice, stream));

    // ---- do the long rows go to column slices?  (Their lengths alone do not say how far the steps are padded.)
    if (n_long > 0) {
      BUILD_HIP(hipStreamSynchronize(stream));
      if (opt.column_slices != 1 && !spmm_slices_even(slice_build, long_nnz)) {
        no_slices();
      } else {
        st = spmm_slices_plan(&slice_build, opt.feat_hint, !one_value_per_row, &h->slices, alloc, actx, stream);
        h->blobs[3] = h->slices.blob;
        if (!slices_or_none()) goto fail;
      }
      h->blobs[3] = h->slices.blob;  // (none: NULL)
      h->device_bytes += h->slices.device_bytes;
    }
    sums.not_taken = n_long > 0 ? d_flags + kValidationWords : nullptr;

    // ---- stable placement
    if (s.NB > 0) {
      PlaceArgs a;
      a.indptr = csr->indptr; a.bound = d_bound; a.counts = d_counts; a.rem_nnz = d_rnnz;
      a.bucket_row_ptr = h->bucket_row_ptr; a.rem_part_ptr = h->rem_part_ptr;
      a.rem_nnz_base = (const int64_t*)((char*)h->blobs[0] + a_rnnz_base);
      a.row_ids = h->row_ids; a.rem_ptr = h->rem_ptr; a.row_len = h->row_len; a.piece_of = d_piece_of;
      a.R = h->R; a.M = M; a.T = T; a.min_deg = min_deg;
      hipLaunchKernelGGL(k_place, dim3((unsigned)n_pair_blocks), dim3(kBuildBlock), 0, stream, s, a);
    } else {
      int64_t* zero = (int64_t*)(host.base + h_misc + 8);
      *zero = 0;
      BUILD_HIP(hipMemcpyAsync(h->rem_ptr, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
      BUILD_HIP(hipMemsetAsync(h->row_ids + h->R + M, 0, sizeof(int32_t) * kChunkSlots, stream));
      BUILD_HIP(hipMemsetAsync(h->cols + h->S + T, 0, sizeof(int32_t) * kChunkSlots, stream));
      BUILD_HIP(hipMemsetAsync(h->vals + h->S + T, 0, sizeof(float) * kChunkSlots, stream));
    }
    BUILD_HIP(hipGetLastError());
    {
      const int64_t n_wg = n_spans + (n_cells > 0 ? (n_bounds + kBuildBlock - 1) / kBuildBlock : 0);
      if (n_wg > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
      if (n_wg > 0)
        hipLaunchKernelGGL(k_sums_and_cells, dim3((unsigned)n_wg), dim3(kBuildBlock), 0, stream, (unsigned)n_spans, n_pieces,
                           h->row_len, cs.long_len, sums, cs, h->bucket_row_ptr, h->rem_part_ptr, h->row_ids, d_bounds);
    }

    // ---- the pieces of every (launch, row block, partition) dealt to its queues; chunks of the lists
    if (n_cells > 0) {
      hipLaunchKernelGGL(cs.cut_queues ? k_deal<true> : k_deal<false>, dim3((unsigned)((n_parts + kDealParts - 1) / kDealParts)), dim3(8 * kDealParts),
                         (sizeof(int) * 2 * kDealParts) << cs.log2_rb, stream, cs, n_parts, d_bounds, h->row_len, d_cell_chunks,
                         d_dealt, d_queue_len);
      hipLaunchKernelGGL(k_group_scan, dim3((unsigned)((n_groups + 3) / 4)), dim3(256), 0, stream, cs, n_groups,
                         d_cell_chunks, d_group_tot);
    }
    hipLaunchKernelGGL(k_totals, dim3(4), dim3(kOneBlock), 0, stream, n_cells > 0 ? n_groups : 0, d_group_tot, n_spans,
                       sums, (long long*)(host.base + h_report2));
    BUILD_HIP(hipGetLastError());
    BUILD_HIP(hipStreamSynchronize(stream));
    const long long* report2 = (const long long*)(host.base + h_report2);
    const long long n_chunks = report2[0];
    h->n_heavy_nnz = report2[4];
    const int64_t max_list_len = report2[1];
    h->longest_list = max_list_len;
    // the lists' chunks come first in the stream (each list a whole number of quads), then the heavy chunks
    // (report2[3]: slots of the heavy sequence)
    const int64_t n_heavy_chunks = (chunks_of_slots(report2[3]) + kChunksPerQuad - 1) / kChunksPerQuad * kChunksPerQuad;
    h->n_chunks = n_chunks;
    h->n_heavy = report2[2];
    h->heavy_chunk0 = n_chunks;
    h->n_heavy_chunks = n_heavy_chunks;
    // Chunks per heavy list: 16 where that still gives thousands of lists; a graph with few heavy chunks gets
    // shorter lists, or its heavy launch would be a handful of wavefronts walking 16 chunks each while the GPU idles.
    int32_t list_chunks = kHeavyListChunks;
    while (list_chunks > kChunksPerQuad && n_heavy_chunks / list_chunks < 4096) list_chunks /= 2;
    h->heavy_list_chunks = list_chunks;
    h->n_heavy_lists = (int32_t)((n_heavy_chunks + list_chunks - 1) / list_chunks);
    h->n_partial_rows = h->n_heavy + h->n_heavy_lists;
    {
      const int64_t chunks = (chunks_of_slots(report2[3] + report2[6]) + kChunksPerQuad - 1) / kChunksPerQuad * kChunksPerQuad;
      int32_t per_list = kHeavyListChunks;
      while (per_list > kChunksPerQuad && chunks / per_list < 4096) per_list /= 2;
      h->whole_partial_rows = h->n_heavy + report2[5] + (chunks + per_list - 1) / per_list;
    }
    if (n_long > 0) {
      h->slices.nnz = long_nnz;
      st = spmm_slices_fill(slice_build, csr, h->slices, stream);
      if (st != SPTIR_OK) goto fail;
    }
    h->partial_feat = h->n_partial_rows <= kWidePartialRows ? kWidePartialFeat : kPartialFeat;
    if (h->n_heavy == 0) h->row_slot_ptr = nullptr;  // (its room in the first allocation stays unused)
    const int64_t all_chunks = n_chunks + n_heavy_chunks;
    if (h->n_partial_rows > 0x7FFFFFFF || all_chunks > 0x7FFFFFFF || report2[3] > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
    // ---- the arrays of the SpMM plan, one allocation.  A row of Y takes
    // one partial-sum row per heavy piece it has plus one per list boundary such a piece crosses, so there are at
    // most n_partial_rows of them; the rows with heavy pieces are at most as many as there are such pieces.
    {
      Blob bc;
      const bool heavy = h->n_heavy > 0;
      const size_t c_first_slot = bc.reserve(heavy ? sizeof(int32_t) * (size_t)h->n_heavy_lists : 0);
      const size_t c_row_slots = bc.reserve(heavy ? sizeof(int32_t) * (size_t)h->n_partial_rows : 0);
      const size_t c_heavy_rows = bc.reserve(heavy ? sizeof(int32_t) * (size_t)std::min<int64_t>(s.n_rows, h->n_heavy) : 0);
      const size_t c_rb_order = bc.reserve(sizeof(int32_t) * (size_t)(n_groups ? n_groups : 1));
      const size_t c_stream = bc.reserve(sizeof(int32_t) * ((h->compact_stream ? 2 : 3) - (one_value_per_row ? 1 : 0)) *
                                         kChunkSlots * (size_t)(all_chunks ? all_chunks : 1));
      const size_t c_partial = bc.reserve(heavy ? sizeof(float) * (size_t)h->partial_feat * (size_t)h->n_partial_rows : 0);
      size_t plan_bytes = 0;
      h->blobs[2] = scratch_alloc(bc.size, alloc, actx, stream, &plan_bytes);
      if (!h->blobs[2]) { st = SPTIR_ERR_ALLOC; goto fail; }
      h->device_bytes += plan_bytes;
      char* c0 = (char*)h->blobs[2];
      if (heavy) {
        h->hlist_first_slot = (int32_t*)(c0 + c_first_slot); h->row_slots = (int32_t*)(c0 + c_row_slots);
        h->heavy_rows = (int32_t*)(c0 + c_heavy_rows); h->partial = (float*)(c0 + c_partial);
      }
      if (n_groups > 0) h->rb_order = (int32_t*)(c0 + c_rb_order);
      h->stream = (int32_t*)(c0 + c_stream);
    }
    // ---- launch order of the row blocks: longest list first.  One digit is enough for most graphs; its steps then go with the
    // launches below.  (169,343 rows, 1.17 M entries, build + SpMM + release, with all that shares a launch in the build: 246 -> 217 us.)
    SortPass sort;
    memset(&sort, 0, sizeof(sort));
    const bool sort_here = n_groups > 0 && max_list_len < kDigits;
    if (sort_here) {
      sort.in.list_ptr = (const int64_t*)d_group_tot;
      sort.n_rb = cs.n_rb; sort.n_launches = cs.n_phases;
      sort.tiles = (cs.n_rb + kSortTile - 1) / kSortTile;
      sort.order = h->rb_order;
      tmp_order = scratch_alloc(sizeof(int32_t) * kDigits * (size_t)sort.tiles * (size_t)sort.n_launches, alloc, actx, stream);
      if (!tmp_order) { st = SPTIR_ERR_ALLOC; goto fail; }
      sort.hist = (int32_t*)tmp_order;
    }
    const unsigned sort_wgs = (unsigned)sort.tiles * (unsigned)sort.n_launches;
    // ---- heavy pieces: their numbers and slots, the first partial-sum row of every heavy list, which
    // partial-sum rows each row of Y takes, the rows that have any (the launch that adds them visits only those)
    const bool heavy = h->n_heavy > 0;
    RowSlotArgs slots;
    memset(&slots, 0, sizeof(slots));
    slots.n_rows = s.n_rows; slots.c = s.c; slots.list_chunks = list_chunks; slots.heavy_len = cs.long_len;
    slots.indptr = csr->indptr; slots.piece_of = d_piece_of; slots.row_len = h->row_len; slots.unit = d_unit;
    slots.sums = (unsigned long long*)(tmp2.base + o_row_sums);
    slots.row_slot_ptr = h->row_slot_ptr; slots.row_slots = h->row_slots; slots.heavy_rows = h->heavy_rows;
    const unsigned unit_wgs = heavy ? (unsigned)n_spans : 0, slot_wgs = heavy ? (unsigned)s.NB : 0;
    if (unit_wgs + sort_wgs > 0)
      hipLaunchKernelGGL(k_units_and_hist, dim3(unit_wgs + sort_wgs), dim3(kBuildBlock), 0, stream, unit_wgs, n_pieces, h->row_len,
                         cs.long_len, sums, list_chunks, d_unit, h->hlist_first_slot, sort);
    if (slot_wgs + (unsigned)sort.n_launches > 0)
      hipLaunchKernelGGL(k_row_slot_sums, dim3(slot_wgs + (unsigned)sort.n_launches), dim3(kBuildBlock), 0, stream, slot_wgs, slots,
                         sort);
    if (heavy)
      hipLaunchKernelGGL(k_row_slot_scan, dim3(1), dim3(kOneBlock), 0, stream, slots.sums, (int64_t)s.NB,
                         (int32_t*)(host.base + h_report3));
    StreamShape ss;
    ss.stream = h->stream; ss.compact = h->compact_stream; ss.log2_rb = cs.log2_rb; ss.unit = h->row_val ? 1 : 0;
    ss.phase_width = (int32_t)((int64_t)cs.ppg * s.w > 0x7FFFFFFF ? 0x7FFFFFFF : (int64_t)cs.ppg * s.w);
    if (!with_spmm_plan) ss.stream = nullptr;
    if (s.NB > 0) {
      CopyArgs a;
      a.indptr = csr->indptr; a.indices = csr->indices; a.values = csr->values; a.bound = d_bound; a.piece_of = d_piece_of;
      a.bucket_row_ptr = h->bucket_row_ptr; a.bucket_slot_ptr = h->bucket_slot_ptr; a.rem_ptr = h->rem_ptr;
      a.cols = h->cols; a.vals = h->vals; a.R = h->R; a.S = h->S; a.T = T;
      a.inv_w = 1.0 / (double)(s.w > 0 ? s.w : 1);
      a.dealt = d_dealt; a.unit = d_unit; a.cell_first_chunk = d_cell_chunks; a.group_first_chunk = d_group_tot;
      a.min_deg = min_deg;
      a.heavy_chunk0 = n_chunks; a.heavy_slots = report2[3]; a.n_heavy_chunks = n_heavy_chunks;
      // Entries per workgroup: 512 give a medium graph's grid eight workgroups per CU; large inputs take up to 4096, which
      // share the search and the pieces' data among more entries.  Rows per block: about what those entries belong to.
      a.nnz = csr->nnz;
      a.per_wg = (int32_t)std::min<int64_t>(4096, std::max<int64_t>(512, csr->nnz / 8192 / 512 * 512));
      a.log2_rows = 0;
      while (a.log2_rows < kCopyLog2Rows && ((int64_t)csr->nnz << a.log2_rows) < (int64_t)a.per_wg * s.n_rows) ++a.log2_rows;
      while (a.log2_rows > 0 && ((int64_t)s.c << a.log2_rows) > kCopyPieces) --a.log2_rows;
      const int pieces = (int)std::min<int64_t>((int64_t)s.c << a.log2_rows, kCopyPieces);
      const int64_t n_wg = std::max<int64_t>(1, (csr->nnz + a.per_wg - 1) / a.per_wg);
      CopyCompany with;
      with.n_slots = slot_wgs; with.n_ends = (unsigned)((n_parts + 3) / 4); with.n_sort = sort_wgs;
      with.n_copy = (unsigned)n_wg;
      const int64_t n_company = (int64_t)with.n_slots + with.n_ends + with.n_sort;
      with.n_parts = n_parts; with.queue_len = d_queue_len; with.rb_chunk_ptr = h->rb_chunk_ptr; with.n_chunks = n_chunks;
      with.slots = slots; with.sort = sort;
      if (n_wg + n_company > 0x7FFFFFFF) { st = SPTIR_ERR_OVERFLOW; goto fail; }
      hipLaunchKernelGGL(cs.cut_queues ? k_copy<true> : k_copy<false>, dim3((unsigned)(n_wg + n_company)), dim3(256),
                         sizeof(int) * kCopyWords * (size_t)pieces, stream, s, cs, ss, a, pieces, with);
    }
    BUILD_HIP(hipGetLastError());
    if (n_parts == 0) {  // no lists: the one element of rb_chunk_ptr
      int64_t* zero = (int64_t*)(host.base + h_misc + 16);
      *zero = 0;
      BUILD_HIP(hipMemcpyAsync(h->rb_chunk_ptr, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
    }
    if (n_groups > 0 && !sort_here) {
      st = order_row_blocks(h->rb_chunk_ptr, cs.n_phases, cs.n_rb, max_list_len, h->rb_order, alloc, free_, actx,
                            stream, &tmp_order);
      if (st != SPTIR_OK) goto fail;
    }
    BUILD_HIP(hipStreamSynchronize(stream));
    if (h->n_heavy > 0) {
      const int32_t* report3 = (const int32_t*)(host.base + h_report3);
      h->n_row_slots = report3[0];
      h->n_heavy_rows = report3[1];
    }
    if (opt.release_canonical && with_spmm_plan) {
      // sptir_spmm reads the stream only
      scratch_free(h->blobs[1], free_, actx);
      h->blobs[1] = nullptr;
      h->cols = nullptr; h->vals = nullptr;
      h->device_bytes -= h->canonical_bytes;
      h->canonical_released = 1;
    }
  }
  scratch_free(tmp.base, free_, actx);
  scratch_free(tmp2.base, free_, actx);
  scratch_free(tmp_order, free_, actx);
  spmm_slices_done(&slice_build, free_, actx);
  pinned_pool().release(pinned);
  *out = h;
  return SPTIR_OK;

fail:
  (void)hipStreamSynchronize(stream);
  scratch_free(tmp.base, free_, actx);
  scratch_free(tmp2.base, free_, actx);
  scratch_free(tmp_order, free_, actx);
  spmm_slices_done(&slice_build, free_, actx);
  pinned_pool().release(pinned);
  sptir_hyb_destroy(h);
  return st;
#undef BUILD_HIP
}
