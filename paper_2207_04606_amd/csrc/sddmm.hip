// SDDMM on CSR: B[i,j] = A[i,j] * sum_k X[i,k] * Y[k,j] for the stored (i,j)
// of A (the SDDMM equation of section 4.2 of arXiv 2207.04606).  The paper
// runs SDDMM on plain CSR ("no composable formats"), iterates over the
// non-zeros directly (its sparse_fuse primitive) and reduces in two stages
// with vector loads; the mapping below keeps those three ideas.
//
// Mapping (gfx950, wave64).  The non-zeros are cut into runs of up to 64*kChunks
// consecutive entries, one wavefront each, so the work per wavefront is the
// same whatever the row lengths.  A wavefront takes 64 entries at a time with
// one coalesced load of their columns and values, a chunk ahead.  In CSR order the
// first row of a run is found by a 64-way search and the rows of a chunk by
// counting row starts across the lanes (halving searches and walking indptr took
// longer than the products on small graphs).  Eight lane groups of eight
// lanes then work on eight entries at once (group g on entries 8g .. 8g+7 of
// the 64, one after the other, so that its row changes rarely): lane fl of a group holds floats
// 4*(8t + fl) .. +3 (t = 0..T-1) of the entry's row of X in registers (loaded
// only when the row changes) and gathers the same floats of row j of Yt, one
// 128-byte line per group and load.  Stage one of the reduction is the lane's
// own dot product; stage two is a reduce-scatter over the eight lanes of the
// group, which leaves lane 8g + fl with the result of entry 8g + fl: the 64
// results are in entry order for one coalesced store.
//
// With a plan (sptir_sddmm_plan_build) the entries are visited in column-
// partition order instead of CSR order, the locality argument section 4.2.1
// makes for SpMM applied to SDDMM: the plan lists the entries of partition p
// (rows ascending) as (row, column, CSR position) triples, every XCD is given
// its own partitions, and the workgroups of an XCD sweep them one after the
// other, so an XCD's L2 holds the rows of Yt of one partition at a time.
// There is nothing to accumulate across partitions - an entry's result is
// complete where it is computed - so one launch covers all of them.
// Rows with entries in every slice of columns that fits LDS leave the lists (sddmm_slices.hip).
//
// Measured: CSR order, 169,343 rows, 1.17 M entries: 64 features 97 -> 52 us (50 on the same operands again), 32: 91 -> 27, 128:
// 127 -> 102 (5.8 TB/s of gathered rows, all beyond L2); 41 features, 1.5 M entries 612 -> 47 us; 2,708 rows 42 -> 7 us, most of
// which is the call.  With a plan, 232,965 rows, 114.6 M entries, 128 features: 3.46 ms, with the slices 2.64, with the
// lists read past L2 and X staged 2.46; 20 M entries, 53 features 3.20 -> 0.55 ms.
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "sddmm_lanes.h"
#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

constexpr int kSddmmWaves = 4;
constexpr int kSddmmChunks = 8;  // 64-entry chunks per wavefront
constexpr int kSddmmRun = 64 * kSddmmChunks;

struct SddmmArgs {
  const int32_t* indptr;
  const int32_t* indices;
  const float* values;
  const float* X;   // [n_rows, feat]
  const float* Yt;  // [n_cols, feat]
  float* B;         // [nnz]
  int64_t nnz;
  int32_t n_rows;
  int32_t feat;
  int32_t run;      // CSR order: entries per wavefront
  // with a plan: entries in partition order, and where each XCD's runs start
  const int32_t* e_row;
  const int32_t* e_col;
  const int32_t* e_pos;
  const int64_t* run_first_entry;  // [n_runs]: first entry of every run (at most kSddmmRun entries of one
  const int32_t* run_len;          //           partition, run_len of them), runs grouped by XCD
  const int32_t* xcd_run_ptr;      // [9]: the runs of XCD x are xcd_run_ptr[x] .. xcd_run_ptr[x+1]
};

// The 64 entries of a chunk as the lanes hold them.
struct ChunkEntries {
  int col, row;
  int pos;    // CSR position
  float val;  // CSR order only
};

// Number of the 64 ascending values, one per lane, that are <= v.
__device__ __forceinline__ int count_not_above(int ascending, int v) {
  int n = 0;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n += __shfl(ascending, n + d - 1, 64) <= v ? d : 0;
  return n + (n == 63 && __shfl(ascending, 63, 64) <= v ? 1 : 0);
}

// T float4 per lane cover 32*T floats of a row; wider rows (MANY) are taken 32*T floats at a time.  kWhole: that is the
// row.  kQuads: lanes past its end read nothing.  kTail: feat is no multiple of 4, and the lane that holds the end of
// a row reads the row's last four floats and drops those its neighbour has.  No other load is conditional: behind a branch
// the compiler cannot count the loads in flight, and a wait covers all of them.
// (The second launch bound tells the register allocator how many wavefronts per SIMD to leave room for; left
//  alone it spreads the pipeline stages over 280+ registers although 16*T + 30 are live at any time.)
enum RowEnd { kWhole, kQuads, kTail };
// Where the entries come from: CSR order, a plan, one of few entries (below; four float4 only), or one whose lists the memory-side
// cache does not hold from call to call.  Those are read, and B is written, past the rows of Yt that L2 is to keep (45 M listed
// entries 2636 -> 2560 us; lists that the cache does hold would come from memory every time: 7.9 M entries 70 -> 105 us).
enum Source { kCsr, kPlan, kShortPlan, kLargePlan };
constexpr int64_t kLargeList = 24 << 20;  // entries: 12 bytes each, 256 MB and more
template <int T, Source SOURCE>
constexpr int sddmm_waves() { return T == 4 && (SOURCE == kPlan || SOURCE == kLargePlan) ? 3 : T <= 4 ? 4 : 2; }
// Rows of X a wavefront stages per chunk with a plan.  A chunk of more rows loads them entry by entry: with 16 for four float4 half of
// the chunks of short pieces did (45 M listed entries of 232,965 rows, 128 features, the call: 16 rows 2.56 ms, 20 2.49, 26 2.47, 32,
// which leave room for 8 wavefronts a CU, 2.60).  One float4: none 632, 24 600 us (50 M entries); five: 8 1370, 16 1200 us (25 M).
// Two: none, as 16 to 32 lose up to 15 % where pieces are long.  The 26 rows leave room for three wavefronts a SIMD, which pays where
// gathers miss L2 or the runs are many turns of the GPU.  Elsewhere 16 rows and four wavefronts: 1.9 M entries of 45,461 rows, 128
// features, 102 against 84 us, 4.1 M of 21,584 108 against 95; but 5.9 M of 112,672 rows, 7 MB of Yt a partition, 213 against 252.
// (42 plans of up to 8.4 M entries and 4 MB: 0.96 times as fast with 26 rows, 0.80 to 1.09; 15 of more than 4 MB 1.04, 0.98 to 1.19;
//  30 from 8.4 M entries on 1.09, 0.95 to 1.38.)
template <int T, Source SOURCE>
constexpr int sddmm_staged_rows() {
  return T == 1 ? 24 : T == 2 ? 0 : T == 3 ? 24 : T == 4 && SOURCE != kShortPlan ? 26 : 16;
}
constexpr int64_t kShortList = 8 << 20;       // entries
constexpr int64_t kShortPartBytes = 4 << 20;  // rows of Yt of a partition
template <int T, RowEnd END, bool MANY, Source SOURCE>
__global__ __launch_bounds__(64 * kSddmmWaves, (sddmm_waves<T, SOURCE>())) void k_sddmm(SddmmArgs a) {
  constexpr bool PLAN = SOURCE != kCsr;
  const int lane = threadIdx.x & 63, g = lane >> 3, fl = lane & 7;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int64_t e_begin, e_end;
  if constexpr (PLAN) {
    // consecutive workgroup ids go to consecutive XCDs: workgroup (x + 8*j) is the j-th of XCD x
    const int xcd = blockIdx.x & 7;
    const int64_t run = (int64_t)a.xcd_run_ptr[xcd] + (int64_t)(blockIdx.x >> 3) * kSddmmWaves + wave;
    if (run >= a.xcd_run_ptr[xcd + 1]) return;
    e_begin = a.run_first_entry[run];
    e_end = e_begin + a.run_len[run];
  } else {
    e_begin = ((int64_t)blockIdx.x * kSddmmWaves + wave) * a.run;
    if (e_begin >= a.nnz) return;
    e_end = min(a.nnz, e_begin + a.run);
  }
  const size_t feat = (size_t)a.feat;

  // this lane's floats of a row, from feature f_base on
  auto load_row = [&](const float* row, int f_base, float4 (&v)[T]) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int f = f_base + 32 * t + 4 * fl;
      const int at = END == kWhole ? f : min(f, a.feat - 4);
      if (END == kQuads && (MANY || t == T - 1) && f >= a.feat) {  // (few lanes left: their loads would cost L1 as much)
        v[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        continue;
      }
      const float4u u = *reinterpret_cast<const float4u*>(row + at);
      v[t] = make_float4(u.x, u.y, u.z, u.w);
      if constexpr (END == kTail) {
        const int drop = f - at;  // floats that belong to the lane below (4 and more: all of them)
        if (drop > 0) v[t].x = 0.f;
        if (drop > 1) v[t].y = 0.f;
        if (drop > 2) v[t].z = 0.f;
        if (drop > 3) v[t].w = 0.f;
      }
    }
  };

  auto fetch = [&](int64_t base) {
    ChunkEntries c;
    const int64_t e = min(base + lane, e_end - 1);  // (a lane past the end repeats the last entry)
    if constexpr (PLAN) {
      if constexpr (SOURCE == kLargePlan) {
        c.col = __builtin_nontemporal_load(a.e_col + e);
        c.row = __builtin_nontemporal_load(a.e_row + e);
        c.pos = __builtin_nontemporal_load(a.e_pos + e);
      } else {
        c.col = a.e_col[e]; c.row = a.e_row[e]; c.pos = a.e_pos[e];
      }
      c.val = 0.f;
    } else {
      c.col = a.indices[e]; c.val = a.values[e];
      c.row = 0; c.pos = (int)e;
    }
    return c;
  };
  // CSR order: the starts of the 64 rows after row_lo, the row of a chunk's first entry, say which row each of its
  // entries is in; they are asked for a chunk ahead, and the counting is done while gathers are in flight
  int row_lo = 0, starts = 0;
  auto fetch_starts = [&](int row) { return a.indptr[min(row + 1 + lane, a.n_rows)]; };
  auto find_rows = [&](ChunkEntries& c) {
    if (__builtin_amdgcn_readlane(starts, 0) > __builtin_amdgcn_readlane(c.pos, 63)) {  // still the same row
      c.row = row_lo;
      return;
    }
    bool open = true;
    while (true) {  // (once, unless the chunk touches more than 64 rows)
      const int n = count_not_above(starts, c.pos);
      if (open) c.row = row_lo + n;
      open = open && n == 64;
      if (!__any(open)) break;
      row_lo += 64;
      starts = fetch_starts(row_lo);
    }
    row_lo = __builtin_amdgcn_readlane(c.row, 63);
    starts = fetch_starts(row_lo);
  };
  ChunkEntries next = fetch(e_begin);
  if constexpr (!PLAN) {
    row_lo = row_of_entry(a.indptr, a.n_rows, e_begin, lane);
    starts = fetch_starts(row_lo);
    find_rows(next);
  }

  // The rows of X a chunk needs are staged in LDS once per chunk: every load instruction then brings up to eight
  // different rows (one per lane group), where a reload inside the entry loop costs the address path a whole
  // instruction even if a single lane group asks for it - and in partition order a row lasts only a few entries.
  // (CSR order: no gain, measured.)
  constexpr int kStage = MANY || !PLAN ? 0 : sddmm_staged_rows<T, SOURCE>();
  __shared__ __align__(16) float x_stage[kSddmmWaves][kStage > 0 ? kStage : 1][32 * T];
  __shared__ int row_table[kSddmmWaves][kStage > 0 ? kStage : 1];
  float4 x[T];
  int x_row = -1;
#pragma unroll
  for (int t = 0; t < T; ++t) x[t] = make_float4(0.f, 0.f, 0.f, 0.f);

  for (int64_t base = e_begin; base < e_end; base += 64) {
    ChunkEntries c = next;
    next = fetch(min(base + 64, e_end - 1));  // travels during this chunk
    const bool in = base + lane < e_end;
    if constexpr (PLAN) c.val = a.values[c.pos];
    // Gathers run kAhead entries ahead of the multiplies; the scheduling barriers keep the compiler from
    // hoisting all eight entries' loads to the top (T*8 float4 of registers).
    constexpr int kAhead = T == 4 && (SOURCE == kPlan || SOURCE == kLargePlan) ? 3 : 2;
    float p[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = 0.f;
    for (int f_base = 0; f_base < (MANY ? a.feat : 1); f_base += 32 * T) {
      float4 y[kAhead + 1][T];
      auto issue = [&](int i, float4 (&yb)[T]) {
        const int col = __shfl(c.col, g * 8 + i, 64);  // lane g*8+i fetched this group's i-th entry
        load_row(a.Yt + (size_t)col * feat, f_base, yb);
      };
#pragma unroll
      for (int i = 0; i < kAhead && !PLAN; ++i) issue(i, y[i]);
      if constexpr (!PLAN) {
        if (f_base == 0) find_rows(next);
      }
      bool staged = false;
      int rank_reg = 0, x_rank = -1;
      if constexpr (kStage > 0) {
        // entries arrive row by row: a lane whose row differs from its left neighbour's starts a new row
        const int left = __shfl_up(c.row, 1, 64);
        const bool head = lane == 0 || c.row != left;
        const unsigned long long heads = __ballot(head);
        const int n_distinct = __popcll(heads);
        rank_reg = __popcll(heads & ((2ull << lane) - 1ull)) - 1;  // which of the chunk's rows this lane's entry uses
        staged = n_distinct <= kStage;                             // (wave-uniform)
        if (staged) {
          if (head) row_table[wave][rank_reg] = c.row;
          for (int k0 = 0; k0 < n_distinct; k0 += 8) {
            const int k = k0 + g;
            if (k < n_distinct) {
              float4 v[T];
              load_row(a.X + (size_t)row_table[wave][k] * feat, f_base, v);
#pragma unroll
              for (int t = 0; t < T; ++t) *reinterpret_cast<float4*>(&x_stage[wave][k][32 * t + 4 * fl]) = v[t];
            }
          }
          x_row = -1;  // the registers are about to hold staged rows
        }
      }
#pragma unroll
      for (int i = 0; i < kAhead && PLAN; ++i) issue(i, y[i]);
      if constexpr (MANY) x_row = -1;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (staged) {
          const int rk = __shfl(rank_reg, g * 8 + i, 64);
          if (rk != x_rank) {
#pragma unroll
            for (int t = 0; t < T; ++t) x[t] = *reinterpret_cast<const float4*>(&x_stage[wave][rk][32 * t + 4 * fl]);
            x_rank = rk;
          }
        } else {
          const int r = __shfl(c.row, g * 8 + i, 64);
          if (r != x_row) {
            load_row(a.X + (size_t)r * feat, f_base, x);
            x_row = r;
          }
        }
        if (i + kAhead < 8) issue(i + kAhead, y[(i + kAhead) % (kAhead + 1)]);
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < T; ++t) acc = dot4(x[t], y[i % (kAhead + 1)][t], acc);
        // pin the multiplies here: left free, they are sunk to the use of p[] after the loop and every
        // gathered line stays live (and spills) until then
        asm volatile("" : "+v"(acc));
        p[i] += acc;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // lane (g, fl) ends with the total of p[fl], i.e. of entry base + g*8 + fl = base + lane: its own entry
    const float mine = reduce_scatter8(p, fl);
    if (in) {
      if constexpr (SOURCE == kLargePlan) __builtin_nontemporal_store(c.val * mine, a.B + c.pos);
      else a.B[c.pos] = c.val * mine;
    }
  }
}

// fewer than four features: a lane per entry
template <bool PLAN>
__global__ __launch_bounds__(256) void k_sddmm_narrow(SddmmArgs a) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t wave_first = e & ~(int64_t)63;
  if (wave_first >= a.nnz) return;
  const int64_t at = min(e, a.nnz - 1);
  int row, col;
  int64_t pos;
  if constexpr (PLAN) {
    row = a.e_row[at]; col = a.e_col[at]; pos = a.e_pos[at];
  } else {
    row = row_of_entry(a.indptr, a.n_rows, wave_first, (int)(threadIdx.x & 63));
    while (row + 1 < a.n_rows && at >= (int64_t)a.indptr[row + 1]) ++row;
    col = a.indices[at]; pos = at;
  }
  float acc = 0.f;
  for (int f = 0; f < a.feat; ++f) acc = fmaf(a.X[(size_t)row * a.feat + f], a.Yt[(size_t)col * a.feat + f], acc);
  if (e < a.nnz) a.B[pos] = a.values[pos] * acc;
}

template <Source SOURCE, int T>
void launch_stripes(const SddmmArgs& a, dim3 grid, hipStream_t stream) {
  const dim3 block(64 * kSddmmWaves);
  if (a.feat == 32 * T) hipLaunchKernelGGL((k_sddmm<T, kWhole, false, SOURCE>), grid, block, 0, stream, a);
  else if (a.feat % 4 == 0) hipLaunchKernelGGL((k_sddmm<T, kQuads, false, SOURCE>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((k_sddmm<T, kTail, false, SOURCE>), grid, block, 0, stream, a);
}

// grid: the workgroups of k_sddmm
template <Source SOURCE>
void launch_sddmm(const SddmmArgs& a, dim3 grid, hipStream_t stream) {
  const dim3 block(64 * kSddmmWaves);
  if (a.feat < 4) {
    hipLaunchKernelGGL(k_sddmm_narrow<SOURCE != kCsr>, dim3((unsigned)((a.nnz + 255) / 256)), dim3(256), 0, stream, a);
    return;
  }
  switch ((a.feat + 31) / 32) {
    case 1: return launch_stripes<SOURCE, 1>(a, grid, stream);
    case 2: return launch_stripes<SOURCE, 2>(a, grid, stream);
    case 3: return launch_stripes<SOURCE, 3>(a, grid, stream);
    case 4: return launch_stripes<SOURCE, 4>(a, grid, stream);
    case 5: return launch_stripes<SOURCE, 5>(a, grid, stream);
    case 6: return launch_stripes<SOURCE, 6>(a, grid, stream);
    case 7: return launch_stripes<SOURCE, 7>(a, grid, stream);
    case 8: return launch_stripes<SOURCE, 8>(a, grid, stream);
    default:
      if (a.feat % 4) hipLaunchKernelGGL((k_sddmm<8, kTail, true, SOURCE>), grid, block, 0, stream, a);
      else hipLaunchKernelGGL((k_sddmm<8, kQuads, true, SOURCE>), grid, block, 0, stream, a);
  }
}

// Entries per wavefront in CSR order: short runs while there are few entries, so that every CU has 16 wavefronts; six times as many,
// whose last ones leave less of the GPU idle, where what an entry costs is large against finding a run's first row: more than 32
// features, and gathers that miss L2 or rows of more than 64.  (60 graphs of more than 32 features: three times as many 1.026 times as
// fast, six times 1.030, twelve times 1.033, 0.92 to 1.18; 33 to 64 features out of L2 0.88 to 0.97, up to 32 features 0.85 to 1.07.)
int32_t csr_run(int64_t nnz, int32_t feat, int32_t n_cols) {
  const bool costly = feat > 64 || (feat > 32 && (int64_t)n_cols * feat >= (int64_t)1 << 21);
  const int64_t chunks = nnz / (64 * (costly ? 24576 : 4096));
  return 64 * (int32_t)std::min<int64_t>(kSddmmChunks, std::max<int64_t>(1, chunks));
}

// ------------------------------------------------------------------- plan
// lens[p * n_rows + r] = entries of row r in column partition p; none where the slices have the row (rank, may be NULL, goes up)
__global__ void k_piece_lengths(int32_t n_rows, int32_t c, int32_t w, const int32_t* __restrict__ indptr,
                                const int32_t* __restrict__ indices, const int32_t* __restrict__ rank, int32_t* lens) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)n_rows * c) return;
  int r = (int)(t % n_rows), p = (int)(t / n_rows);
  if (rank && rank[r + 1] > rank[r]) {
    lens[t] = 0;
    return;
  }
  int a = indptr[r], b = indptr[r + 1];
  int first = (p == 0) ? a : lower_bound_col(indices, a, b, (int64_t)p * w);
  int last = (p == c - 1) ? b : lower_bound_col(indices, first, b, (int64_t)(p + 1) * w);
  lens[t] = last - first;
}

// Copies every (row, partition) piece to its place in the partition-ordered entry list:
// offs[p * n_rows + r] is the piece's offset inside partition p, part_first[p] the partition's first entry.
__global__ void k_scatter_entries(int32_t n_rows, int32_t c, int32_t w, const int32_t* __restrict__ indptr,
                                  const int32_t* __restrict__ indices, const int32_t* __restrict__ rank,
                                  const int32_t* __restrict__ offs, const int64_t* __restrict__ part_first, int32_t* e_row,
                                  int32_t* e_col, int32_t* e_pos) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)n_rows * c) return;
  int r = (int)(t % n_rows), p = (int)(t / n_rows);
  if (rank && rank[r + 1] > rank[r]) return;
  int a = indptr[r], b = indptr[r + 1];
  int first = (p == 0) ? a : lower_bound_col(indices, a, b, (int64_t)p * w);
  int last = (p == c - 1) ? b : lower_bound_col(indices, first, b, (int64_t)(p + 1) * w);
  int64_t dst = part_first[p] + offs[t];
  for (int q = first; q < last; ++q, ++dst) {
    e_row[dst] = r;
    e_col[dst] = indices[q];
    e_pos[dst] = q;
  }
}

bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb) {
  uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return na && nb && a0 < b0 + nb && b0 < a0 + na;
}

}  // namespace
}  // namespace sptir

// The handle behind sptir_sddmm_plan_t.
struct sptir_sddmm_plan {
  int32_t n_rows, n_cols, c, w;
  int64_t nnz;
  // otherwise: the long rows in column slices, the entries of the others in partition order and the runs of every XCD
  sptir::SddmmSlices slices;
  int32_t *e_row, *e_col, *e_pos;
  int64_t* run_first_entry;
  int32_t* run_len;
  int32_t* xcd_run_ptr;
  int64_t n_runs;
  int64_t max_runs_per_xcd;
  // c == 1 and no long rows: entries stay in CSR order; the plan keeps its own copy of the structure
  int32_t *indptr, *indices;
  size_t device_bytes;
  sptir_alloc_fn alloc;
  sptir_free_fn free_;
  void* alloc_ctx;
};

using namespace sptir;

extern "C" sptir_status_t sptir_sddmm_plan_destroy(sptir_sddmm_plan_t* p) {
  if (!p) return SPTIR_OK;
  void* ptrs[] = {p->e_row, p->e_col, p->e_pos, p->run_first_entry, p->run_len, p->xcd_run_ptr, p->indptr, p->indices};
  for (void* q : ptrs)
    if (q) p->free_(q, p->alloc_ctx);
  sddmm_slices_free(&p->slices, p->free_, p->alloc_ctx);
  delete p;
  return SPTIR_OK;
}

extern "C" sptir_status_t sptir_sddmm_plan_info(const sptir_sddmm_plan_t* p, sptir_sddmm_plan_info_t* out) {
  if (!p || !out) return SPTIR_ERR_INVALID_ARG;
  sptir_sddmm_plan_info_t o;
  o.n_rows = p->n_rows; o.n_cols = p->n_cols; o.n_col_parts = p->c; o.part_width = p->w;
  o.nnz = p->nnz; o.n_runs = p->n_runs; o.device_bytes = (int64_t)p->device_bytes;
  *out = o;
  return SPTIR_OK;
}

extern "C" int32_t sptir_sddmm_default_col_parts(int32_t n_rows, int32_t n_cols, int64_t nnz, int32_t feat_hint) {
  // The rows of Yt of one partition should fit an XCD's L2 next to the rest of the traffic (2.5 of 4 MB); every
  // (row, partition) piece re-reads its row of X, so a piece should hold a few entries; every XCD wants its
  // own partitions, so c is a multiple of 8 - or 1, which leaves the entries in CSR order.
  if (n_rows <= 0 || n_cols <= 0 || nnz <= 0) return 1;
  const int64_t feat = feat_hint > 0 ? feat_hint : 128;
  const int64_t w_fit = std::max<int64_t>(1, (int64_t)(2.5 * 1024 * 1024) / (feat * 4));
  int64_t want = (n_cols + w_fit - 1) / w_fit;
  const int64_t by_piece = nnz / ((int64_t)n_rows * 4);
  // (to the nearest multiple of 8, as far as the pieces allow: measured, 7 wanted runs best with 8, 12 with 8)
  want = std::min((want + 3) / 8 * 8, by_piece / 8 * 8);
  return (want >= 8 && n_cols > w_fit) ? (int32_t)std::min<int64_t>(want, 1024) : 1;
}

extern "C" sptir_status_t sptir_sddmm_plan_build(const sptir_csr_t* csr, int32_t n_col_parts, int32_t feat_hint,
                                                 void* stream_, sptir_sddmm_plan_t** out) {
  if (!csr || !out || n_col_parts < 0 || feat_hint < 0) return SPTIR_ERR_INVALID_ARG;
  if (csr->n_rows < 0 || csr->n_cols < 0 || csr->nnz < 0) return SPTIR_ERR_INVALID_ARG;
  if (csr->nnz >= ((int64_t)1 << 31)) return SPTIR_ERR_OVERFLOW;
  if (!csr->indptr || (csr->nnz > 0 && !csr->indices)) return SPTIR_ERR_INVALID_ARG;
  if (csr->nnz > 0 && (csr->n_rows == 0 || csr->n_cols == 0)) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;
  const int32_t n_rows = csr->n_rows, n_cols = csr->n_cols;
  const int64_t nnz = csr->nnz;

  // ---- number of column partitions
  int32_t c = n_col_parts > 0 ? n_col_parts : sptir_sddmm_default_col_parts(n_rows, n_cols, nnz, feat_hint);
  if (c > std::max(n_cols, 1)) c = std::max(n_cols, 1);
  if ((int64_t)n_rows * c > ((int64_t)1 << 36)) return SPTIR_ERR_OVERFLOW;

  sptir_sddmm_plan* p = new (std::nothrow) sptir_sddmm_plan();
  if (!p) return SPTIR_ERR_ALLOC;
  current_allocator(&p->alloc, &p->free_, &p->alloc_ctx);
  p->n_rows = n_rows; p->n_cols = n_cols; p->c = c; p->nnz = nnz;
  p->w = (int32_t)(((int64_t)n_cols + c - 1) / c);
  sptir_alloc_fn alloc = p->alloc; sptir_free_fn free_ = p->free_; void* actx = p->alloc_ctx;
  int32_t* rank = nullptr;
  int32_t* lens = nullptr;
  int32_t* d_totals = nullptr;
  int64_t* d_part_first = nullptr;
  sptir_status_t st = SPTIR_OK;
  auto take = [&](void** dst, size_t bytes) {
    *dst = alloc(bytes ? bytes : 16, actx, stream);
    if (*dst) p->device_bytes += bytes ? bytes : 16;
    return *dst != nullptr;
  };
#define PLAN_HIP(call)                                                 \
  do {                                                                 \
    hipError_t e_ = (call);                                            \
    if (e_ != hipSuccess) { st = note_hip_error(e_, #call); goto fail; } \
  } while (0)

  st = sddmm_slices_build(csr, feat_hint, alloc, free_, actx, stream, &p->slices, &rank);
  if (st != SPTIR_OK) goto fail;
  p->device_bytes += p->slices.device_bytes;
  if (nnz == 0 || (c == 1 && p->slices.n_units == 0)) {
    p->c = 1; p->w = n_cols;
    if (!take((void**)&p->indptr, sizeof(int32_t) * ((size_t)n_rows + 1)) ||
        !take((void**)&p->indices, sizeof(int32_t) * (size_t)nnz)) { st = SPTIR_ERR_ALLOC; goto fail; }
    PLAN_HIP(hipMemcpyAsync(p->indptr, csr->indptr, sizeof(int32_t) * ((size_t)n_rows + 1), hipMemcpyDeviceToDevice,
                            stream));
    if (nnz > 0)
      PLAN_HIP(hipMemcpyAsync(p->indices, csr->indices, sizeof(int32_t) * (size_t)nnz, hipMemcpyDeviceToDevice,
                              stream));
    PLAN_HIP(hipStreamSynchronize(stream));
    *out = p;
    return SPTIR_OK;
  }
  {
    const int64_t n_pairs = (int64_t)n_rows * c, n_listed = nnz - p->slices.nnz;
    lens = (int32_t*)alloc(sizeof(int32_t) * (size_t)n_pairs, actx, stream);
    d_totals = (int32_t*)alloc(sizeof(int32_t) * (size_t)c, actx, stream);
    d_part_first = (int64_t*)alloc(sizeof(int64_t) * (size_t)c, actx, stream);
    if (!lens || !d_totals || !d_part_first) { st = SPTIR_ERR_ALLOC; goto fail; }
    const unsigned pair_blocks = (unsigned)((n_pairs + 255) / 256);
    hipLaunchKernelGGL(k_piece_lengths, dim3(pair_blocks), dim3(256), 0, stream, n_rows, c, p->w, csr->indptr,
                       csr->indices, rank, lens);
    hipLaunchKernelGGL(k_scan_sequences<int32_t>, dim3((unsigned)c), dim3(kBuildBlock), 0, stream, lens, n_rows,
                       d_totals);
    PLAN_HIP(hipGetLastError());
    std::vector<int32_t> totals((size_t)c);
    PLAN_HIP(hipMemcpyAsync(totals.data(), d_totals, sizeof(int32_t) * (size_t)c, hipMemcpyDeviceToHost, stream));
    PLAN_HIP(hipStreamSynchronize(stream));
    std::vector<int64_t> part_first((size_t)c + 1, 0);
    for (int32_t q = 0; q < c; ++q) {
      if (totals[q] < 0) { st = SPTIR_ERR_UNSORTED; goto fail; }
      part_first[q + 1] = part_first[q] + totals[q];
    }
    // the pieces tile every row exactly when its columns ascend; anything else would not fit the arrays below
    if (part_first[c] != n_listed) { st = SPTIR_ERR_UNSORTED; goto fail; }
    if (!take((void**)&p->e_row, sizeof(int32_t) * (size_t)n_listed) ||
        !take((void**)&p->e_col, sizeof(int32_t) * (size_t)n_listed) ||
        !take((void**)&p->e_pos, sizeof(int32_t) * (size_t)n_listed)) { st = SPTIR_ERR_ALLOC; goto fail; }
    PLAN_HIP(hipMemcpyAsync(d_part_first, part_first.data(), sizeof(int64_t) * (size_t)c, hipMemcpyHostToDevice,
                            stream));
    hipLaunchKernelGGL(k_scatter_entries, dim3(pair_blocks), dim3(256), 0, stream, n_rows, c, p->w, csr->indptr,
                       csr->indices, rank, lens, d_part_first, p->e_row, p->e_col, p->e_pos);
    PLAN_HIP(hipGetLastError());

    // ---- partitions to XCDs (largest first onto the least loaded), runs of every XCD in partition order
    std::vector<int32_t> order((size_t)c);
    for (int32_t q = 0; q < c; ++q) order[q] = q;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return totals[x] > totals[y]; });
    int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    std::vector<int32_t> of_xcd[8];
    for (int32_t q : order) {
      int best = 0;
      for (int x = 1; x < 8; ++x)
        if (load[x] < load[best]) best = x;
      load[best] += totals[q];
      of_xcd[best].push_back(q);
    }
    std::vector<int64_t> run_first;
    std::vector<int32_t> run_len;
    int32_t xcd_run_ptr[9];
    int64_t max_runs = 0;
    for (int x = 0; x < 8; ++x) {
      xcd_run_ptr[x] = (int32_t)run_first.size();
      auto runs_of = [&](int64_t begin, int64_t end) {
        for (int64_t at = begin; at < end; at += kSddmmRun) {
          run_first.push_back(at);
          run_len.push_back((int32_t)std::min<int64_t>(kSddmmRun, end - at));
        }
      };
      if (c == 1) {  // one partition: an eighth of its entries each
        runs_of(n_listed * x / 8, n_listed * (x + 1) / 8);
      } else {
        std::sort(of_xcd[x].begin(), of_xcd[x].end());
        for (int32_t q : of_xcd[x]) runs_of(part_first[q], part_first[q + 1]);
      }
      max_runs = std::max<int64_t>(max_runs, (int64_t)run_first.size() - xcd_run_ptr[x]);
    }
    xcd_run_ptr[8] = (int32_t)run_first.size();
    p->n_runs = (int64_t)run_first.size();
    p->max_runs_per_xcd = max_runs;
    if (!take((void**)&p->run_first_entry, sizeof(int64_t) * run_first.size()) ||
        !take((void**)&p->run_len, sizeof(int32_t) * run_len.size()) ||
        !take((void**)&p->xcd_run_ptr, sizeof(xcd_run_ptr))) { st = SPTIR_ERR_ALLOC; goto fail; }
    PLAN_HIP(hipMemcpyAsync(p->run_first_entry, run_first.data(), sizeof(int64_t) * run_first.size(),
                            hipMemcpyHostToDevice, stream));
    PLAN_HIP(hipMemcpyAsync(p->run_len, run_len.data(), sizeof(int32_t) * run_len.size(), hipMemcpyHostToDevice,
                            stream));
    PLAN_HIP(hipMemcpyAsync(p->xcd_run_ptr, xcd_run_ptr, sizeof(xcd_run_ptr), hipMemcpyHostToDevice, stream));
    PLAN_HIP(hipStreamSynchronize(stream));  // the host vectors go out of scope
  }
  free_(lens, actx); free_(d_totals, actx); free_(d_part_first, actx);
  if (rank) free_(rank, actx);
  *out = p;
  return SPTIR_OK;

fail:
  (void)hipStreamSynchronize(stream);
  if (rank) free_(rank, actx);
  if (lens) free_(lens, actx);
  if (d_totals) free_(d_totals, actx);
  if (d_part_first) free_(d_part_first, actx);
  sptir_sddmm_plan_destroy(p);
  return st;
#undef PLAN_HIP
}

extern "C" sptir_status_t sptir_sddmm(const sptir_sddmm_plan_t* p, const float* values, const float* X,
                                      const float* Yt, float* B_values, int32_t feat, void* stream_) {
  if (!p || feat < 1) return SPTIR_ERR_INVALID_ARG;
  if (p->nnz == 0) return SPTIR_OK;
  if (!values || !X || !Yt || !B_values) return SPTIR_ERR_INVALID_ARG;
  const size_t b_bytes = sizeof(float) * (size_t)p->nnz;
  if (ranges_overlap(B_values, b_bytes, X, sizeof(float) * (size_t)p->n_rows * feat) ||
      ranges_overlap(B_values, b_bytes, Yt, sizeof(float) * (size_t)p->n_cols * feat))
    return SPTIR_ERR_INVALID_ARG;
  if (B_values != values && ranges_overlap(B_values, b_bytes, values, b_bytes)) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;
  SddmmArgs a;
  a.indptr = p->indptr; a.indices = p->indices; a.values = values;
  a.X = X; a.Yt = Yt; a.B = B_values; a.nnz = p->nnz; a.n_rows = p->n_rows; a.feat = feat;
  a.e_row = p->e_row; a.e_col = p->e_col; a.e_pos = p->e_pos;
  a.run_first_entry = p->run_first_entry; a.run_len = p->run_len; a.xcd_run_ptr = p->xcd_run_ptr;
  a.run = csr_run(p->nnz, feat, p->n_cols);
  if (p->indptr) {
    const int64_t runs = (p->nnz + a.run - 1) / a.run;
    launch_sddmm<kCsr>(a, dim3((unsigned)((runs + kSddmmWaves - 1) / kSddmmWaves)), stream);
  } else {
    if (p->slices.n_units > 0) {
      const sptir_status_t st = sddmm_slices_run(p->slices, p->n_cols, values, X, Yt, B_values, feat, stream);
      if (st != SPTIR_OK) return st;
    }
    a.nnz = p->nnz - p->slices.nnz;
    if (a.nnz == 0) return SPTIR_OK;
    const dim3 grid((unsigned)(8 * ((p->max_runs_per_xcd + kSddmmWaves - 1) / kSddmmWaves)));
    const bool short_list = a.nnz < kShortList && (int64_t)p->w * feat * (int64_t)sizeof(float) <= kShortPartBytes;
    if (a.nnz >= kLargeList) launch_sddmm<kLargePlan>(a, grid, stream);
    else if (short_list && feat > 96 && feat <= 128) launch_stripes<kShortPlan, 4>(a, grid, stream);
    else launch_sddmm<kPlan>(a, grid, stream);
  }
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

extern "C" sptir_status_t sptir_sddmm_csr(const sptir_csr_t* csr, const float* X, const float* Yt, float* B_values,
                                          int32_t feat, void* stream_) {
  if (!csr || feat < 1 || csr->n_rows < 0 || csr->n_cols < 0 || csr->nnz < 0) return SPTIR_ERR_INVALID_ARG;
  if (csr->nnz >= ((int64_t)1 << 31)) return SPTIR_ERR_OVERFLOW;
  if (csr->nnz == 0) return SPTIR_OK;
  if (!csr->indptr || !csr->indices || !csr->values || !X || !Yt || !B_values) return SPTIR_ERR_INVALID_ARG;
  if (csr->n_rows == 0 || csr->n_cols == 0) return SPTIR_ERR_INVALID_ARG;
  const size_t b_bytes = sizeof(float) * (size_t)csr->nnz;
  if (ranges_overlap(B_values, b_bytes, X, sizeof(float) * (size_t)csr->n_rows * feat) ||
      ranges_overlap(B_values, b_bytes, Yt, sizeof(float) * (size_t)csr->n_cols * feat) ||
      ranges_overlap(B_values, b_bytes, csr->indices, sizeof(int32_t) * (size_t)csr->nnz) ||
      ranges_overlap(B_values, b_bytes, csr->indptr, sizeof(int32_t) * ((size_t)csr->n_rows + 1)))
    return SPTIR_ERR_INVALID_ARG;
  SddmmArgs a;
  a.indptr = csr->indptr; a.indices = csr->indices; a.values = csr->values;
  a.X = X; a.Yt = Yt; a.B = B_values; a.nnz = csr->nnz; a.n_rows = csr->n_rows; a.feat = feat;
  a.run = csr_run(csr->nnz, feat, csr->n_cols);
  const int64_t runs = (csr->nnz + a.run - 1) / a.run;
  dim3 grid((unsigned)((runs + kSddmmWaves - 1) / kSddmmWaves));
  hipStream_t stream = (hipStream_t)stream_;
  a.e_row = a.e_col = a.e_pos = nullptr; a.run_first_entry = nullptr; a.run_len = nullptr; a.xcd_run_ptr = nullptr;
  launch_sddmm<kCsr>(a, grid, stream);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}
