// SDDMM of the long rows of a plan, from column slices in LDS.
//
// A column of A costs its row of Yt once per entry, and through L1 no more than 32 TB/s of them arrive whatever the caches
// hold (40 at 64 bytes a cycle and CU).  LDS delivers twice that and more: random 128-byte rows at 76, random 512-byte rows
// at 77 TB/s (125 bytes a cycle and CU).  Where rows are so long that each has entries in every slice of columns that
// fits LDS, a workgroup loads the slice's rows of Yt once and takes all of its entries from there.
//
// Mapping.  `width` columns make a slice: as many rows of Yt as kSliceBytes hold.  The entries of a (row, slice) pair are
// consecutive in CSR order; they are cut into segments of up to eight, and the segments of a slice are sorted by their number
// of entries, the full ones first, so that the eight lane groups of a wavefront, a segment each, end together.  Lane fl of a
// group holds floats 4*(8t + fl) .. +3 of the segment's row of X, reads the same floats of an entry's column from LDS, and
// the eight partial sums of a lane meet as in k_sddmm: the products of an entry, and their order, are those of the other
// kernels, so its result is the same bit for bit.  Rows of X come from L2, one per segment (an eighth of the bytes of the entries).
// A unit of work is a slice and a range of the long rows, or a piece of what they have; units go by range of rows first, so that the rows of X
// that an XCD's workgroups want at a time stay in its L2, and by neighbouring slices inside an XCD, so that the lines of values
// and results that pieces share do.
// 232,965 rows, 114.6 M entries, 128 features: 70 M entries in 0.78 ms (11.1 ps an entry, 30 in k_sddmm): 46 TB/s of gathered
// rows where LDS gives 85, vector ALU issuing 54 % of it, bank conflicts 24 %; segments not kept apart by range of rows 1.20 ms, slices dealt to the XCDs in turn 1.04 (twice the misses).
#include <algorithm>
#include <new>
#include <vector>

#include "sddmm_lanes.h"
#include "sddmm_slice_shape.h"
#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_slice_bounds.h"
#include "sptir_tiles.h"

namespace sptir {
namespace {

// Rows are long from kMinPiece entries per slice on.  232,965 rows, 114.6 M entries, the call: 2 2645 us, 3 2636, 5 2695, none 3464.
constexpr int64_t kMinPiece = 3;
constexpr int64_t kMinUnits = 2048;
constexpr int64_t kPartBytes = 1 << 20;  // rows of X of a part (2 MB: 1 % slower)
constexpr int64_t kCus = 256;
constexpr int64_t kMinUnitNnz = 4096;    // entries that pay for loading a slice
constexpr int kSegment = 8;             // entries of a segment
constexpr int kClasses = 8;             // full segments, then those of 7 .. 1 entries

struct SliceArgs {
  const int4* units;       // SliceUnit
  const int2* seg_at;      // row, CSR position of the first entry
  const uint4* seg_cols;   // eight 16-bit columns inside the slice (the last one repeated); bits 13 .. 15 of the first: entries - 1
  const float* values;
  const float* X;
  const float* Yt;
  float* B;
  int32_t feat, quads;     // quads: float4 per row, the last one partly used where feat is no multiple of 4
  int32_t stride;          // float4 from one row to the next in LDS
  int32_t width, n_cols;
};

// quad q of a row as lanes of the other kernels hold it: the last one of a row whose length is no multiple of 4 is read
// from the row's last four floats, those of the quad before it dropped
__device__ __forceinline__ float4 load_quad(const float* row, int q, int feat) {
  const int f = 4 * q, at = min(f, feat - 4);
  const float4u u = *reinterpret_cast<const float4u*>(row + at);
  float4 v = make_float4(u.x, u.y, u.z, u.w);
  const int drop = f - at;
  if (drop > 0) v.x = 0.f;
  if (drop > 1) v.y = 0.f;
  if (drop > 2) v.z = 0.f;
  if (drop > 3) v.w = 0.f;
  return v;
}

__device__ __forceinline__ int column_of(const uint4& c, int u) {
  const unsigned w = u < 2 ? c.x : (u < 4 ? c.y : (u < 6 ? c.z : c.w));
  return (int)((u & 1) ? w >> 16 : w & 0xFFFFu);
}

template <int T> constexpr int slice_threads() { return T <= 4 ? 1024 : 512; }

// T float4 per lane cover a row of at most 32 T floats; TAIL: it is shorter.
template <int T, bool TAIL>
__global__ __launch_bounds__(slice_threads<T>()) void k_sddmm_slices(SliceArgs a) {
  constexpr int kThreads = slice_threads<T>(), kGroups = kThreads / 8;
  extern __shared__ __align__(16) float4 y[];  // [width][stride], then a quad of zeros
  const int lane = threadIdx.x & 63, g = lane >> 3, fl = lane & 7;
  const int4 unit = a.units[blockIdx.x];
  if (unit.y == unit.z) return;
  const int quads = TAIL ? a.quads : 8 * T, stride = TAIL ? a.stride : slice_stride(8 * T);
  const int64_t col0 = (int64_t)unit.x * a.width;
  {
    const int n = (int)min((int64_t)a.width, (int64_t)a.n_cols - col0) * quads;
    const float* src = a.Yt + (size_t)col0 * a.feat;
    constexpr int kAtOnce = 8;
    for (int i0 = threadIdx.x; i0 < n; i0 += kAtOnce * kThreads) {
      float4 v[kAtOnce];
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const int i = min(i0 + k * kThreads, n - 1);
        if (!TAIL || (a.feat & 3) == 0) {
          const float4u u = *reinterpret_cast<const float4u*>(src + 4 * (size_t)i);
          v[k] = make_float4(u.x, u.y, u.z, u.w);
        } else {
          const int c = i / quads;
          v[k] = load_quad(src + (size_t)c * a.feat, i - c * quads, a.feat);
        }
      }
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const int i = i0 + k * kThreads, c = i / quads;
        if (i < n) y[c * stride + (i - c * quads)] = v[k];
      }
    }
    if (TAIL && threadIdx.x == 0) y[a.width * stride] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();

  // where this lane's last float4 of a column sits; a lane past the end of a row reads zeros
  const bool ends = TAIL && 8 * (T - 1) + fl >= quads;
  const int last_step = ends ? 0 : stride, last_at = ends ? a.width * stride : 8 * (T - 1) + fl;
  auto load_x = [&](int row, float4 (&v)[T]) {
    const float* p = a.X + (size_t)row * a.feat;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (TAIL) {
        if (t == T - 1 && ends) v[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        else v[t] = load_quad(p, 8 * t + fl, a.feat);
      } else {
        const float4u u = *reinterpret_cast<const float4u*>(p + 4 * (8 * t + fl));
        v[t] = make_float4(u.x, u.y, u.z, u.w);
      }
    }
  };
  const int first = unit.y + (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 8;
  if (first >= unit.z) return;
  // The row of X of a segment is asked for while the one before it is worked on, where a segment is, one before that.
  struct Segment {
    int2 at;
    uint4 cols;
  };
  auto segment = [&](int base) {
    const int i = min(base + g, unit.z - 1);
    return Segment{a.seg_at[i], a.seg_cols[i]};
  };
  auto work = [&](int base, const Segment& seg, const float4 (&x)[T]) {
    const int n = (int)(seg.cols.x >> kColumnBits & 7u) + 1;
    const int n_most = __builtin_amdgcn_readfirstlane(n);  // (sorted: the first group has the longest segment)
    uint4 cols = seg.cols;
    cols.x &= ~(7u << kColumnBits);
    const bool in = base + g < unit.z && fl < n;
    const float value = in ? a.values[seg.at.y + fl] : 0.f;
    auto product = [&](int u) {
      const int c = column_of(cols, u);
      const float4* row = y + c * stride + fl;
      float acc = 0.f;
#pragma unroll
      for (int t = 0; t < T; ++t) acc = dot4(x[t], TAIL && t == T - 1 ? y[c * last_step + last_at] : row[8 * t], acc);
      return acc;
    };
    float p[8];
    if (n_most == kSegment) {
#pragma unroll
      for (int u = 0; u < kSegment; ++u) p[u] = product(u);
    } else {
#pragma unroll
      for (int u = 0; u < kSegment; ++u) {
        p[u] = 0.f;
        if (u < n_most) p[u] = product(u);
      }
    }
    const float mine = reduce_scatter8(p, fl);
    if (in) a.B[seg.at.y + fl] = value * mine;
  };
  Segment s0 = segment(first), s1 = segment(first + kGroups);
  float4 x0[T], x1[T];
  load_x(s0.at.x, x0);
  for (int base = first;; base += 2 * kGroups) {
    load_x(s1.at.x, x1);
    const Segment s2 = segment(base + 2 * kGroups);
    work(base, s0, x0);
    if (base + kGroups >= unit.z) break;
    load_x(s2.at.x, x0);
    const Segment s3 = segment(base + 3 * kGroups);
    work(base + kGroups, s1, x1);
    if (base + 2 * kGroups >= unit.z) break;
    s0 = s2; s1 = s3;
  }
}

// The same segments for the calls that slice_lane_quads() gives no LDS kernel: rows of Yt from memory, 256 features at a time.
__global__ __launch_bounds__(512) void k_sddmm_segments(SliceArgs a) {
  constexpr int T = 8, kGroups = 64;
  const int lane = threadIdx.x & 63, g = lane >> 3, fl = lane & 7;
  const int4 unit = a.units[blockIdx.x];
  const int first = unit.y + (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 8;
  const float* slice = a.Yt + (size_t)unit.x * a.width * a.feat;
  for (int base = first; base < unit.z; base += kGroups) {
    const int seg = min(base + g, unit.z - 1);
    const int2 at = a.seg_at[seg];
    uint4 cols = a.seg_cols[seg];
    const int n = (int)(cols.x >> kColumnBits & 7u) + 1;
    cols.x &= ~(7u << kColumnBits);
    const bool in = base + g < unit.z && fl < n;
    const float* xr = a.X + (size_t)at.x * a.feat;
    float mine = 0.f;
    if (a.feat < 4) {  // a lane per entry
      int c = 0;
#pragma unroll
      for (int u = 0; u < kSegment; ++u) c = fl == u ? column_of(cols, u) : c;
      for (int f = 0; f < a.feat; ++f) mine = fmaf(xr[f], slice[(size_t)c * a.feat + f], mine);
    } else {
      float p[8];
#pragma unroll
      for (int u = 0; u < kSegment; ++u) p[u] = 0.f;
      for (int q0 = 0; q0 < a.quads; q0 += 8 * T) {
        auto load = [&](const float* row, float4 (&v)[T]) {
#pragma unroll
          for (int t = 0; t < T; ++t) {
            const int q = q0 + 8 * t + fl;
            v[t] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (q < a.quads) v[t] = load_quad(row, q, a.feat);
          }
        };
        float4 x[T];
        load(xr, x);
#pragma unroll
        for (int u = 0; u < kSegment; ++u) {
          float4 v[T];
          load(slice + (size_t)column_of(cols, u) * a.feat, v);
          float acc = 0.f;
#pragma unroll
          for (int t = 0; t < T; ++t) acc = dot4(x[t], v[t], acc);
          asm volatile("" : "+v"(acc));  // (or the rows of all eight entries are loaded first, into 256 registers)
          p[u] += acc;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      mine = reduce_scatter8(p, fl);
    }
    if (in) a.B[at.y + fl] = a.values[at.y + fl] * mine;
  }
}

// ------------------------------------------------------------------- build
// taken[r]: 1 where row r is long enough (taken[n_rows] = 0); *entries: their entries together
__global__ __launch_bounds__(kBuildBlock) void k_long_rows(int32_t n_rows, int64_t nnz, const int32_t* __restrict__ indptr,
                                                           int64_t min_deg, int32_t* taken, unsigned long long* entries) {
  __shared__ long long wave_sums[kWaves];
  const int64_t r = (int64_t)blockIdx.x * kBuildBlock + threadIdx.x;
  const long long begin = r < n_rows ? indptr[r] : 0, end = r < n_rows ? indptr[r + 1] : 0;
  const bool is_long = r < n_rows && is_long_row(begin, end, nnz, min_deg);
  if (r <= n_rows) taken[r] = is_long ? 1 : 0;
  long long sum;
  (void)block_exclusive_scan<long long>(is_long ? end - begin : 0, wave_sums, &sum);
  if (threadIdx.x == 0 && sum > 0) atomicAdd(entries, (unsigned long long)sum);
}

__global__ __launch_bounds__(kBuildBlock) void k_list_long_rows(int32_t n_rows, const int32_t* __restrict__ rank, int32_t* rows) {
  const int64_t r = (int64_t)blockIdx.x * kBuildBlock + threadIdx.x;
  if (r < n_rows && rank[r + 1] > rank[r]) rows[rank[r]] = (int32_t)r;
}

// Unit u = part * n_slices + slice: the segments that rows part * part_rows .. of the long rows have in the slice.
// counts[u * kClasses + k]: those of class k; *bad: a row whose pieces are not in order
__global__ __launch_bounds__(kBuildBlock) void k_count_segments(int32_t n_long, int32_t n_slices, int32_t part_rows,
                                                                const int32_t* __restrict__ bound, int32_t* counts, int32_t* bad) {
  __shared__ int32_t total[kClasses];
  if (threadIdx.x < kClasses) total[threadIdx.x] = 0;
  __syncthreads();
  const int32_t* lo = bound + (int64_t)(blockIdx.x % n_slices) * n_long;
  const int p0 = (int)(blockIdx.x / n_slices) * part_rows, p_end = min(n_long, p0 + part_rows);
  int full = 0;
  for (int p = p0 + threadIdx.x; p < p_end; p += kBuildBlock) {
    const int len = lo[n_long + p] - lo[p];
    if (len < 0) { *bad = 1; continue; }
    full += len / kSegment;
    if (len % kSegment) atomicAdd(&total[kSegment - len % kSegment], 1);
  }
  if (full) atomicAdd(&total[0], full);
  __syncthreads();
  if (threadIdx.x < kClasses) counts[blockIdx.x * kClasses + threadIdx.x] = total[threadIdx.x];
}

// writes the segments of a unit; first[u * kClasses + k]: place of the first one of class k.  (Which of them a piece
// gets inside its class does not change any result.)  *bad: a column outside its slice
__global__ __launch_bounds__(kBuildBlock) void k_fill_segments(int32_t n_long, int32_t n_slices, int32_t part_rows, int32_t width,
                                                               int32_t n_cols, const int32_t* __restrict__ rows,
                                                               const int32_t* __restrict__ indices,
                                                               const int32_t* __restrict__ bound,
                                                               const int32_t* __restrict__ first, int2* seg_at, uint4* seg_cols,
                                                               int32_t* bad) {
  __shared__ int32_t next[kClasses];
  const int s = (int)(blockIdx.x % n_slices);
  if (threadIdx.x < kClasses) next[threadIdx.x] = first[blockIdx.x * kClasses + threadIdx.x];
  __syncthreads();
  const int32_t* lo = bound + (int64_t)s * n_long;
  const int p0 = (int)(blockIdx.x / n_slices) * part_rows, p_end = min(n_long, p0 + part_rows);
  const int64_t col0 = (int64_t)s * width;
  const int n_here = (int)min((int64_t)width, (int64_t)n_cols - col0);
  for (int p = p0 + (int)threadIdx.x; p < p_end; p += kBuildBlock) {
    int q = lo[p];
    const int len = lo[n_long + p] - q, full = len / kSegment;
    const int at_full = full ? atomicAdd(&next[0], full) : 0;
    const int at_rest = len % kSegment ? atomicAdd(&next[kSegment - len % kSegment], 1) : 0;
    const int row = rows[p];
    for (int k = 0, left = len; left > 0; ++k, left -= kSegment, q += kSegment) {
      const int n = min(left, kSegment), seg = n == kSegment ? at_full + k : at_rest;
      unsigned c[kSegment];
#pragma unroll
      for (int u = 0; u < kSegment; ++u) {
        const int64_t rel = (int64_t)indices[q + min(u, n - 1)] - col0;
        if (rel < 0 || rel >= n_here) *bad = 1;
        c[u] = (unsigned)rel & ((1u << kColumnBits) - 1u);
      }
      seg_at[seg] = make_int2(row, q);
      seg_cols[seg] = make_uint4(c[0] | (unsigned)(n - 1) << kColumnBits | c[1] << 16, c[2] | c[3] << 16, c[4] | c[5] << 16,
                                 c[6] | c[7] << 16);
    }
  }
}

template <int T, bool TAIL>
hipError_t launch(const SliceArgs& a, unsigned n_units, hipStream_t stream) {
  auto* kernel = &k_sddmm_slices<T, TAIL>;
  const size_t lds = sizeof(float4) * ((size_t)a.width * a.stride + 1);
  static OncePerDevice allowed;
  allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, allowed);
  hipLaunchKernelGGL(kernel, dim3(n_units), dim3(slice_threads<T>()), lds, stream, a);
  return hipGetLastError();
}

template <int T>
hipError_t launch_rows(const SliceArgs& a, unsigned n_units, hipStream_t stream) {
  return a.feat == 32 * T ? launch<T, false>(a, n_units, stream) : launch<T, true>(a, n_units, stream);
}

}  // namespace

void sddmm_slices_free(SddmmSlices* s, sptir_free_fn free_, void* actx) {
  void* ptrs[] = {s->seg_at, s->seg_cols, s->units};
  for (void* q : ptrs)
    if (q) free_(q, actx);
  *s = SddmmSlices();
}

sptir_status_t sddmm_slices_build(const sptir_csr_t* csr, int32_t feat_hint, sptir_alloc_fn alloc, sptir_free_fn free_, void* actx,
                                  hipStream_t stream, SddmmSlices* out, int32_t** rank_out) {
  *out = SddmmSlices();
  *rank_out = nullptr;
  const int64_t feat = feat_hint > 0 ? feat_hint : 128, min_nnz = slice_min_entries(feat);
  const int32_t n_rows = csr->n_rows, n_cols = csr->n_cols, width = slice_width(feat);
  if (width == 0 || csr->nnz < min_nnz) return SPTIR_OK;
  const int64_t n_slices64 = ((int64_t)n_cols + width - 1) / width;
  const int64_t min_deg = std::max<int64_t>(1, kMinPiece * n_cols / width);
  if (n_slices64 > csr->nnz) return SPTIR_OK;
  const int32_t n_slices = (int32_t)n_slices64;

  SddmmSlices s;
  std::vector<void*> temporaries;
  sptir_status_t st = SPTIR_OK;
  auto temporary = [&](size_t bytes) {
    void* p = alloc(bytes, actx, stream);
    if (p) temporaries.push_back(p); else st = SPTIR_ERR_ALLOC;
    return p;
  };
  auto hip = [&](hipError_t e, const char* what) {
    if (e != hipSuccess) st = note_hip_error(e, what);
    return e == hipSuccess;
  };
  auto read_back = [&](void* dst, const void* src, size_t bytes) {
    return hip(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, stream), "hipMemcpyAsync") &&
           hip(hipStreamSynchronize(stream), "hipStreamSynchronize");
  };
  bool use = false;
  int32_t* rank = nullptr;
  auto build = [&]() {
    const size_t room = scan_room((int64_t)n_rows + 1), n_seq = room / kScanSeq;
    rank = (int32_t*)temporary(sizeof(int32_t) * room);
    int32_t* seq_base = (int32_t*)temporary(sizeof(int32_t) * (n_seq + 1));
    unsigned long long* entries = (unsigned long long*)temporary(16);
    if (!rank || !seq_base || !entries) return;
    const unsigned row_blocks = (unsigned)(((int64_t)n_rows + 1 + kBuildBlock - 1) / kBuildBlock);
    if (!hip(hipMemsetAsync(entries, 0, 16, stream), "hipMemsetAsync")) return;
    hipLaunchKernelGGL(k_long_rows, dim3(row_blocks), dim3(kBuildBlock), 0, stream, n_rows, csr->nnz, csr->indptr, min_deg, rank,
                       entries);
    if ((st = device_exclusive_scan(rank, (int64_t)n_rows + 1, seq_base, stream)) != SPTIR_OK) return;
    unsigned long long long_nnz = 0;
    int32_t n_long = 0;
    if (!hip(hipMemcpyAsync(&n_long, seq_base + n_seq, sizeof(n_long), hipMemcpyDeviceToHost, stream), "hipMemcpyAsync") ||
        !read_back(&long_nnz, entries, sizeof(long_nnz)))
      return;
    if (n_long <= 0 || (int64_t)long_nnz > csr->nnz || !slices_pay(n_cols, feat, n_long, (int64_t)long_nnz)) return;

    int32_t* rows = (int32_t*)temporary(sizeof(int32_t) * (size_t)n_long);
    int32_t* bound = (int32_t*)temporary(sizeof(int32_t) * ((size_t)n_slices + 1) * (size_t)n_long);
    // parts: enough units for the GPU, and no more rows of X at a time than leave room in an XCD's L2
    int64_t parts = std::max<int64_t>((kMinUnits + n_slices - 1) / n_slices, (n_long * feat * 4 + kPartBytes - 1) / kPartBytes);
    parts = std::max<int64_t>(1, std::min<int64_t>(parts, (int64_t)long_nnz / ((int64_t)n_slices * kMinUnitNnz)));
    const int32_t part_rows = (int32_t)((n_long + parts - 1) / parts);
    parts = (n_long + part_rows - 1) / part_rows;
    const size_t n_units = (size_t)n_slices * (size_t)parts;
    if (n_units > 0x7FFFFFFF) return;
    int32_t* counts = (int32_t*)temporary(sizeof(int32_t) * kClasses * n_units);
    if (!rows || !bound || !counts) return;
    int32_t* bad = (int32_t*)(entries + 1);
    hipLaunchKernelGGL(k_list_long_rows, dim3(row_blocks), dim3(kBuildBlock), 0, stream, n_rows, rank, rows);
    constexpr int kTile = 64;
    hipLaunchKernelGGL(k_slice_bounds<kTile>, dim3(slice_bounds_workgroups<kTile>(n_slices, n_long)), dim3(kBoundsBlock), 0, stream,
                       n_slices, width, n_long, n_long, rows, csr->indptr, csr->indices, bound);
    hipLaunchKernelGGL(k_count_segments, dim3((unsigned)n_units), dim3(kBuildBlock), 0, stream, n_long, n_slices, part_rows, bound,
                       counts, bad);
    if (!hip(hipGetLastError(), "slice bounds")) return;
    std::vector<int32_t> count(kClasses * n_units);
    int32_t is_bad = 0;
    if (!hip(hipMemcpyAsync(&is_bad, bad, sizeof(is_bad), hipMemcpyDeviceToHost, stream), "hipMemcpyAsync") ||
        !read_back(count.data(), counts, sizeof(int32_t) * count.size()))
      return;
    if (is_bad) return;

    std::vector<int32_t> begin(n_units + 1);
    int64_t at = 0, used = 0;
    for (size_t u = 0; u < n_units; ++u) {
      begin[u] = (int32_t)at;
      for (int k = 0; k < kClasses; ++k) {
        const int32_t n = count[u * kClasses + k];
        count[u * kClasses + k] = (int32_t)at;
        at += n;
      }
      used += at > begin[u];
    }
    begin[n_units] = (int32_t)at;
    if (!slices_pay_as_counted(n_cols, feat, n_long, (int64_t)long_nnz, used, at, n_slices, slices_of_half(begin, n_slices, parts)))
      return;
    const std::vector<SliceUnit> units = slice_units(begin, n_slices, parts, (at + kCus - 1) / kCus);
    if (units.size() > 0x7FFFFFFF) return;
    s.n_segs = at; s.n_units = (int64_t)units.size();
    s.width = width; s.nnz = (int64_t)long_nnz;
    auto keep = [&](size_t bytes) {
      void* p = alloc(bytes, actx, stream);
      if (p) s.device_bytes += bytes; else st = SPTIR_ERR_ALLOC;
      return p;
    };
    s.seg_at = (int2*)keep(sizeof(int2) * (size_t)at);
    s.seg_cols = (uint4*)keep(sizeof(uint4) * (size_t)at);
    s.units = (int4*)keep(sizeof(SliceUnit) * units.size());
    if (!s.seg_at || !s.seg_cols || !s.units) return;
    if (!hip(hipMemcpyAsync(counts, count.data(), sizeof(int32_t) * count.size(), hipMemcpyHostToDevice, stream), "hipMemcpyAsync") ||
        !hip(hipMemcpyAsync(s.units, units.data(), sizeof(SliceUnit) * units.size(), hipMemcpyHostToDevice, stream), "hipMemcpyAsync"))
      return;
    hipLaunchKernelGGL(k_fill_segments, dim3((unsigned)n_units), dim3(kBuildBlock), 0, stream, n_long, n_slices, part_rows, width,
                       n_cols, rows, csr->indices, bound, counts, s.seg_at, s.seg_cols, bad);
    if (!hip(hipGetLastError(), "k_fill_segments")) return;
    if (!read_back(&is_bad, bad, sizeof(is_bad))) return;
    use = !is_bad;
  };
  try {
    temporaries.reserve(8);
    build();
  } catch (const std::bad_alloc&) {
    st = SPTIR_ERR_ALLOC;
  }
  if (st != SPTIR_OK) use = false;
  if (st == SPTIR_ERR_ALLOC) st = SPTIR_OK;  // (a plan without slices needs less at a time)
  (void)hipStreamSynchronize(stream);  // (nothing that is given back below is still written to)
  for (void* p : temporaries)
    if (!(use && p == rank)) free_(p, actx);
  if (use) {
    *out = s;
    *rank_out = rank;
  } else {
    sddmm_slices_free(&s, free_, actx);
  }
  return st;
}

sptir_status_t sddmm_slices_run(const SddmmSlices& s, int32_t n_cols, const float* values, const float* X, const float* Yt, float* B,
                                int32_t feat, hipStream_t stream) {
  SliceArgs a;
  a.units = s.units; a.seg_at = s.seg_at; a.seg_cols = s.seg_cols;
  a.values = values; a.X = X; a.Yt = Yt; a.B = B;
  a.feat = feat; a.quads = (feat + 3) / 4; a.stride = slice_stride(a.quads); a.width = s.width; a.n_cols = n_cols;
  const unsigned n = (unsigned)s.n_units;
  hipError_t e;
  switch (slice_lane_quads(s.width, feat)) {
    case 1: e = launch_rows<1>(a, n, stream); break;
    case 2: e = launch_rows<2>(a, n, stream); break;
    case 3: e = launch_rows<3>(a, n, stream); break;
    case 4: e = launch_rows<4>(a, n, stream); break;
    case 5: e = launch_rows<5>(a, n, stream); break;
    case 6: e = launch_rows<6>(a, n, stream); break;
    case 7: e = launch_rows<7>(a, n, stream); break;
    case 8: e = launch_rows<8>(a, n, stream); break;
    default:
      hipLaunchKernelGGL(k_sddmm_segments, dim3(n), dim3(512), 0, stream, a);
      e = hipGetLastError();
  }
  if (e != hipSuccess) return note_hip_error(e, "sddmm slices");
  return SPTIR_OK;
}

}  // namespace sptir
