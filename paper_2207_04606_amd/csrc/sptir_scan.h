// Device helpers shared by the builder kernels: workgroup scans and the lower
// bound in a sorted row.  Everything here has internal linkage.
#ifndef SPTIR_SCAN_H_
#define SPTIR_SCAN_H_

#include "sptir_internal.h"

namespace sptir {
namespace {

constexpr int kWaves = kBuildBlock / 64;

// first position q in [lo, hi) whose column is >= bound
__device__ __forceinline__ int lower_bound_col(const int32_t* __restrict__ indices, int lo, int hi, int64_t bound) {
  while (lo < hi) {
    int mid = lo + ((hi - lo) >> 1);
    if ((int64_t)indices[mid] < bound) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// largest r in [0, n_rows) with indptr[r] <= e (e < nnz, so it exists); the lanes of a wavefront probe 64 places at a
// time (three dependent loads for 200,000 rows where halving takes 18)
__device__ __forceinline__ int row_of_entry(const int32_t* __restrict__ indptr, int n_rows, int64_t e, int lane) {
  int lo = 0, hi = n_rows;  // invariant: indptr[lo] <= e < indptr[hi]
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int64_t at = lo + (int64_t)(lane + 1) * step;
    const bool below = at < hi && (int64_t)indptr[at] <= e;
    const int n = __popcll(__ballot(below));  // (ascending: the lanes below come first)
    lo += n * step;
    hi = (int)min((int64_t)hi, (int64_t)lo + step);
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// exclusive scan over the 256 threads of a workgroup; *total = sum of all
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* wave_sums /* [kWaves] shared */, T* total) {
  int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T incl = wave_inclusive_scan(v, lane);
  __syncthreads();  // wave_sums may still be read from a previous call
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    T ws = wave_sums[w];
    if (w < wave) base += ws;
    tot += ws;
  }
  *total = tot;
  return base + incl - v;
}

// seq[0 .. len) becomes its exclusive prefix; returns its sum.  By one workgroup of kBuildBlock threads; a thread scans
// kScanPerThread consecutive elements itself, so a long sequence costs few workgroup-wide steps.
constexpr int kScanPerThread = 8;

template <typename T>
__device__ __forceinline__ T scan_sequence(T* seq, int32_t len, T* wave_sums /* [kWaves] shared */) {
  T carry = 0;
  for (int64_t base = 0; base < len; base += (int64_t)kBuildBlock * kScanPerThread) {
    const int64_t e0 = base + (int64_t)threadIdx.x * kScanPerThread;
    T v[kScanPerThread];
    T mine = 0;
#pragma unroll
    for (int i = 0; i < kScanPerThread; ++i) {
      v[i] = (e0 + i < len) ? seq[e0 + i] : (T)0;
      mine += v[i];
    }
    T tot;
    T before = carry + block_exclusive_scan(mine, wave_sums, &tot);
#pragma unroll
    for (int i = 0; i < kScanPerThread; ++i) {
      if (e0 + i < len) seq[e0 + i] = before;
      before += v[i];
    }
    carry += tot;
  }
  return carry;
}

// data[0 .. n), n at most kScanOneMost, becomes its exclusive prefix, by one workgroup with a run of elements per thread
constexpr int kScanThreads = 1024, kScanRun = 16, kScanOneMost = kScanThreads * kScanRun;
__global__ __launch_bounds__(kScanThreads) void k_scan_one(int32_t* data, int32_t n) {
  __shared__ int32_t wave_sum[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i0 = (int)threadIdx.x * kScanRun;
  int32_t v[kScanRun], mine = 0;
#pragma unroll
  for (int k = 0; k < kScanRun; k += 4) {
    int4 q = make_int4(0, 0, 0, 0);
    if (i0 + k + 4 <= n) {
      q = *reinterpret_cast<const int4*>(data + i0 + k);  // (allocations are aligned to 256 bytes)
    } else {
      if (i0 + k < n) q.x = data[i0 + k];
      if (i0 + k + 1 < n) q.y = data[i0 + k + 1];
      if (i0 + k + 2 < n) q.z = data[i0 + k + 2];
    }
    v[k] = q.x; v[k + 1] = q.y; v[k + 2] = q.z; v[k + 3] = q.w;
  }
#pragma unroll
  for (int k = 0; k < kScanRun; ++k) mine += v[k];
  const int32_t incl = wave_inclusive_scan(mine, lane);
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int32_t before = incl - mine;
  for (int w = 0; w < wave; ++w) before += wave_sum[w];
#pragma unroll
  for (int k = 0; k < kScanRun; ++k) {
    if (i0 + k < n) data[i0 + k] = before;
    before += v[k];
  }
}

// One workgroup per sequence: data[seq*len .. +len) becomes its exclusive prefix, totals[seq] its sum.
template <typename T>
__global__ __launch_bounds__(kBuildBlock) void k_scan_sequences(T* data, int32_t len, T* totals) {
  __shared__ T wave_sums[kWaves];
  const T total = scan_sequence(data + (int64_t)blockIdx.x * len, len, wave_sums);
  if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

}  // namespace
}  // namespace sptir

#endif  // SPTIR_SCAN_H_
