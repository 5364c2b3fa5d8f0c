// Microbenchmarks of the on-chip roofs the SpMM and SDDMM kernels are priced against: how fast a CU pulls 128-byte rows
// of X at random through the vector-memory path (the gather every stored non-zero costs), how fast it reads rows at random
// from its LDS (the gather of the column slices), and how fast it issues float32 FMAs.  They belong to the measured product: bench.py runs them next to the SpMM timings so that the
// "binding roof" it reports is a number taken on the same GPU in the same process.
#include "sptir_internal.h"

namespace sptir {
namespace {

__device__ __forceinline__ unsigned lcg(unsigned s) { return s * 1664525u + 1013904223u; }

// Every group of 8 lanes reads one 128-byte line (lane: 16 bytes) of a random row of the window
// [0, n_rows) x [tile * 32, tile * 32 + 32) of X, 8 loads in flight per lane, like the SpMM kernels' gather step.
// The feature tile follows the workgroup id modulo 8 the way the SpMM kernels bind tiles to XCDs when
// `tiles` > 1, so that an XCD's L2 sees n_rows * 128 bytes.
__global__ __launch_bounds__(256) void k_roof_gather(const float* __restrict__ X, unsigned n_rows, int row_floats,
                                                     int tiles, int iters, float* sink) {
  const int lane = threadIdx.x & 63, g = lane >> 3, fl = lane & 7;
  const unsigned wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int tile = tiles > 1 ? (int)(blockIdx.x & 7) % tiles : 0;
  unsigned s = (wave * 8u + g) * 2654435761u + 12345u;
  const float* Xf = X + tile * 32 + fl * 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < iters; ++it) {
    float4 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s = lcg(s);
      const unsigned r = (unsigned)(((unsigned long long)(s >> 4) * n_rows) >> 28);
      x[u] = *reinterpret_cast<const float4*>(Xf + (size_t)r * row_floats);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) { acc[0] += x[u].x; acc[1] += x[u].y; acc[2] += x[u].z; acc[3] += x[u].w; }
  }
  const float t = acc[0] + acc[1] + acc[2] + acc[3];
  if (t == 1234.5f) sink[0] = t;  // keeps the loads alive; X is zero-filled or random, the store all but never happens
}

// Every group of LG lanes reads rows of LG * T float4 at random, `stride` float4 from one to the next, out of the workgroup's LDS:
// eight rows at a time, as the column slices do, their numbers from four 32-bit generators a lane (half a word each, so that
// making them takes less of the issue slots than the reads take of LDS).  mask + 1 rows, a power of two.
constexpr int kRoofLdsThreads = 1024;
constexpr unsigned kRoofLdsBytes = 156 * 1024;
template <int LG, int T>
__global__ __launch_bounds__(kRoofLdsThreads) void k_roof_lds(unsigned mask, unsigned stride, int iters, float* sink) {
  extern __shared__ __align__(16) float4 rows[];
  for (unsigned i = threadIdx.x; i < (mask + 1) * stride; i += kRoofLdsThreads) rows[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  const unsigned group = (blockIdx.x * kRoofLdsThreads + threadIdx.x) / LG;
  const float4* mine = rows + threadIdx.x % LG;
  unsigned s[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) s[w] = lcg(lcg(4 * group + w)) | 1u;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {  // (xorshift)
      s[w] ^= s[w] << 13; s[w] ^= s[w] >> 17; s[w] ^= s[w] << 5;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const unsigned r = ((u & 1) ? s[u / 2] >> 16 : s[u / 2]) & mask;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float4 v = mine[__umul24(r, stride) + LG * t];
        acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
      }
    }
  }
  const float t = acc[0] + acc[1] + acc[2] + acc[3];
  if (t == 1234.5f) sink[0] = t;  // (never: the rows are zeros)
}

// 8 independent FMA chains per lane, `iters` rounds of 8 FMAs each: 16 flops per lane and round
__global__ __launch_bounds__(256) void k_roof_fma(int iters, float seed, float* sink) {
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = seed + (float)(threadIdx.x + i);
  const float m = 1.0000001f, c = 1e-7f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = fmaf(a[i], m, c);
  }
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) t += a[i];
  if (t == 1234.5f) sink[0] = t;
}

}  // namespace
}  // namespace sptir

using namespace sptir;

extern "C" sptir_status_t sptir_roof_gather(const float* X, int64_t n_rows, int32_t row_floats, int32_t tiles,
                                            int32_t n_workgroups, int32_t iters, float* sink, void* stream_,
                                            float* ms_out, double* bytes_out) {
  if (!X || !sink || !ms_out || !bytes_out) return SPTIR_ERR_INVALID_ARG;
  if (n_rows < 1 || n_rows > 0x0FFFFFFF || row_floats < 32 || row_floats % 4 != 0 || ((uintptr_t)X & 15) != 0)
    return SPTIR_ERR_INVALID_ARG;
  if (tiles < 1 || tiles > 8 || tiles * 32 > row_floats || n_workgroups < 1 || iters < 1) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  SPTIR_HIP(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return note_hip_error(hipGetLastError(), "hipEventCreate"); }
  sptir_status_t st = SPTIR_OK;
  // one untimed launch, then the timed one
  hipLaunchKernelGGL(k_roof_gather, dim3((unsigned)n_workgroups), dim3(256), 0, stream, X, (unsigned)n_rows,
                     row_floats, tiles, iters, sink);
  if (hipEventRecord(e0, stream) != hipSuccess) st = note_hip_error(hipGetLastError(), "hipEventRecord");
  hipLaunchKernelGGL(k_roof_gather, dim3((unsigned)n_workgroups), dim3(256), 0, stream, X, (unsigned)n_rows,
                     row_floats, tiles, iters, sink);
  if (st == SPTIR_OK && (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(ms_out, e0, e1) != hipSuccess))
    st = note_hip_error(hipGetLastError(), "timing the gather roof");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  // 4 wavefronts per workgroup, 8 loads of 64 lanes x 16 bytes per round
  *bytes_out = (double)n_workgroups * 4.0 * (double)iters * 8.0 * 1024.0;
  return st;
}

extern "C" sptir_status_t sptir_roof_lds_gather(int32_t row_floats, int32_t row_stride, int32_t n_workgroups, int32_t iters,
                                                float* sink, void* stream_, float* ms_out, double* bytes_out) {
  if (!sink || !ms_out || !bytes_out || n_workgroups < 1 || iters < 1) return SPTIR_ERR_INVALID_ARG;
  if (row_stride < row_floats || row_stride % 4 != 0 || row_stride > 256) return SPTIR_ERR_INVALID_ARG;
  void (*kernel)(unsigned, unsigned, int, float*) = nullptr;
  static OncePerDevice allowed[5];
  int which = 0;
  switch (row_floats) {
    case 4: kernel = k_roof_lds<1, 1>; which = 0; break;
    case 8: kernel = k_roof_lds<2, 1>; which = 1; break;
    case 16: kernel = k_roof_lds<4, 1>; which = 2; break;
    case 32: kernel = k_roof_lds<8, 1>; which = 3; break;
    case 128: kernel = k_roof_lds<8, 4>; which = 4; break;
    default: return SPTIR_ERR_INVALID_ARG;
  }
  const unsigned stride = (unsigned)row_stride / 4;
  unsigned n_rows = 1;
  while (2 * n_rows * stride * sizeof(float4) <= kRoofLdsBytes) n_rows *= 2;
  const size_t lds = (size_t)n_rows * stride * sizeof(float4);
  allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, allowed[which]);
  hipStream_t stream = (hipStream_t)stream_;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  SPTIR_HIP(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return note_hip_error(hipGetLastError(), "hipEventCreate"); }
  sptir_status_t st = SPTIR_OK;
  auto launch = [&] {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_workgroups), dim3(kRoofLdsThreads), lds, stream, n_rows - 1, stride, iters, sink);
    if (st == SPTIR_OK && hipGetLastError() != hipSuccess) st = note_hip_error(hipErrorLaunchFailure, "k_roof_lds");
  };
  launch();  // one untimed, then the timed one
  if (hipEventRecord(e0, stream) != hipSuccess) st = note_hip_error(hipGetLastError(), "hipEventRecord");
  launch();
  if (st == SPTIR_OK && (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(ms_out, e0, e1) != hipSuccess))
    st = note_hip_error(hipGetLastError(), "timing the LDS gather roof");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  const double lanes = row_floats == 128 ? 8 : row_floats / 4;
  *bytes_out = (double)n_workgroups * kRoofLdsThreads / lanes * (double)iters * 8.0 * 4.0 * row_floats;
  return st;
}

extern "C" sptir_status_t sptir_roof_fma(int32_t n_workgroups, int32_t iters, float* sink, void* stream_,
                                         float* ms_out, double* flops_out) {
  if (!sink || !ms_out || !flops_out || n_workgroups < 1 || iters < 1) return SPTIR_ERR_INVALID_ARG;
  hipStream_t stream = (hipStream_t)stream_;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  SPTIR_HIP(hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return note_hip_error(hipGetLastError(), "hipEventCreate"); }
  sptir_status_t st = SPTIR_OK;
  hipLaunchKernelGGL(k_roof_fma, dim3((unsigned)n_workgroups), dim3(256), 0, stream, iters, 1.0f, sink);
  if (hipEventRecord(e0, stream) != hipSuccess) st = note_hip_error(hipGetLastError(), "hipEventRecord");
  hipLaunchKernelGGL(k_roof_fma, dim3((unsigned)n_workgroups), dim3(256), 0, stream, iters, 1.0f, sink);
  if (st == SPTIR_OK && (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                         hipEventElapsedTime(ms_out, e0, e1) != hipSuccess))
    st = note_hip_error(hipGetLastError(), "timing the FMA roof");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *flops_out = (double)n_workgroups * 256.0 * (double)iters * 16.0;
  return st;
}
