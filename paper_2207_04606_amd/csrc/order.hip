// Launch order of the row blocks of every SpMM launch: longest chunk list first, so that the last wavefronts of a
// launch to finish are short ones (the row blocks of a power-law graph differ several-fold in work).  The launches
// are sorted independently of each other by a stable least-significant-digit radix sort, 8 bits a pass:
// key = 2^32 - 1 - list length, value = row block, so equal lengths stay in ascending row block order.  Only the
// digits that can differ are sorted: the caller says how long a list can be at most.
#include <math.h>

#include <algorithm>
#include <cstring>

#include "sptir_internal.h"
#include "sptir_scan.h"
#include "sptir_sort.h"

namespace sptir {
namespace {

__global__ __launch_bounds__(256) void k_sort_hist(SortInput in, int32_t n_rb, int tiles, int shift, int32_t* __restrict__ hist) {
  sort_hist_workgroup(in, n_rb, tiles, shift, blockIdx.x, hist);
}

__global__ __launch_bounds__(256) void k_sort_scatter(SortInput in, int32_t n_rb, int tiles, int shift,
                                                      const int32_t* __restrict__ hist, uint32_t* __restrict__ keys_out,
                                                      int32_t* __restrict__ vals_out) {
  sort_scatter_workgroup(in, n_rb, tiles, shift, blockIdx.x, hist, keys_out, vals_out);
}

}  // namespace

sptir_status_t order_row_blocks(const int64_t* rb_chunk_ptr, int32_t n_launches, int32_t n_rb, int64_t max_list_len,
                                int32_t* rb_order, sptir_alloc_fn alloc, sptir_free_fn free_, void* actx,
                                hipStream_t stream, void** scratch_out) {
  (void)free_;
  *scratch_out = nullptr;
  const int64_t n = (int64_t)n_launches * n_rb;
  if (n <= 0) return SPTIR_OK;
  if (n > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  // the keys of a launch differ in the bits of (2^32 - 1 - length) below the highest bit a length can have
  int bits = 1;
  while (bits < 32 && ((int64_t)1 << bits) <= max_list_len) ++bits;
  const int passes = (bits + 7) / 8;
  const int64_t tiles = ((int64_t)n_rb + kSortTile - 1) / kSortTile;
  const int64_t n_hist = (int64_t)n_launches * kDigits * tiles;
  if (n_hist > 0x7FFFFFFF || tiles * n_launches > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  const size_t key_bytes = (sizeof(uint32_t) * (size_t)n + 255) & ~(size_t)255;
  const size_t hist_bytes = (sizeof(int32_t) * (size_t)n_hist + 255) & ~(size_t)255;
  const size_t tot_bytes = (sizeof(int32_t) * (size_t)n_launches + 255) & ~(size_t)255;
  char* scratch = (char*)scratch_alloc(3 * key_bytes + hist_bytes + tot_bytes, alloc, actx, stream);
  if (!scratch) return SPTIR_ERR_ALLOC;
  *scratch_out = scratch;  // the caller gives it back (scratch_free) once the stream has drained
  uint32_t* keys[2] = {(uint32_t*)scratch, (uint32_t*)(scratch + key_bytes)};
  int32_t* other_vals = (int32_t*)(scratch + 2 * key_bytes);
  int32_t* hist = (int32_t*)(scratch + 3 * key_bytes);
  int32_t* totals = (int32_t*)(scratch + 3 * key_bytes + hist_bytes);
  // values ping-pong between rb_order and the scratch copy so that the last pass writes rb_order
  int32_t* vals[2];
  vals[passes % 2] = rb_order;
  vals[1 - passes % 2] = other_vals;
  for (int pass = 0; pass < passes; ++pass) {
    const int from = pass % 2, to = 1 - from;
    const SortInput in{pass == 0 ? rb_chunk_ptr : nullptr, nullptr, 0, 0.f, 0.f, keys[from], vals[from]};
    hipLaunchKernelGGL(k_sort_hist, dim3((unsigned)(tiles * n_launches)), dim3(256), 0, stream, in, n_rb,
                       (int)tiles, 8 * pass, hist);
    hipLaunchKernelGGL(k_scan_sequences<int32_t>, dim3((unsigned)n_launches), dim3(kBuildBlock), 0, stream, hist,
                       (int32_t)(kDigits * tiles), totals);
    hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)(tiles * n_launches)), dim3(256), 0, stream, in, n_rb, (int)tiles,
                       8 * pass, hist, pass + 1 < passes ? keys[to] : nullptr, vals[to]);
  }
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

size_t order_rows_scratch(int32_t n_rows) {
  const int64_t n_hist = (int64_t)kDigits * (((int64_t)n_rows + kSortTile - 1) / kSortTile);
  return sizeof(int32_t) * (scan_room(n_hist) + scan_room(n_hist) / kScanSeq + 1);
}

sptir_status_t order_rows_by_class(const int32_t* row_ptr, int32_t n_rows, int32_t min_len, int64_t max_len, int32_t* order,
                                   void* scratch, hipStream_t stream) {
  const int64_t tiles = ((int64_t)n_rows + kSortTile - 1) / kSortTile, n_hist = kDigits * tiles;
  if (n_hist > 0x7FFFFFFF) return SPTIR_ERR_OVERFLOW;
  int32_t *hist = (int32_t*)scratch, *seq_base = hist + scan_room(n_hist);
  const float top = log2f((float)max_len), span = top - log2f((float)min_len);
  const SortInput in{nullptr, row_ptr, min_len, top, (kDigits - 1) / std::max(span, 0.01f), nullptr, nullptr};
  hipLaunchKernelGGL(k_sort_hist, dim3((unsigned)tiles), dim3(256), 0, stream, in, n_rows, (int)tiles, 0, hist);
  if (n_hist <= kScanOneMost) {  // (one launch instead of four)
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanThreads), 0, stream, hist, (int32_t)n_hist);
  } else {
    const sptir_status_t st = device_exclusive_scan(hist, n_hist, seq_base, stream);
    if (st != SPTIR_OK) return st;
  }
  hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)tiles), dim3(256), 0, stream, in, n_rows, (int)tiles, 0, hist,
                     (uint32_t*)nullptr, order);
  SPTIR_HIP(hipGetLastError());
  return SPTIR_OK;
}

}  // namespace sptir
