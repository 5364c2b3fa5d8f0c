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

namespace sptir {
namespace {

constexpr int kSortTile = 1024;            // elements per workgroup and pass
constexpr int kSortRounds = kSortTile / 256;
constexpr int kDigits = 256;

// What a pass sorts: the first one takes list lengths and row block numbers as they come, the later ones what the pass
// before them wrote.
struct SortInput {
  const int64_t* list_ptr;  // first pass: first chunk of every list (NULL otherwise)
  const int32_t* row_ptr;   // or first entry of every row: those of min_len to max_len entries by class of length, the others last
  int32_t min_len;
  float log2_max, per_log2;
  const uint32_t* keys;
  const int32_t* vals;
  __device__ uint32_t key(int64_t at) const {
    if (row_ptr) {
      const int32_t len = row_ptr[at + 1] - row_ptr[at];
      if (len < min_len) return kDigits - 1;
      return (uint32_t)min(max((int)((log2_max - log2f((float)len)) * per_log2), 0), kDigits - 2);
    }
    if (!list_ptr) return keys[at];
    const int64_t len = list_ptr[at + 1] - list_ptr[at];
    return 0xFFFFFFFFu - (len < 0xFFFFFFFFll ? (uint32_t)len : 0xFFFFFFFFu);
  }
  __device__ int32_t val(int64_t at, int i) const { return list_ptr || row_ptr ? i : vals[at]; }
};

// hist[(launch * 256 + digit) * tiles + tile] = elements of the tile with that digit; workgroup = launch * tiles + tile
__global__ __launch_bounds__(256) void k_sort_hist(SortInput in, int32_t n_rb, int tiles, int shift,
                                                   int32_t* __restrict__ hist) {
  __shared__ int count[kDigits];
  const int tile = blockIdx.x % tiles, launch = blockIdx.x / tiles;
  count[threadIdx.x] = 0;
  __syncthreads();
  const int64_t seg0 = (int64_t)launch * n_rb;
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = tile * kSortTile + r * 256 + threadIdx.x;
    if (i < n_rb) atomicAdd(&count[(in.key(seg0 + i) >> shift) & 255u], 1);
  }
  __syncthreads();
  hist[((int64_t)launch * kDigits + threadIdx.x) * tiles + tile] = count[threadIdx.x];
}

// `hist` scanned per launch (exclusive, digit-major): the first output position of each (digit, tile).  Elements
// keep their order inside a digit: the tile is walked 256 elements at a time, in order, and inside such a round a
// lane's rank is the number of lower lanes, then of lower wavefronts, with the same digit.
__global__ __launch_bounds__(256) void k_sort_scatter(SortInput in, int32_t n_rb, int tiles, int shift,
                                                      const int32_t* __restrict__ hist,
                                                      uint32_t* __restrict__ keys_out /* NULL: the last pass */,
                                                      int32_t* __restrict__ vals_out) {
  __shared__ int base[kDigits];
  __shared__ int wave_cnt[4][kDigits];
  const int tile = blockIdx.x % tiles, launch = blockIdx.x / tiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  base[tid] = hist[((int64_t)launch * kDigits + tid) * tiles + tile];
#pragma unroll
  for (int w = 0; w < 4; ++w) wave_cnt[w][tid] = 0;
  __syncthreads();
  const int64_t seg0 = (int64_t)launch * n_rb;
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = tile * kSortTile + r * 256 + tid;
    const bool valid = i < n_rb;
    const uint32_t key = valid ? in.key(seg0 + i) : 0u;
    const int32_t val = valid ? in.val(seg0 + i, i) : 0;
    const int digit = (int)((key >> shift) & 255u);
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool mine = (digit >> bit) & 1;
      const unsigned long long b = __ballot(mine);
      peers &= mine ? b : ~b;
    }
    const int rank_in_wave = __popcll(peers & ((1ull << lane) - 1ull));
    if (valid && rank_in_wave == 0) wave_cnt[wave][digit] = __popcll(peers);
    __syncthreads();
    if (valid) {
      int before = 0;
      for (int w = 0; w < wave; ++w) before += wave_cnt[w][digit];
      const int64_t at = seg0 + base[digit] + before + rank_in_wave;
      if (keys_out) keys_out[at] = key;
      vals_out[at] = val;
    }
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) { all += wave_cnt[w][tid]; wave_cnt[w][tid] = 0; }
    base[tid] += all;
    __syncthreads();
  }
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
