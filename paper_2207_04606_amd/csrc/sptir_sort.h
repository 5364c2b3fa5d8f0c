// Device code of the radix sort by length (order.hip), for kernels that do a pass of it next to other work.
#ifndef SPTIR_SORT_H_
#define SPTIR_SORT_H_

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

// hist[(launch * 256 + digit) * tiles + tile] = elements of the tile with that digit; wg = launch * tiles + tile
__device__ __forceinline__ void sort_hist_workgroup(const SortInput& in, int32_t n_rb, int tiles, int shift, unsigned wg,
                                                    int32_t* __restrict__ hist) {
  __shared__ int count[kDigits];
  const int tile = (int)(wg % (unsigned)tiles), launch = (int)(wg / (unsigned)tiles);
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
__device__ __forceinline__ void sort_scatter_workgroup(const SortInput& in, int32_t n_rb, int tiles, int shift, unsigned wg,
                                                       const int32_t* __restrict__ hist,
                                                       uint32_t* __restrict__ keys_out /* NULL: the last pass */,
                                                       int32_t* __restrict__ vals_out) {
  __shared__ int base[kDigits];
  __shared__ int wave_cnt[4][kDigits];
  const int tile = (int)(wg % (unsigned)tiles), launch = (int)(wg / (unsigned)tiles);
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
}  // namespace sptir

#endif  // SPTIR_SORT_H_
