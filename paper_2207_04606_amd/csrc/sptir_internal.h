// Internal declarations shared by the translation units of libsptir.so.
#ifndef SPTIR_INTERNAL_H_
#define SPTIR_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "per_device.h"
#include "sptir.h"

namespace sptir {

// The SpMM kernel walks the real entries of the stored rows in chunks of kChunkSlots slots.
constexpr int kChunkSlots = 64;
constexpr int kRowLog2W = 31;
constexpr int kChunksPerQuad = 4;  // chunks the SpMM kernel fetches with one load per lane and array
constexpr int kBuildBlock = 256;  // rows per workgroup in the builder kernels
// Row pieces of more than `heavy_len` real entries leave the chunk lists (a wavefront walks a list alone and keeps
// the Y rows of its row block on chip).  Their entries form one sequence of 64-slot chunks, piece after piece in the
// order of the canonical arrays (partition-major); the sequence is cut into "heavy lists" of kHeavyListChunks chunks,
// a wavefront each, which write one partial sum per finished piece plus one for whatever piece is unfinished where
// the list ends.  A last launch adds a row's partial sums to Y in a fixed order.
constexpr int kHeavyLenMax = 2048;      // largest threshold the size rules choose
constexpr int kHeavyListChunks = 16;    // most chunks per heavy list (a multiple of kChunksPerQuad; on the largest graph 16
                                        // beat 32 by 2 % and 64 by 4 % of the heavy launch; graphs with few heavy
                                        // chunks get shorter lists)
// features per partial-sum row: a wider Y is produced in sweeps of this many.  Wide rows (one sweep for most Y) where there
// are few of them; narrow ones only for sptir_spmm_noalloc.  (All of them hold whole feature tiles: lanes past the last
// feature of a sweep store too.)
constexpr int kPartialFeat = 128, kWidePartialFeat = 512, kNarrowPartialFeat = 64;
constexpr int64_t kWidePartialRows = 8192;  // (16 MB)
// Compact stream records spend 8 bytes per slot instead of 12: one word holds the column relative to the first
// column of the launch (bits 0..19), the row relative to the row block (20..26), "slot is real" (27), the chunk's
// log2w code (28..30; 3 = queue chunk, 7 = cut from one long row) and the hand-over flag (31; of the chunk, or in a
// queue chunk of the slot: the last entry of a row piece in its queue); the other word the value.
constexpr int kCompactColBits = 20;
constexpr int kCompactMaxLog2RowBlock = 7;

// The long rows of a hyb handle (spmm_slices.hip): their entries by slices of kSliceCols columns.  n_long 0: none.
constexpr int kSliceCols = 2496;      // of X in LDS: 64 bytes of each, next to a row of zeros
// A row is long from so many entries per slice on.  70 power-law graphs of 1.5 M entries and more, against no slices: 6 1.066 times
// as fast, 8 1.065, 12 1.049, 16 1.027, 24 1.007; 232,965 rows, 114.6 M entries: 6 1.82 ms, 8 1.80, 12 1.84, 16 1.88.
constexpr int kMinSlicePiece = 8;
struct SpmmSlices {
  int32_t n_long = 0, n_units = 0, n_slices = 0;
  int64_t nnz = 0;
  void* blob = nullptr;               // one allocation that holds all of it
  size_t device_bytes = 0;
  const void *units = nullptr, *panels = nullptr;
  const int32_t* panel_of = nullptr;
  int32_t *rows = nullptr, *step_of = nullptr;
  uint4* cols = nullptr;
  float4* vals = nullptr;
  float* partial = nullptr;           // partial sums of kPartialFeat features
};
}  // namespace sptir

// The handle behind sptir_hyb_t.  ELL and remainder share three device
// allocations so that one SpMM launch can walk both:
//   row_ids = [ELL_ROW | REM_ROW], cols = [ELL_COL | REM_COL], vals likewise.
struct sptir_hyb {
  int32_t n_rows, n_cols, c, k, w;
  int64_t nnz;
  int64_t B, R, S, M, T;
  int64_t* bucket_row_ptr;   // device [B+1]
  int64_t* bucket_slot_ptr;  // device [B+1]
  int32_t* rem_part_ptr;     // device [c+1]
  int64_t* rem_ptr;          // device [M+1]
  int32_t* row_ids;          // device [R+M]
  int32_t* cols;             // device [S+T]
  float* vals;               // device [S+T]
  int32_t* row_len;          // device [R+M], real length of every ELL row / remainder piece; negative: of a long row
  float* row_val;            // device [n_rows] or NULL: set when every row of A has one value for all its entries;
                             // the stream then holds no values and Y is scaled row by row at the end
  int32_t* stream;           // device [n_chunks * 128 or 192]: the chunks as fixed records, grouped by (phase, row block)
  int32_t spmm_plan;         // 0: built without the chunk stream (canonical arrays only); sptir_spmm refuses it
  int32_t compact_stream;    // 1: 8-byte slots (columns relative to the launch), 0: 12-byte slots (global columns)
  int64_t* rb_chunk_ptr;     // device [n_phases * n_row_blocks + 1], first chunk of each group
  int32_t* rb_order;         // device [n_phases * n_row_blocks]: the row blocks of a launch, longest list first
  int64_t n_chunks;
  int64_t longest_list;      // chunks
  // heavy pieces (see kHeavyListChunks): their chunks sit in `stream` from chunk heavy_chunk0 on
  int32_t heavy_len;
  int64_t n_heavy;            // heavy pieces
  int64_t n_heavy_nnz;        // their real entries
  int64_t n_heavy_chunks;     // their chunks, rounded up to whole quads
  int64_t heavy_chunk0;       // a multiple of kChunksPerQuad
  int32_t n_heavy_lists;
  int32_t* hlist_first_slot;  // device [n_heavy_lists]: partial-sum row the list's first write goes to
  int32_t* row_slot_ptr;      // device [n_rows + 1]: the partial-sum rows of row r are row_slots[row_slot_ptr[r] ..)
  int32_t* row_slots;         // device, in the order they are added to Y (partition-major)
  int32_t n_heavy_rows;       // rows with at least one heavy piece
  int32_t n_row_slots;        // elements of row_slots
  int32_t* heavy_rows;        // device [n_heavy_rows], ascending
  float* partial;             // device [(n_heavy + n_heavy_lists)][partial_feat]
  int32_t partial_feat;
  int32_t lowered_heavy_len;  // 1: heavy_len was chosen below kHeavyLenMax to even out the lists of a single sweep
  int64_t n_partial_rows;
  int32_t log2_row_block;    // rows of Y one wavefront accumulates in LDS (power of two)
  int32_t n_row_blocks;
  int32_t parts_per_phase;   // column partitions swept by one chunk list
  int32_t n_phases;
  int32_t rounds;            // 1: the lists sweep all partitions and are launched in rounds (Y written once)
  int32_t sweep_kb;          // kilobytes of Y (no rounds) or X (rounds) one sweep may touch; 0: the rules' defaults
  int32_t canonical_released;
  size_t device_bytes;
  // The device arrays above are parts of these allocations: [0] the index arrays whose sizes the
  // bucket totals fix, [1] cols and vals (can be released on their own), [2] the SpMM plan, [3] the long rows.
  int32_t heavy_list_chunks;  // chunks per heavy list of this handle: 4, 8, 16 or 32
  int32_t full_rows;        // sptir_spmm may use the 128-float tile (the row blocks are sized for it)
  sptir::SpmmSlices slices;   // the long rows: in no list and no heavy piece (their words in row_len are negative)
  int64_t whole_partial_rows; // partial-sum rows the heavy pieces would need with them
  void* blobs[4];
  size_t canonical_bytes;  // size of blobs[1]
  sptir_alloc_fn alloc;
  sptir_free_fn free_;
  void* alloc_ctx;
};

namespace sptir {

// allocator currently installed (api.hip)
void current_allocator(sptir_alloc_fn* a, sptir_free_fn* f, void** ctx);
void* default_alloc(size_t bytes, void* ctx, void* stream);
// Temporaries of a call: from `alloc`, or, when that is the default allocator, from a small cache of blocks that
// earlier calls have released (api.hip).  scratch_free takes back what scratch_alloc gave.  *got: the size of the block,
// which may be up to a quarter and 1 MB more than was asked for.
void* scratch_alloc(size_t bytes, sptir_alloc_fn alloc, void* actx, void* stream, size_t* got = nullptr);
void scratch_free(void* p, sptir_free_fn free_, void* actx);
// the same for the blocks of a handle that launches on any stream may still be reading
void handle_free(void* const* blobs, int n, sptir_free_fn free_, void* actx);
void default_free(void* p, void* ctx);

// sptir_hyb_build_ex; `opt` is complete (defaults filled in by the caller)
sptir_status_t hyb_build_impl(const sptir_csr_t* csr, int32_t n_col_parts, int32_t max_bucket_log2,
                              const sptir_build_options_t& opt, void* stream, sptir_hyb_t** out);
// the options a NULL pointer stands for / a caller's struct with unknown tail fields zeroed
sptir_build_options_t complete_options(const sptir_build_options_t* given);

// Validation of a CSR input on the GPU (builder.hip): `flags` is device memory, kValidationWords zeroed 64-bit words;
// the verdict is read from a host copy of them.  *one_value_per_row is only meaningful if the values were looked at.
constexpr int kValidationWords = 64 * 8;
// min_deg: rows of so many entries are counted as long
void launch_validation(const sptir_csr_t* csr, bool with_values, unsigned long long* flags, hipStream_t stream,
                       int32_t min_deg = INT32_MAX);
sptir_status_t validation_verdict(const unsigned long long* flags, bool* one_value_per_row);

// Exclusive scan of data[0 .. n) in place; data has room for scan_room(n) elements, seq_base for one int per
// kScanSeq of them plus one, which receives the total (at element n_seq = scan_room(n) / kScanSeq).
constexpr int kScanSeq = 4096;
sptir_status_t device_exclusive_scan(int32_t* data, int64_t n, int32_t* seq_base, hipStream_t stream);
size_t scan_room(int64_t n);

// pinned host memory, kept between calls
struct PinnedBuf { char* p = nullptr; size_t size = 0; };
PinnedBuf pinned_acquire(size_t bytes);
void pinned_release(PinnedBuf b);

// What the builder decides about the SpMM launches from the sizes alone (builder.hip; host code, no device access).
struct LaunchShape {
  int32_t log2_row_block;   // rows of Y per wavefront
  int32_t parts_per_phase;  // column partitions per chunk list
  int32_t n_phases;         // chunk-list launches per sweep (1 when rounds)
  int32_t compact;          // 1: 8-byte stream records
  int32_t rounds;           // 1: lists sweep all partitions, launched in rounds
  int32_t full_rows;        // 1: feature tiles of 128 floats (32 lanes per entry) where feat allows
};
LaunchShape decide_launch_shape(int32_t n_rows, int32_t n_cols, int32_t c, int32_t w, int64_t stored_slots,
                                const sptir_build_options_t& opt);

// Lane geometry sptir_spmm uses for `feat` (aligned16: X and Y are 16-byte aligned), and the feature tiles one sweep
// over the launches covers (spmm.hip; host code).
struct ListShape {
  bool rounds, full_rows;
  int log2_row_block;
  int64_t n_row_blocks, n_cols;
};
void lane_shape(int32_t feat, bool aligned16, const ListShape& lists, int* vec, int* lg);
// 512-byte feature tiles need row blocks whose Y tiles (rows x 512 bytes and the chunk rings, for the most wavefronts a workgroup can have: 4)
// fit a CU's LDS: up to 64 rows.  With larger row blocks sptir_spmm uses the 128-byte tiles whatever the handle asks for.  (A workgroup of one wavefront
// could have them beside more rows; what that would give was not measured.)
inline bool full_rows_fit(int log2_row_block) {
  return (size_t)4 * (((size_t)512 << log2_row_block) + 6 * 1024) <= (size_t)159 * 1024;
}
// ... and 256-byte tiles up to 128 rows
inline bool half_rows_fit(int log2_row_block) {
  return (size_t)4 * (((size_t)256 << log2_row_block) + 6 * 1024) <= (size_t)159 * 1024;
}
int tiles_per_sweep(int n_tiles, int tile_floats, int64_t n_rows, int n_launches, int sweep_kb);
int round_tiles_per_sweep(int n_tiles, int tile_floats, int64_t n_cols, int sweep_kb);

// rb_order[launch][i] = the row block with the i-th longest chunk list of that launch (order.hip).  Works on
// `stream`; *scratch_out is device memory the caller frees once the stream has drained.
sptir_status_t order_row_blocks(const int64_t* rb_chunk_ptr, int32_t n_launches, int32_t n_rb, int64_t max_list_len,
                                int32_t* rb_order, sptir_alloc_fn alloc, sptir_free_fn free_, void* actx,
                                hipStream_t stream, void** scratch_out);

// The long rows of an SDDMM plan (sddmm_slices.hip): their entries by slices of `width` columns, in segments of up to eight entries of
// one row.  n_units 0: none.
struct SddmmSlices {
  int32_t width = 0;
  int64_t nnz = 0, n_segs = 0, n_units = 0;
  int2* seg_at = nullptr;      // device
  uint4* seg_cols = nullptr;
  int4* units = nullptr;
  size_t device_bytes = 0;
};
// *rank: device memory the caller frees, NULL if no row is taken; rank[r + 1] > rank[r] where row r is
sptir_status_t sddmm_slices_build(const sptir_csr_t* csr, int32_t feat_hint, sptir_alloc_fn alloc, sptir_free_fn free_, void* actx,
                                  hipStream_t stream, SddmmSlices* out, int32_t** rank);
void sddmm_slices_free(SddmmSlices* s, sptir_free_fn free_, void* actx);
sptir_status_t sddmm_slices_run(const SddmmSlices& s, int32_t n_cols, const float* values, const float* X, const float* Yt, float* B,
                                int32_t feat, hipStream_t stream);

struct SpmmSliceBuild {               // between the parts of the build
  int32_t n_long = 0, n_blocks = 0, n_slices = 0;
  void* temporary = nullptr;
  int32_t *bound = nullptr, *count = nullptr, *order = nullptr;
  PinnedBuf host, tables;
  int64_t n_steps = 0, words = 0;
  size_t table_bytes = 0;
  int32_t *first_step = nullptr, *seq_base = nullptr;
};
int64_t slice_min_degree(int32_t n_cols);
sptir_status_t spmm_slices_count(SpmmSliceBuild* b, const sptir_csr_t* csr, int32_t min_deg, int32_t n_long, int64_t longest,
                                 sptir_alloc_fn alloc, void* actx, hipStream_t stream);
bool spmm_slices_even(const SpmmSliceBuild& b, int64_t long_nnz);
sptir_status_t spmm_slices_plan(SpmmSliceBuild* b, int32_t feat_hint, bool with_values, SpmmSlices* out, sptir_alloc_fn alloc,
                                void* actx, hipStream_t stream);
sptir_status_t spmm_slices_fill(const SpmmSliceBuild& b, const sptir_csr_t* csr, const SpmmSlices& s, hipStream_t stream);
void spmm_slices_done(SpmmSliceBuild* b, sptir_free_fn free_, void* actx);
sptir_status_t spmm_slices_gather(const SpmmSlices& s, int32_t n_cols, const float* X, int32_t feat, int32_t feat0, int32_t width,
                                  hipStream_t stream);
sptir_status_t spmm_slices_add(const SpmmSlices& s, const float* row_val, float* Y, int32_t feat, int32_t feat0, int32_t width,
                               hipStream_t stream);
// order[0 .. n_rows): the rows of at least min_len entries, longest first up to a class of length (a 255th of the logarithms
// from min_len to max_len, the longest row) and ascending inside one, then the others (order.hip).  Only enqueues work.
size_t order_rows_scratch(int32_t n_rows);
sptir_status_t order_rows_by_class(const int32_t* row_ptr, int32_t n_rows, int32_t min_len, int64_t max_len, int32_t* order,
                                   void* scratch, hipStream_t stream);

// records a failed HIP call for sptir_last_hip_error(); returns SPTIR_ERR_HIP
sptir_status_t note_hip_error(hipError_t e, const char* what);

// A launch with more than the default 64 KB of dynamic LDS has to be allowed on the device it runs on, which is the current one.
// (Where it cannot be, the launch says so.)
inline void allow_dynamic_lds(const void* kernel, size_t lds_bytes, OncePerDevice& allowed) {
  constexpr size_t kDefaultLds = 64 * 1024, kMostLds = 159 * 1024;  // (a kilobyte is for static arrays)
  int device = 0;
  if (lds_bytes <= kDefaultLds || hipGetDevice(&device) != hipSuccess) return;
  allowed(device, [&] {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMostLds) == hipSuccess;
  });
}

// text for sptir_last_hip_error() where a refusal needs more than its status code
void note_error_text(const char* text);

#define SPTIR_HIP(call)                                                   \
  do {                                                                    \
    hipError_t e_ = (call);                                               \
    if (e_ != hipSuccess) return ::sptir::note_hip_error(e_, #call);      \
  } while (0)

}  // namespace sptir

#endif  // SPTIR_INTERNAL_H_
