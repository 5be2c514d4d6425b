// Launchers behind the C ABI.  Each takes validated arguments, enqueues its kernels on
// `stream` and returns the hipError_t of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mts_attn_rules.hpp"
#include "mts_layout.hpp"

namespace mts {

// records the calling thread's error text (what mts_last_error returns) and returns `code`
int32_t set_error(int32_t code, const char* fmt, ...);

struct BatchDev {            // device metadata arrays, as in mts_batch_meta
  int32_t        batch;
  const int32_t* page_indptr;
  const int32_t* page_indices;
  const int32_t* prefix_lens;
  const int32_t* new_indptr;
  int32_t        total_new;
  int32_t        max_new;
  int32_t        max_total_len;
  int32_t        total_pages;
};

// What a kernel's first loads need comes first among its arguments: the compiler is told to have up to 14 words of such
// arguments in scalar registers when a wavefront starts (vectors and scalars, not structures), so that the tables'
// loads do not wait until the arguments have come from memory; those behind them travel beside the tables.  A kernel
// that is a chain of round trips gets 0.3 us shorter: 8 layers of one user's 32 new tokens behind 6375 x 4 heads of 128,
// 24 launches, 152.1 -> 143.9 us; 64 users x 8 heads of 64, 4 layers, 230.2 -> 228.9.  (Not the prefill kernel's: its registers
// are full, 442 -> 444 us for one user's 5189 tokens, where without it 439.)  As vectors and few structures, because every argument
// costs the host at a launch: with each table an argument, 2 layers of 16 queries x 272 keys x 4 heads of 32 in fp32, four
// launches that the host is the limit of, 21.4 -> 22.2 us; as it is, 21.3.
typedef uint64_t TableWords __attribute__((ext_vector_type(2)));   // addresses of two tables
typedef int32_t CallWords __attribute__((ext_vector_type(4)));
typedef int32_t CallWords2 __attribute__((ext_vector_type(2)));
inline TableWords table_words(const void* a, const void* b) { return TableWords{(uint64_t)(uintptr_t)a, (uint64_t)(uintptr_t)b}; }
inline TableWords run_tables(const BatchDev& b) { return table_words(b.new_indptr, b.prefix_lens); }
inline TableWords page_tables(const BatchDev& b) { return table_words(b.page_indptr, b.page_indices); }
// (by way of the global address space, so that loads through it are global ones)
__device__ __forceinline__ const int32_t* table(uint64_t address) {
  return (const int32_t*)(const __attribute__((address_space(1))) int32_t*)address;
}

// Inclusive sums over the 64 lanes of a wavefront, all of them active: six additions that read other lanes on the way (six
// shuffles through LDS took 0.25 us more of every launch that schedules itself: 8 layers of one user's 32 new tokens behind
// 6375 x 4 heads of 128 133.6 -> 131.7 us).
__device__ __forceinline__ int scan_lanes(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8: inside 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast 15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast 31 into rows 2 and 3
  return v;
}

struct SegDev {              // segment lists of unpack / pack
  int32_t        num_segs;
  const int32_t* seg_user;
  const int32_t* seg_pos;
  const int64_t* seg_tok_indptr;
  int32_t        max_seg_tokens;
};

// `layers` consecutive layers starting at g.layer_base in one launch: layer i of the pool lies
// i * pool_layer_stride bytes further, its runs i * staging_layer_stride bytes further.
hipError_t launch_unpack(const PoolGeom& g, const void* staging, const SegDev& segs, const BatchDev& b,
                         hipStream_t stream, int layers = 1, int64_t pool_layer_stride = 0,
                         int64_t staging_layer_stride = 0);
hipError_t launch_pack(const PoolGeom& g, void* staging_out, const SegDev& segs, const BatchDev& b,
                       hipStream_t stream, int layers = 1, int64_t pool_layer_stride = 0,
                       int64_t staging_layer_stride = 0);
hipError_t launch_append(const PoolGeom& g, const void* k_new, const void* v_new, const BatchDev& b,
                         hipStream_t stream, int layers = 1, int64_t pool_layer_stride = 0,
                         int64_t rows_layer_stride = 0);

// Shape plan of one attention call: computed on the host from the scalar bounds only.
struct AttnPlan {
  bool    use_mfma;      // bf16 matrix-core kernels; with neither this nor use_f32, the plain kernel
  bool    use_f32;       // fp32 matrix-core kernel
  bool    use_prefill;   // workgroup-per-query-block kernel for long new segments (workspace optional)
  bool    too_large;     // more (user, query tile) items than the schedule can hold
  int32_t q_tile;        // queries per query tile (multiple of 16, <= 64)
  int32_t q_tiles_max;   // ceil(max_new / q_tile)
  int32_t n_items;       // batch * q_tiles_max
  int32_t min_tiles;     // least kv tiles a wavefront's share may hold
  int32_t pair_cost;     // schedule allowance per (query tile, head), in tiles
  int32_t staged_tile_cost; // what a kv tile in the onload buffer counts, in tiles of the pool
  int32_t max_waves;     // most wavefronts the launch may use (sizes the partial buffers)
  int64_t ws_desc_bytes; // per-wavefront merge descriptors at the start of the workspace
  int64_t ws_bytes;      // whole workspace
  int64_t ws_required;   // what the call cannot do without (the rest only lets it split further)
  bool    past_caches;   // streaming kernel: K/V tiles are loaded past the caches' retention
  int32_t piece_wgs;     // streaming kernel: workgroups of a launch of one piece each, 0 = even shares of wavefronts
  int32_t piece_tiles;   // ... most kv tiles of such a piece, 0 = (query tile, head)s are not cut
  int32_t prefill_wgs;   // prefill kernel: workgroups of a split launch, 0 = one per query block
};
// Fits the plan to the workspace that the caller handed over (any pointer, any size).
void fit_plan_to_workspace(AttnPlan& p, const PoolGeom& g, const void* workspace, int64_t workspace_bytes);
constexpr int kPrefillMaxWgs = 512;          // 256 CUs x 2 resident workgroups
constexpr int kPrefillSplitMaxBatch = 1024;  // users in the schedule of a split launch: 16 a lane
// `layers` of the cache; the call's kind chooses between forms of the same workspace
AttnPlan plan_attention(const PoolGeom& g, const BatchDev& b, int layers, StreamCall call = StreamCall::kSoftmax);
constexpr int kAttnMaxWaves = 1024;   // 256 CUs x 4 SIMDs: one wavefront per SIMD


// inv_norm selects the aggregation: 0 = softmax (Sec. 2, Eq. 6-7); > 0 = pointwise,
// out = inv_norm * sum_j silu(sm_scale * q.k_j) v_j (no softmax statistics).
hipError_t launch_attn_generic(const PoolGeom& g, const void* q, void* out, const BatchDev& b,
                               float sm_scale, float inv_norm, hipStream_t stream);
hipError_t launch_attn_f32(const PoolGeom& g, const void* q, void* out, const BatchDev& b, float sm_scale,
                           float inv_norm, hipStream_t stream);
bool attn_prefill_applicable(const PoolGeom& g, const BatchDev& b);
int attn_prefill_block(const PoolGeom& g);
hipError_t launch_attn_prefill(const PoolGeom& g, const AttnPlan& plan, const void* q, void* out, const BatchDev& b,
                               float sm_scale, float inv_norm, void* workspace, hipStream_t stream);
// Prefixes still in the contiguous onload buffer (device arrays; see mts_attn_incremental_staged).
struct StagedHistories {
  const void*    rows;        // the layer's runs, [2][n][H][D] each
  const int32_t* first_run;   // [batch]: first run of user u's prefix, -1 = prefix in the pool
  const int64_t* run_tok;     // [runs + 1]: token offset of every run in `rows`
  int32_t        chunk;       // tokens per run (the last run of a user may be shorter)
};

// k_new / v_new non-NULL: this step's K/V rows ([token][H][D]) are read from there and the
// pool's slots for them are not touched, so the layer's append need not have happened; with
// `hist`, the prefixes of the users it names are read from the onload buffer as well.
hipError_t launch_attn_mfma(const PoolGeom& g, const AttnPlan& plan, const void* q, void* out,
                            const BatchDev& b, float sm_scale, float inv_norm, void* workspace,
                            hipStream_t stream, const void* k_new = nullptr, const void* v_new = nullptr,
                            const StagedHistories* hist = nullptr);

}  // namespace mts
