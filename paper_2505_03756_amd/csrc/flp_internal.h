// Internal declarations shared by the host logic (pool.cpp, dispatch.cpp) and the
// kernel translation units.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <mutex>
#include <vector>

#include "flpool.h"

void flp_set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));

#define FLP_TRY_HIP(expr)                                                                        \
  do {                                                                                           \
    hipError_t e_ = (expr);                                                                      \
    if (e_ != hipSuccess) {                                                                      \
      flp_set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__);  \
      return FLP_EHIP;                                                                           \
    }                                                                                            \
  } while (0)

#define FLP_TRY(expr)            \
  do {                           \
    flp_status s_ = (expr);      \
    if (s_ != FLP_OK) return s_; \
  } while (0)

// LIFO free list of one tier.
struct FlpFreeList {
  int64_t n = 0;
  std::vector<int32_t> stack;     // stack.back() is handed out next
  std::vector<uint8_t> is_free;
  std::vector<uint32_t> stamp;    // scratch for duplicate detection
  uint32_t gen = 0;
};

// One slot of the ring that carries small host arrays (id lists, work lists) to the
// device: pinned host buffer + device mirror + the event that marks the slot's last use.
struct FlpStageSlot {
  void* host = nullptr;
  void* dev = nullptr;
  size_t cap = 0;
  hipEvent_t ev = nullptr;
  bool in_flight = false;
};

constexpr int kStageSlots = 16;

struct flp_pool {
  flp_pool_config cfg{};
  int elem_bytes = 0;
  int64_t block_elems = 0;
  int64_t block_bytes = 0;
  int device = 0;
  uint8_t* dev_base = nullptr;
  uint8_t* host_base = nullptr;
  bool own_dev = false, own_host = false;
  bool host_tier_in_hbm = false;  // the caller placed the "host" tier in device memory
  FlpFreeList tier[2];
  FlpStageSlot stage[kStageSlots];
  int stage_next = 0;
  void* work = nullptr;           // device workspace (LoRA intermediates), grown on demand
  size_t work_cap = 0;
  void* attn_work = nullptr;      // device workspace of the attention call (split-KV partial results)
  size_t attn_work_cap = 0;
  FlpStageSlot* attn_slot = nullptr;   // its event follows the last call that used attn_work, which ran on attn_stream
  hipStream_t attn_stream = nullptr;
  void* dense_work = nullptr;          // slices of a layer's dense products without LoRA, batches of more than 1024 tokens
  size_t dense_work_cap = 0;
  hipEvent_t dense_ev = nullptr;       // follows the last use of dense_work, which was on dense_stream
  hipStream_t dense_stream = nullptr;
  std::vector<void*> retired;     // outgrown workspace buffers, freed with the pool
  mutable std::mutex mu;          // guards the free lists, the staging slots and the workspace
};

// Staging: acquire a slot with room for `bytes` (waits for the slot's previous use),
// fill slot->host, then flp_stage_upload() copies to slot->dev on the stream; after the
// consuming kernels are enqueued call flp_stage_release().
flp_status flp_stage_acquire(flp_pool* pool, size_t bytes, FlpStageSlot** slot);
flp_status flp_stage_upload(FlpStageSlot* slot, size_t bytes, hipStream_t stream);
flp_status flp_stage_release(FlpStageSlot* slot, hipStream_t stream);
flp_status flp_workspace(flp_pool* pool, size_t bytes, void** out);
// a workspace for slices of dense products that is handed from call to call, also between streams (with the pool's lock held)
flp_status flp_dense_workspace_acquire(flp_pool* pool, size_t bytes, hipStream_t stream, void** out);
flp_status flp_dense_workspace_release(flp_pool* pool, hipStream_t stream);
// the host-side checks of flp_pool_swap_in (src_tier 1) / flp_pool_swap_out (src_tier 0) without enqueuing anything
flp_status flp_swap_check(flp_pool* pool, int32_t n, const int32_t* src_ids, const int32_t* dst_ids, int src_tier,
                          const char* who);

// A workspace of fixed size that the caller of the LoRA path brings along instead of the pool's growing one:
// `resolve` returns its device address for the pool's device (called only after the size check has passed).
struct FlpFixedWorkspace {
  size_t cap;
  flp_status (*resolve)(flp_pool* pool, void** out);
  const char* who;
};
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;   // what flp_lora_apply_paged_static has per GPU
constexpr size_t kLayerSliceBytes = (size_t)1 << 30;       // what slices of a layer's dense products may take
// flp_lora_apply_paged with its intermediates in `ws` (no allocation, no growth)
flp_status flp_lora_apply_fixed(flp_pool* pool, const flp_lora_batch* batch, void* hip_stream, const FlpFixedWorkspace& ws);
// The sequences that a layer's tokens come in, which as a rule have one adapter each: sequence i is the tokens cu[i] .. cu[i + 1] - 1
// of the layer's batch (host memory, as the caller passed it), and a LoRA call works on `first` and those behind it.  They decide
// between forms of the LoRA steps that differ in speed and in the order of sums, not in the bits that v is held in.
struct FlpSequences {
  const int32_t* cu;
  int32_t n, first;
};
// flp_lora_apply_paged for the layer step, whose larger slice room only the pool's growing workspace has
flp_status flp_lora_apply_layer(flp_pool* pool, const flp_lora_batch* batch, const FlpSequences& seqs, void* hip_stream);
// which steps a layer's call takes, for tests: FLP_LORA_*
enum { FLP_LORA_TOKENS = 0, FLP_LORA_TOKENS_LONG, FLP_LORA_SORTED, FLP_LORA_IN_PRODUCT };
extern "C" int32_t flp_lora_layer_route(int32_t dtype, int32_t n_tokens, int32_t d_in, int32_t n_proj, const int32_t* d_out,
                                        int32_t max_rank, int32_t n_seqs, const int32_t* cu, int32_t first);
// set-up of the file-scope scratch array for the current device (looks its device address up once per device);
// called when a pool is created, and again by the entry point that uses the array if that first attempt failed
flp_status flp_static_scratch_setup(int device, void** out);

// ---- kernel launchers (defined in the .hip files) ---------------------------------------
flp_status flp_launch_copy_blocks(const uint8_t* src_base, uint8_t* dst_base, const int32_t* src_ids_dev,
                                  const int32_t* dst_ids_dev, int32_t n, int64_t block_bytes,
                                  int host_link, hipStream_t stream);
// host_link: which side of the copy is the pinned host tier, and how wide the caller wants the launch
enum { FLP_LINK_NONE = 0, FLP_LINK_IN = 1, FLP_LINK_OUT = 2, FLP_LINK_IN_DUPLEX = 3, FLP_LINK_OUT_DUPLEX = 4,
       FLP_LINK_IN_NARROW = 5, FLP_LINK_OUT_NARROW = 6 };
// flp_pool_swap_in / flp_pool_swap_out (src_tier 1 / 0) for a caller that knows what runs beside the move: one
// direction alone, both directions together, or moves that need not hurry
enum { FLP_WIDTH_SINGLE = 0, FLP_WIDTH_DUPLEX = 1, FLP_WIDTH_NARROW = 2 };
flp_status flp_swap_width(flp_pool* p, int32_t n, const int32_t* src_ids, const int32_t* dst_ids, int src_tier,
                           void* hip_stream, int width);

flp_status flp_launch_stage_copy(const void* src_pinned, void* dst_dev, size_t bytes, hipStream_t stream);

// Kernels work on groups of 16 token positions; a block of 32 positions is two such groups (group index
// gi = position / 16 lives in block gi / (bt / 16), at slots 16 * (gi % (bt / 16)) ...).
struct FlpAppendUnit {   // the slots [s0, s1) of the 16-position group `blk_idx` of sequence `seq`
  int32_t seq, blk_idx, s0, s1, t_first, pad0, pad1, pad2;
};
struct FlpAttnUnit {     // new tokens t .. t + n_tok - 1 of sequence `seq`; positions 0 .. ctx - 1 are visible to the first one
  int32_t seq, t, n_tok, ctx;
  // part >= 0 (split-KV, long contexts): the unit is ONE token and its unnormalised result is piece `part` of the
  // partials buffer.  The unit covers the 16-position groups [g_lo, g_hi) of the context (row kernel: only where it is split)
  int32_t g_lo, g_hi, part, pad;
};

// query rows [r0, r0+n_rows) of (sequence, kv head g); n_rows == 0: padding; n_rows < 0: single tokens, the pairs r0 .. r0 + 7 of
// `seq` (unit, kv head) pairs of the decode list, a wave each
struct FlpMfmaItem {
  int32_t seq, g, r0, n_rows;
};

struct FlpAttnArgs {
  uint8_t* pool;
  int64_t block_elems;
  const int32_t* tables;
  int32_t max_blocks;
  int32_t n_h, n_kv;
  int32_t bt;                  // token positions per block: 16 or 32
  const void* q;
  void* out;
  const void* k_new;
  const void* v_new;
  const int32_t* cu_new;       // device copies
  const int32_t* prefix_len;
  float scale_log2e;
  float* partials;             // split-KV: [piece][n_h][head_dim + 2] fp32 (running max, sum, channels)
};

// Every unit is read by flp_kv_append_columns workgroups, from pinned host memory or the device; beside them the launch copies
// copy_bytes (rounded up to 16) of the attention call's lists from pinned memory to their device mirror.
int flp_kv_append_columns(int dtype, int n_kv, int head_dim);
flp_status flp_launch_kv_append(int dtype, int head_dim, const FlpAttnArgs& a, const FlpAppendUnit* units, int32_t n_units,
                                const void* copy_src, void* copy_dst, size_t copy_bytes, hipStream_t stream);
flp_status flp_launch_attn_rows(int dtype, int head_dim, const FlpAttnArgs& a, const FlpAttnUnit* units_dev,
                                int32_t n_units, hipStream_t stream);
// single new tokens on the matrix cores: 16-bit pools, head_dim 128, n_h / n_kv <= kDecodeMaxGroup; every unit is ONE token
// with its groups [g_lo, g_hi) filled in
constexpr int kDecodeMaxGroup = 16;
flp_status flp_launch_attn_decode(int dtype, const FlpAttnArgs& a, const FlpAttnUnit* units_dev, int32_t n_units,
                                  hipStream_t stream);
// split-KV: one merged row per (row of the lists, head): token t = merge_tok[row], the merge_first[row + 1] -
// merge_first[row] <= 64 pieces from merge_first[row] on combined in piece order (so the result does not depend on
// which piece finished first)
flp_status flp_launch_attn_merge(int dtype, int head_dim, const FlpAttnArgs& a, const int32_t* merge_tok_dev,
                                 const int32_t* merge_first_dev, int32_t n_rows, hipStream_t stream);
// the workspace of an attention call that splits, for work on `stream`: a call on another stream waits for the one before it
// (the caller owes no ordering to calls whose sequences are different ones, and cannot see which of them split)
flp_status flp_attn_workspace(flp_pool* pool, size_t bytes, hipStream_t stream, void** out);

flp_status flp_launch_attn_mfma(int dtype, const FlpAttnArgs& a, const FlpMfmaItem* items_dev, int32_t n_items,
                                const FlpAttnUnit* units_dev, hipStream_t stream);
// how single tokens run beside tiles on a 16-bit pool with head_dim 128, for tests: 0 a launch of their own, 1 behind the tiles, 2 between them
extern "C" int32_t flp_attention_route(int32_t n_q_heads, int32_t n_kv_heads, int32_t block_tokens, int32_t n_seqs, const int32_t* cu,
                                       const int32_t* prefix);
constexpr int kMfmaRowsPerItem = 256;
constexpr int kMfmaMaxBlocks = 4096;       // longest context of the matrix-core kernel: 65536 positions

struct FlpLoraArgs {
  const uint8_t* pool;
  int64_t block_elems;
  int32_t T, d_in, n_adapters, max_rank, n_proj;
  int64_t ld_x;
  const void* x;
  const int32_t* token_adapter;
  const int32_t* rank;
  const float* scale;
  const int32_t* tables;
  flp_lora_proj proj[FLP_MAX_PROJ];
  // unrounded base term x.W_base [T, d_out] of a projection whose w_base was given (16-bit pools), else null:
  // the expand kernels then take the base from here instead of y and round base + delta once
  const float* base32[FLP_MAX_PROJ];
  int32_t base_slices[FLP_MAX_PROJ];   // slices of it, T * d_out apart (more than one: lora_small.hip only)
  // workspace
  float* v;                    // [T, n_proj, max_rank] fp32
  int32_t* n_seg;
  int32_t* seg_adapter;
  int32_t* seg_start;
  int32_t* perm;
  int32_t* tile_start;         // [n_seg + 1] first tile of each segment (matrix-core kernels)
  int32_t* group_start;        // [n_seg + 1] first tile group of each segment (expand kernel)
};

struct FlpLoraMfma {
  int32_t mt;                  // 16-token tiles per work item (1 or 2)
  int32_t k_splits, k_per_split;
  int32_t v_rows;              // rows of one split's partial v buffer (= tiles_bound * 16 * mt)
  int32_t tiles_bound;         // host-side upper bound of the number of tiles (sizes the v buffer)
  int32_t tiles_grid;          // tiles the shrink launch covers in one pass (multiple of 8); more are looped over
  int32_t group_tokens;        // tokens per tile group of the expand kernel (multiple of 16*mt)
  int32_t groups_bound;
  int32_t groups_grid;         // tile groups the expand launch covers in one pass (multiple of 8)
  int32_t slabs;               // slabs of 256 columns per projection (set by the launcher)
  int32_t shrink_only;         // 1: stop after the shrink step (the expand step runs inside the dense product)
};

// Batches of up to kLoraSmallTokens tokens (lora_small.hip): v is [k_splits][T][n_proj][16 n_tiles] by token, and the shrink step
// leaves a record per token: how many tokens of its adapter it works for (0: none), which, and what the adapter is.
constexpr int kLoraSmallTokens = 1024;
struct FlpLoraGroup {
  int32_t n, r;
  float scale;
  int32_t pad;
  int32_t tok[16];
  int32_t tab[FLP_MAX_PROJ], row[FLP_MAX_PROJ];      // where the projections' B lies: offset into the tables, first page row
};
constexpr int kLoraLongBlock = 8;      // neighbouring tokens that a wave of the expand step may take
struct FlpLoraSmall {
  int32_t k_splits, n_tiles;   // slices of d_in; tiles of 16 ranks
  bool long_runs;              // the expand step takes kLoraLongBlock neighbouring tokens per wave (one or two rank tiles)
  FlpLoraGroup* groups;        // [T]
};

// What the large-batch dense product needs to add one projection's LoRA branch to its accumulators before it
// rounds (the expand step as an epilogue: y = round(x . W + s (x A^T) B), no fp32 copy of the product, no second
// pass over y).  v is the shrink step's output, rows in segment order: token t of adapter a sits in row
// vrow_base[a] + inv_perm[t] (both written by the segmentation kernel).
struct FlpGemmLora {
  const int32_t* token_adapter;
  const int32_t* rank;
  const float* scale;
  const int32_t* tables;
  const int32_t* b_tab_off;    // this projection's
  const int32_t* b_row_base;
  const void* pool;
  int64_t block_elems;
  const float* v;              // [k_splits][v_rows][n_proj][rp] fp32
  int32_t v_rows, k_splits, n_proj, p, rp;
  int32_t n_adapters, max_rank;
  const int32_t* inv_perm;     // [T] token -> position in segment order
  const int32_t* vrow_base;    // [n_adapters]
};

flp_status flp_launch_lora_segment(int32_t T, const int32_t* token_adapter, int32_t n_adapters, int32_t* n_seg,
                                   int32_t* seg_adapter, int32_t* seg_start, int32_t* perm, int32_t tm,
                                   int32_t* tile_start, int32_t tg, int32_t* group_start, hipStream_t stream,
                                   int32_t* inv_perm = nullptr, int32_t* vrow_base = nullptr);
flp_status flp_launch_lora_mfma(int dtype, const FlpLoraArgs& a, const FlpLoraMfma& c, hipStream_t stream);
flp_status flp_launch_lora_simple(int dtype, const FlpLoraArgs& a, hipStream_t stream);
flp_status flp_launch_lora_small(int dtype, const FlpLoraArgs& a, const FlpLoraSmall& c, hipStream_t stream);   // d_in % 64 == 0

// ---- dense products (gemm.hip): up to FLP_MAX_PROJ matrices [N, K] over one input, 16-bit types
enum { FLP_GEMM_64x32 = 0, FLP_GEMM_128x64, FLP_GEMM_128x128, FLP_GEMM_256x128, FLP_GEMM_256x256, FLP_GEMM_KINDS };
struct FlpGemmPlan {
  int kind;                    // tile, features x tokens
  int splits;                  // slices of the contraction
  float us;                    // what the planner reckons with, the launch that adds slices included
};
struct FlpGemmOut {
  const void* w;               // [N, K]
  const void* w2;              // gated pair: the up matrix (w is the gate matrix), each [N / 2, K]
  void* y;                     // rounded result (with several slices: written by flp_launch_gemm_reduce), or null
  int64_t ld_y;
  float* part;                 // unrounded slices [splits][M][N], or null (only with one slice)
  int32_t N;
};
struct FlpGemmProj {           // the kernel's view of one FlpGemmOut
  const uint16_t* w;
  const uint16_t* w2;
  uint16_t* y;
  int64_t ld_y;
  float* part;
  int32_t N, tile0;            // tile0: first feature tile of this projection
};
struct FlpGemmArgs {
  const uint16_t* x;
  int64_t ld_x;
  int32_t M, K, n_proj, f_tiles, m_tiles, splits;
  int32_t gf, bands;           // tiles that run next to each other on one XCD: gf (feature tile, slice) units x a band of token tiles
  FlpGemmProj proj[FLP_MAX_PROJ];
};
enum { FLP_GEMM_NO_SPLIT = 1, FLP_GEMM_LARGE_ONLY = 2 };   // whole contractions only; only the tiles that take a LoRA epilogue
// N: features of every projection (of a gated pair: both matrices' together)
FlpGemmPlan flp_gemm_plan(int M, int K, int n_proj, const int* N, unsigned allow, size_t max_part_bytes);
// the same through the C ABI, for tests that state which tile and how many slices a shape gets; room < 0: a layer's
extern "C" void flp_dense_plan(int32_t M, int32_t K, int32_t n_proj, const int32_t* N, int32_t large_only, int64_t room,
                               int32_t* kind, int32_t* splits);
// which unit (feature tile, slice) and token tile a workgroup of a launch takes, for tests; 0: none
extern "C" int32_t flp_dense_tile(int32_t block, int32_t n_units, int32_t m_tiles, int32_t* u, int32_t* tm);
// rows of x this far apart can be addressed inside a tile of this kind
bool flp_gemm_offsets_fit(int kind, int M, int64_t ld_x);
size_t flp_gemm_part_bytes(const FlpGemmPlan& plan, int M, int n_proj, const int* N);
// lora: one per projection (gated: gate, up), or null
flp_status flp_launch_gemm(int dtype, const void* x, int64_t ld_x, int M, int K, const FlpGemmPlan& plan, int n_proj,
                           const FlpGemmOut* out, bool gated, const FlpGemmLora* lora, hipStream_t stream);
// adds the slices; KEEP: the unrounded sum stays in slice 0; ADD: the rounded sum is added to what `y` holds (not gated)
enum { FLP_REDUCE_PLAIN = 0, FLP_REDUCE_KEEP, FLP_REDUCE_ADD };
flp_status flp_launch_gemm_reduce(int dtype, int M, int n_proj, const FlpGemmOut* out, int splits, bool gated, int mode,
                                  hipStream_t stream);
flp_status flp_launch_transpose16(const void* w, void* wt, int K, int N, hipStream_t stream);   // [K, N] -> [N, K]
flp_status flp_launch_gemm_f32(const float* x, int64_t ld_x, const float* w, int w_layout, float* y, int64_t ld_y, int M, int N,
                               int K, hipStream_t stream);
// flp_lora_apply_paged for exactly two projections with dense bases stored [d_out, d_in] and equal widths (gate and
// up of an MLP), whose results are not stored: out = silu(y0) * y1 in one pass of the large-batch GEMM, each product
// with its LoRA branch added before it is rounded.  FLP_ENOTSUP, nothing launched, when the batch is not one that
// this path takes; the caller then runs flp_lora_apply_layer and the element-wise step.
flp_status flp_lora_apply_gated(flp_pool* pool, const flp_lora_batch* batch, const FlpSequences& seqs, void* out, int64_t ld_out,
                                void* hip_stream);
