// Kernel-argument structs passed by value (kernarg segment) to the MSSA
// kernels.  Plain data; shared by the host launch code and the kernels.
#pragma once

#include <cstdint>

namespace mssa {

constexpr int kMaxGroups = 8;      // distinct query scales (<= num_states)
constexpr int kMaxRuns = 6;        // contiguous context runs per query scale
constexpr int kMaxPoolJobs = 16;   // pool jobs per launch

// Tile shapes of the bf16 attention kernel: 8 waves x 32 queries (two
// groups of four waves that alternate matrix-core and softmax phases), 64 keys.
constexpr int kFwdBM = 256;
constexpr int kFwdBN = 64;
constexpr int kFwdThreads = 512;
// Merge of split items: threads per block (32 queries of an item).
constexpr int kCombineThreads = 256;
// Kernels whose eight waves split the context of 32 queries (fp32 plans, and
// the bf16 forward of small layers): queries per item, waves per block.
constexpr int kFwdF32BM = 32;
constexpr int kSplitWaves = 8;
constexpr int kSplitThreads = 64 * kSplitWaves;

constexpr int kPoolThreads = 256;

// Byte offset past any buffer range the kernels build: a transfer lane pointed
// here writes zeros, a store is dropped (no 32-bit wrap of offset + 16).
constexpr uint32_t kPastEnd = 0x7ffffff0u;

struct FwdRunArgs {
  const void* k;   // first token of the run (head 0, channel 0)
  const void* v;
  int32_t n_tok;
  int32_t pad;
};

struct FwdGroupArgs {
  int32_t q_begin, q_end;   // query token range of this scale
  int32_t n_qtiles;         // ceil((q_end - q_begin) / BM)
  int32_t block_begin;      // first item (fp32 kernel: first block) of this group
  int32_t n_runs;
  int32_t tiles_per_item;   // bf16 kernel: sum over runs of ceil(n_tok / BN)
  int64_t tile_begin;       // bf16 kernel: first tile of this group in the linear tile space
  FwdRunArgs runs[kMaxRuns];
};

struct FwdArgs {
  const void* q;
  void* out;
  int64_t ld;               // elements between tokens: heads * head_dim
  int32_t n_groups;
  int32_t num_heads;
  int32_t n_blocks;
  float scale_log2e;        // softmax scale * log2(e)
  float scale;              // softmax scale
  int32_t n_ranges;         // bf16 kernel: persistent blocks
  int64_t total_tiles;      // bf16 kernel: tiles of all (group, head, query tile) items
  int64_t tail_begin;       // bf16 kernel: first tile after the whole-item rounds
  int32_t dp_rounds;        // bf16 kernel: rounds of whole items before the tail ranges
  int32_t key_splits;       // 32-query items (fp32; bf16 if > 0): blocks that share an item's context
  float* partial;           // bf16 kernel: 2 * n_ranges partial records; key_splits > 1: a record per item and split
  int64_t* range_table;     // bf16 kernel: first tile of each tail range (n_ranges + 1), written by the attention kernel
  float* lse;               // optional [heads, n_q]: log of the softmax denominator (natural log)
  int32_t n_q;
  int32_t q_prescaled;      // bf16 kernel: queries arrive multiplied by scale * log2(e)
  FwdGroupArgs groups[kMaxGroups];  // in launch order (longest context first)
};

// One partial record: unnormalised O of 256 queries (fp32, [wave][D / 4][32
// queries][4 channels]), running max m [BM] and row sum l [BM] of one piece of
// an item that spans several tile ranges.
constexpr int64_t partial_record_floats(int head_dim) { return static_cast<int64_t>(kFwdBM) * (head_dim + 2); }

// One record of an item whose context is split over key_splits blocks: O
// [32][D] (fp32, unnormalised), m [32] and l [32].
constexpr int64_t split_record_floats(int head_dim) { return 32 * static_cast<int64_t>(head_dim + 2); }

// ---------------------------------------------------------------- backward

// bf16 backward kernels: 8 waves of 32 queries (dQ kernel), 4 waves of 32 or 64
// keys, one per SIMD (dK/dV kernel); the other operand streams through LDS in
// stages.
constexpr int kBwdQ = 256;     // dQ kernel: queries per block (8 waves x 32)
constexpr int kBwdQThreads = 512;   // dQ kernel: 8 waves, two per SIMD
constexpr int kBwdKS = 64;     // dQ kernel: keys per LDS stage (and per dS tile)
constexpr int kBwdKVKeys = 128;     // dK/dV kernel: keys per block with 32 a wave, twice as many with 64 (BwdArgs::kv_keys)
constexpr int kBwdKVThreads = 256;  // dK/dV kernel: 4 waves
constexpr int kBwdQS = 64;     // dS tiles: queries are rounded up to this
constexpr int kBwdStage = 32;  // dK/dV kernel: queries per LDS stage
constexpr int64_t kBwdDsBudget = int64_t(8) << 30;  // bytes of dS tiles held at once (whole heads, at least one)
constexpr int kBwdF32 = 32;    // fp32 kernels: queries (dQ) or keys (dK, dV) per block
constexpr int kDotThreads = 256;
constexpr int kMaxScatterJobs = 10;

struct BwdGroupArgs {
  int32_t q_begin, q_end;     // query token range of this scale
  int32_t n_kv;               // context tokens
  int32_t n_runs;
  int32_t dq_block_begin;     // first block of the group in the dQ grid (head-major inside)
  int32_t kv_block_begin;     // first block of the group in the dK/dV grid
  int32_t n_qblocks;          // dQ blocks per head
  int32_t n_kblocks;          // dK/dV blocks per head
  FwdRunArgs runs[kMaxRuns];  // context runs (K, V source tokens), context order
  float* dk_ctx;              // [n_kv, heads * head_dim] fp32 context gradients
  float* dv_ctx;
  void* ds;                   // bf16: dS tiles [launch heads][ds_qblocks][ds_stages][64 keys][32 queries]
  int32_t ds_stages;          // 64-key stages of the runs (each run starts a stage)
  int32_t ds_qblocks;         // 32-query blocks (even)
  int32_t dq_splits;          // bf16 dQ kernel: blocks that share the context of 256 queries
  int32_t pad;
};

struct BwdArgs {
  const void* q;
  const void* d_out;
  const float* lse;         // [heads, n_q] from the forward
  float* dsum;              // [heads, n_q]: -rowsum(d_out * out), written by dot_kernel
  float* lse2;              // [heads, n_q]: -lse / scale, in units of q k^T (bf16), written by dot_kernel
  void* dq;
  int64_t ld;               // elements between tokens: heads * head_dim
  int32_t n_q;
  int32_t num_heads;        // heads of this launch: head0 .. head0 + num_heads - 1
  int32_t head0;            // first head of this launch (the dS tiles hold these heads)
  int32_t n_groups;
  float scale;              // softmax scale
  float scale_log2e;
  int32_t q_prescaled;      // queries arrive multiplied by scale * log2(e)
  int32_t dq_blocks;        // bf16 dQ kernel: blocks per split (set by the launcher)
  int32_t kv_keys;          // bf16 dK/dV kernel: keys per block
  int32_t pad;
  BwdGroupArgs groups[kMaxGroups];  // longest query range first
};
static_assert(sizeof(BwdArgs) <= 4096, "kernel argument block");

struct DotArgs {
  const void* out;
  const void* d_out;
  float* dsum;              // [heads, n_q]: -rowsum(d_out * out)
  const float* lse;         // [heads, n_q] natural log (bf16 plans; may be null)
  float* lse2;              // [heads, n_q] -lse / scale: minus the row max of q k^T (written when lse is set)
  int64_t ld;
  int32_t n_q;
  int32_t num_heads;
  int32_t head_dim;
  float inv_scale;          // 1 / the natural-log score factor
};

// One run of source frames (sink, history, or window frames of one scale)
// whose gradient gathers from every query scale's context gradient: frame f
// of the job sits in group g's context at token ctx_begin + f * frame_stride,
// resampled by factor.
struct ScatterGroupArgs {
  int64_t ctx_begin;
  int32_t frame_stride;
  int32_t factor;
};

struct ScatterJobArgs {
  void* dst_k;              // gradient of the job's first source token (head 0, channel 0)
  void* dst_v;
  int32_t n_frames;
  int32_t gh, gw;           // source grid
  int32_t block_begin;
  ScatterGroupArgs g[kMaxGroups];
};

struct ScatterArgs {
  const float* ctx_k[kMaxGroups];
  const float* ctx_v[kMaxGroups];
  int64_t ld;
  int32_t chunks_per_tok;   // output chunks per token: 8 elements (bf16) or 4 (fp32)
  int32_t n_jobs;
  int32_t n_groups;
  int32_t pick_first;       // strided resampling: only each block's first cell
  ScatterJobArgs jobs[kMaxScatterJobs];
};

// ---------------------------------------------------------------- MSP tiers

constexpr int kTierThreads = 256;
// Output tile (rows x features) and K stage of the 4-wave GEMM kernels.
constexpr int kGemmTile = 128, kGemmStage = 64;

// Patch rows of consecutive latent frames of one tier: frame frame0 + f of
// `latent` [frames, C, H, W] <-> rows [(f * gh + Y) * gw + X][C * P * P].
struct PatchArgs {
  void* latent;
  void* rows;
  int64_t frame0;
  int64_t n_frames;
  int32_t C, H, W, P;
  int32_t gh, gw;
};

// Y = X W^T + b: X [M, K] (row stride ldx), W [N, K] dense, b [N]; output
// feature j goes to y[j / split] at column j % split (row stride ldy).
struct GemmArgs {
  const void* x;
  const void* w;
  const void* bias;
  void* y[3];
  int32_t M, N, K;
  int32_t split;
  int64_t ldx, ldy;
  float* partial;     // k_splits > 1: fp32 partial tiles of every K slice (launch_gemm_split)
  int32_t k_splits;   // 0 or 1: the whole K in one block
  float y0_scale;     // factor on the outputs of y[0] (columns < split), applied to the fp32 sum before rounding
};

// Tiers whose GEMM gathers its rows from the latent (embedding) or scatters
// its outputs to it (de-embedding), in one launch (launch_tiers).
struct TierProblem {
  const void* x;      // de-embedding: tokens [M, K]
  const void* w;      // [N, K]
  const void* bias;   // [N]
  void* y;            // embedding: tokens [M, N]
  PatchArgs patch;    // rows not used
  int32_t M, N, K;
  int32_t block_begin;      // (set by tier_blocks)
  int32_t tiles_per_block;  // embedding: feature tiles of one block (set by tier_blocks)
};
struct TierArgs {
  TierProblem g[kMaxGroups];
  int32_t n;
};
constexpr int kEmbedTile = 64;    // rows of a block and features of a wave's step of the fused embedding
constexpr int kEmbedMaxK = 256;   // its longest K
constexpr int kUnembedTile = 64;  // output tile (rows and features) of the fused de-embedding

struct PoolJobArgs {
  const void* src_k;        // first source token of the job (head 0, ch 0)
  const void* src_v;
  void* dst_k;              // first destination token of the job (pooled by factor)
  void* dst_v;
  void* dst2_k;             // levels == 2: first destination token pooled by 2 * factor
  void* dst2_v;
  int32_t src_gh, src_gw;
  int32_t dst_gh, dst_gw;
  int32_t dst2_gh, dst2_gw;
  int32_t factor;
  int32_t levels;           // 1, or 2: the same source frames pooled by factor and by 2 * factor
  int32_t n_frames;
  int32_t block_begin;
};

struct PoolArgs {
  int64_t ld;               // elements between tokens
  int32_t chunks_per_tok;   // 16-byte chunks per token (all heads)
  int32_t n_jobs;
  int32_t pick_first;       // 1: copy each block's first cell (stride); 0: block mean
  int32_t pad;
  PoolJobArgs jobs[kMaxPoolJobs];
};

}  // namespace mssa
