// Host-side declarations shared by the translation units of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fff {

// One FFF call, as validated by the C ABI.
struct Problem {
    const void* x;
    const void* node_w;
    const void* node_b;
    const void* leaf_w1;
    const void* leaf_b1;
    const void* leaf_w2;
    const void* leaf_b2;
    void* out;
    int32_t* leaf_idx;
    int64_t T, D, O;
    int depth, L, act;
    bool bf16;
};

// Per-device scratch, carved out of one allocation (all int32 words).
struct Workspace {
    int32_t* leaf_idx;   // [T]      when the caller passes none
    int32_t* rank;       // [T]      rank of a token among same-leaf tokens of its chunk
    int32_t* slot_leaf;  // [T]      leaf of every slot of perm
    int32_t* perm;       // [T]      token ids grouped by leaf
    int32_t* count;      // [NL]
    int32_t* offset;     // [NL + 1]
    int32_t* tile_off;   // [NL + 1] exclusive prefix of per-leaf tile counts
    int32_t* chunk_cnt;  // [C, NL]  per-chunk histograms, then per-chunk bases
    int32_t* fold;       // [kFoldWords] per-block leaf counts of the descent (DescentCounts::M)
    int32_t* hidden;     // [16 T]   hidden activations of the tile path, T * L bf16 (L <= 32)
    int32_t* extra;      // caller-specific region (gating candidates of the mixture of experts)
    int32_t* ctrl;       // [16]     ticket counters and totals
    int64_t n_chunks;
};

constexpr int kChunkTokens = 256;   // tokens per bucketing chunk
constexpr int kTileRows = 16;       // rows of one MFMA tile
constexpr int kTilesMaxLeafWidth = 32;   // widest leaf the MFMA tile path takes

bool vec_ok(const void* p, int64_t row_elems, bool bf16);

// Every launch function names the kernel it starts, with the tile parameters that select the
// instantiation ("walk_kernel<bf16,16,6,4,512,fused,tight>"); a forward call's names, joined by
// " + ", are what fff_last_launch returns.
// The note is kept as it is handed over and put into text only when asked for (formatting it cost a
// fifth of the host time of a small call): `fmt` and every %s argument must be string literals,
// the others are printed with %d.
struct LaunchNote {
    static constexpr int kMaxArgs = 10;
    const char* fmt;
    intptr_t args[kMaxArgs];
};
void add_launch_note(const LaunchNote& note);
template <class... A> inline void note_launch(const char* fmt, A... args) {
    static_assert(sizeof...(A) <= LaunchNote::kMaxArgs, "");
    add_launch_note(LaunchNote{fmt, {(intptr_t)args...}});
}

// Per-block leaf counts, the hand-over from the descent to the bucketing stage: block b of the
// descent owns tokens [b * share, (b + 1) * share) and leaves M[b][leaf] = how many of them reach
// `leaf`, so that the bucketing stage needs no histogram pass of its own (launch_bucket_fold).
struct DescentCounts {
    int32_t* M = nullptr;    // in: room for `capacity` words
    int64_t capacity = 0;
    int blocks = 0;          // out: blocks that wrote a row of M; 0 = the launch left no counts
    int64_t share = 0;       // out: tokens per block
    int rows = 1, n_rows = 0; // out: rows of M a block's tokens are counted in (0 rows in all: one a block)
};
constexpr int kFoldMaxLeaves = 1024;
constexpr int kFoldMaxShare = 1024;
constexpr int64_t kFoldWords = 128 * 1024;   // [blocks, leaves] counters the fold kernel reads per block
bool bucket_fold_ok(int depth, int64_t blocks, int64_t share);

// K1: tree descent.  leaf_idx[t] for all t (any shape: falls back to element loads).
// dc (optional): the launch also leaves per-block leaf counts there when bucket_fold_ok.
hipError_t launch_descend(const Problem& p, int32_t* leaf_idx, hipStream_t s, DescentCounts* dc = nullptr);
// Descent + leaf network + output row in one launch; needs fused_shape_ok(p).
hipError_t launch_walk_fused(const Problem& p, int32_t* leaf_idx, hipStream_t s);
// The same for batches of up to 48 tokens a compute unit, a wave a token, leaves of up to 64 neurons (launch_walk_wave needs
// wave_shape_ok; wave_better: whether it is the faster one).
bool wave_shape_ok(const Problem& p);
bool wave_better(const Problem& p);
hipError_t launch_walk_wave(const Problem& p, int32_t* leaf_idx, hipStream_t s);
// The fused launch's lower part for tokens grouped (perm) by the node of level base_level they have reached (start [T]); needs
// fused_shape_ok(p).
hipError_t launch_walk_grouped(const Problem& p, int base_level, const int32_t* perm, const int32_t* start, int32_t* leaf_idx, hipStream_t s);
// The fused launch cut in two for leaf tables that outgrow an L2: walk + hidden neurons per token
// (launch_walk_hidden: leaf_idx [T] and hidden [T, L] fp32 out), then the output rows by column
// slices (launch_leaf_slices): every XCD writes one slice of all rows, so that its L2 only ever
// holds that slice of the output weights and biases.  Same arithmetic in the same order as the
// single launch.  Needs fused_shape_ok and slices_shape_ok.
hipError_t launch_walk_hidden(const Problem& p, int32_t* leaf_idx, float* hidden, hipStream_t s);
bool slices_shape_ok(const Problem& p);
hipError_t launch_leaf_slices(const Problem& p, const int32_t* leaf_idx, const float* hidden, hipStream_t s);
// Experiment switches of the walk kernel (0 = the built-in choice).
// Compute units, the dynamic LDS a block may ask for, the L2 of one XCD and the index of the current device (cached).
struct DeviceInfo {
    int cus = 0;
    size_t lds_per_block = 0;
    int dev = 0;
    int64_t l2_bytes = 0;   // one XCD's L2
};
DeviceInfo device_info();

struct WalkTuning {
    int64_t tpg = 0;     // tokens per lane group
    int64_t block = 0;   // threads per block
    int64_t top = 0;     // k + 1 forces at most k LDS-staged levels
    int64_t bpc = 0;     // persistent blocks per compute unit
    int64_t prefetch = 0; // 1: request the next tile's token rows one iteration ahead
    int64_t plain_x = 0;  // descent: 1 = read token rows without the streaming hint, 2 = with it, 0 = by batch size
    int64_t last_top = 0; // read-only: tree levels the last walk launch kept in LDS
};
extern WalkTuning g_walk_tuning;
bool walk_shape_ok(const Problem& p);
bool fused_shape_ok(const Problem& p);

// K2: bucketing.  Needs ws.chunk_cnt zeroed on entry; leaves it dirty.
//   slot_leaf (optional): the leaf of every slot of perm
hipError_t launch_bucket(const int32_t* leaf_idx, int64_t T, int depth, const Workspace& ws,
                         int32_t* count, int32_t* offset, int32_t* perm, int32_t* slot_leaf, hipStream_t s);
hipError_t launch_zero(int32_t* p, int64_t n, hipStream_t s);
// K2 in one launch (no workspace besides the outputs); any output may be null.
bool bucket_onepass_ok(int64_t T, int depth);
hipError_t launch_bucket_onepass(const int32_t* leaf_idx, int64_t T, int depth, int32_t* count,
                                 int32_t* offset, int32_t* perm, int32_t* slot_leaf, hipStream_t s);

// K2 in one launch with a block per chunk of tokens (every block histograms all tokens in LDS);
// for T up to 131072 and up to 4096 leaves; same outputs, any may be null.
bool bucket_hist_ok(int64_t T, int depth);
hipError_t launch_bucket_hist(const int32_t* leaf_idx, int64_t T, int depth, int32_t* count, int32_t* offset,
                              int32_t* perm, int32_t* slot_leaf, hipStream_t s);

// K2 from per-block leaf counts (the descent's, or launch_chunk_counts' for a leaf_idx array that
// came from elsewhere): one launch of dc.blocks blocks, each sums the columns of M, scans the leaves
// and places its own share of the tokens.  Needs dc.blocks > 0.
hipError_t launch_chunk_counts(const int32_t* leaf_idx, int64_t T, int depth, DescentCounts* dc, hipStream_t s);
hipError_t launch_bucket_fold(const int32_t* leaf_idx, int64_t T, int depth, const DescentCounts& dc,
                              int32_t* count, int32_t* offset, int32_t* perm, int32_t* slot_leaf, hipStream_t s);

// K2 for many tokens over few leaves (up to 4096): segments of 1024 tokens, three launches (count, scan,
// scatter); the matrix region of the workspace must hold a column per segment (bucket_segments_ok).
bool bucket_segments_ok(int64_t T, int depth, const Workspace& ws);
hipError_t launch_bucket_segments(const int32_t* leaf_idx, int64_t T, int depth, const Workspace& ws,
                                  int32_t* count, int32_t* offset, int32_t* perm, int32_t* slot_leaf,
                                  hipStream_t s);

// K3 + K4: leaf networks and output rows.
//   order == nullptr: slot i is token i.  Otherwise slot i is token order[i].
//   split > 0 (needs order, the leaf of every slot, and gather_takes_split(p)): only the tiles of 16
//   consecutive slots with at least `split` runs of equal leaf are handled, the rest is left to
//   launch_leaf_tiles with the same value.
bool gather_takes_split(const Problem& p);
hipError_t launch_leaf_gather(const Problem& p, const int32_t* leaf_idx, const int32_t* order,
                              hipStream_t s, const int32_t* slot_leaf = nullptr, int split = 0);
// MFMA tile path over tokens grouped by leaf (perm, and the leaf of every slot); needs tiles_shape_ok(p).
// Two launches (hidden activations, output rows); `between`, if given, is called between them.
bool tiles_shape_ok(const Problem& p);
//   split > 0: tiles with at least `split` runs of equal leaf are skipped (launch_leaf_gather's).
hipError_t launch_leaf_tiles(const Problem& p, const int32_t* slot_leaf, const int32_t* perm, void* hidden,
                             hipStream_t s, void (*between)(hipStream_t) = nullptr, int split = 0);

// Whole forward pass in one launch, one block per token: the small-batch path, built for the
// latency of the dependent loads rather than for throughput; needs token_shape_ok(p).
// given_leaf (optional): the leaf of every token, or gate: the candidates to pick it from (the pick goes to
// leaf_idx); then only the leaf networks run (the node weights are not read, token_shape_ok's
// condition on them does not apply).
struct GateCandidates;
// wide (optional): nodes of `n` hidden neurons on the layer-normalised token (gamma null: no normalisation), plus the
// token itself when `residual`: fff_forward_block's small batches; needs token_wide_ok(p, n).
struct WideNodes {
    const void* gamma = nullptr;
    const void* beta = nullptr;
    const void* w1 = nullptr;   // [nodes, n, D]
    const void* b1 = nullptr;   // [nodes, n]
    const void* w2 = nullptr;   // [nodes, n]
    const void* b2 = nullptr;   // [nodes]
    int n = 1;
    bool residual = false;
    float eps = 0;
};
// The last k levels of the walk, the leaf network and the output row of tokens grouped by the node of
// level depth - k they have reached (perm, and offset [2^(depth - k) + 1]); needs subtree_shape_ok(p, k).
// leaf_idx (optional): the leaf reached.  k = 0: the leaf networks alone.
// fp32_hidden (bf16 calls): hidden activations in all bits of fp32, not in the 16 of two bf16 values.
// wide (optional): fff_forward_block's nodes, norm and residual (hidden activations in all bits of fp32); stats [2 T]: what launch_subtree_levels from the root left.
constexpr int kSubtreeMaxColumns = 128;
int64_t subtree_columns(int k, int node_size, int L);
int subtree_row_parts(const Problem& p);
bool subtree_shape_ok(const Problem& p, int k, const WideNodes* wide = nullptr);
hipError_t launch_subtree(const Problem& p, int k, const int32_t* perm, const int32_t* offset, int32_t* leaf_idx, hipStream_t s,
                          bool fp32_hidden, const WideNodes* wide = nullptr, float* stats = nullptr);
// Levels base_level .. base_level + k - 1 of wide nodes: node_idx[t] = position of the node reached in its level.  perm and offset as above
// for base_level > 0, null for the root (dc, optional: per-tile counts for launch_bucket_fold).
hipError_t launch_subtree_levels(const Problem& p, int base_level, int k, const int32_t* perm, const int32_t* offset, int32_t* node_idx,
                                 hipStream_t s, const WideNodes& wide, float* stats, DescentCounts* dc);

bool token_shape_ok(const Problem& p);
bool token_wide_ok(const Problem& p, int node_size);
hipError_t launch_token_block(const Problem& p, int32_t* leaf_idx, hipStream_t s,
                              const int32_t* given_leaf = nullptr, const GateCandidates* gate = nullptr,
                              const WideNodes* wide = nullptr);

// The same for whole aligned rows of up to 512 pieces, a wave holding whole rows; blocks stride over the batch.
// token_rows_better: whether it takes the call and is the faster one (picks: of a mixture, whose pick the other launch saves).
extern int64_t g_token_kernel;      // experiment switch "token_kernel"
bool token_rows_ok(const Problem& p);
bool token_rows_better(const Problem& p, bool picks = false);
hipError_t launch_token_rows(const Problem& p, int32_t* leaf_idx, hipStream_t s, const int32_t* given_leaf = nullptr);

// Gating of a mixture of experts with one engaged expert (fff_moe_gate.hip).  launch_moe_gate leaves, per
// token, the best (logit, expert) of every block of experts in `cand` (moe_gate_words(T, n_experts)
// words); the token-block launch picks among them itself, launch_moe_pick writes expert_idx[t] =
// argmax_e gate_w[e] . x[t] (+ gate_b[e]) for the other routes.
struct GateCandidates {
    const float* val = nullptr;      // [T][n]
    const int32_t* idx = nullptr;
    int n = 0;
};
int64_t moe_gate_words(int64_t T, int64_t n_experts);
bool moe_gate_shape_ok(const void* x, const void* gate_w, int64_t D, bool bf16);
hipError_t launch_moe_gate(const void* x, const void* gate_w, const void* gate_b, int64_t T, int64_t D,
                           int64_t n_experts, int32_t* cand, GateCandidates* out, hipStream_t s);
hipError_t launch_moe_pick(const GateCandidates& c, int64_t T, int32_t* expert_idx, hipStream_t s);

// Forward_T (fff_soft.hip): the soft mixture over all leaves on the matrix cores.  scratch holds
// soft_scratch_words(p) 32-bit words; mix [T, 2^depth] and entropy [2^depth - 1] (fp32) are optional outputs.
extern int64_t g_soft_small_tiles;
bool soft_shape_ok(const Problem& p);
int64_t soft_scratch_words(const Problem& p);
hipError_t launch_forward_soft(const Problem& p, int32_t* scratch, float* mix_out, float* entropy_out,
                               hipStream_t s);

// Forward_I with nodes of `node_size` hidden neurons on the layer-normalised token (gamma null:
// no normalisation), plus the token itself when `residual` (fff_block.hip); one launch, a wave per
// token.  p.node_w / p.node_b are not used.  vector_rows needs block_shape_ok (and 16-byte aligned
// rows of every other tensor); without it an element-wise kernel takes any shape.
struct BlockTuning {
    int64_t top = 0;      // k + 1 forces at most k LDS-staged node levels
    int64_t last_top = 0; // read-only: node levels the last fff_forward_block launch kept in LDS
};
extern BlockTuning g_block_tuning;
bool block_shape_ok(const void* x, const void* out, const void* leaf_w1, const void* leaf_w2, int64_t D,
                    int64_t O, bool bf16);
hipError_t launch_forward_block(const Problem& p, const void* gamma, const void* beta, float eps,
                                const void* node_w1, const void* node_b1, const void* node_w2,
                                const void* node_b2, int node_size, bool residual, int32_t* leaf_idx,
                                hipStream_t s, bool vector_rows = true);

// Whole forward pass in one launch for rows at any element, 16-byte pieces; needs rows_shape_ok(p).
bool rows_shape_ok(const Problem& p);
hipError_t launch_fused_rows(const Problem& p, int32_t* leaf_idx, hipStream_t s);
// Whole forward pass in one launch, a wave a token, element-wise (any shape).
hipError_t launch_fused_generic(const Problem& p, int32_t* leaf_idx, hipStream_t s);

// Contractions [T, K] x [K, N]: blocks of 16 mt x 16 nt results, and estimates of the time in us with a
// block's waves on slices of K (mfma_wave_slice) and with 64 x 128 tiles, fitted to kernel times over
// T = 64 .. 8192, N = 15 .. 2048, K = 80 .. 3504 (within about 25 %).  own: the soft pass's hidden
// launch that multiplies its own mixture weights.
inline int64_t small_blocks(int64_t T, int64_t N, int mt, int nt) {
    return ((T + 16 * mt - 1) / (16 * mt)) * ((N + 16 * nt - 1) / (16 * nt));
}
inline double small_cost(double T, double N, double K, bool own = false) {
    return 4 + T / 32 * N / 64 * (0.0076 + (own ? 0.005 : 0) + 1.9e-5 * K);
}
inline double tile_cost(int64_t T, int64_t N, double K) {
    const double blocks = (double)((T + 63) / 64 * ((N + 127) / 128));
    return 10.5 + 0.0067 * K + (blocks > 256 ? (blocks - 256) * (2e-3 + 2.8e-5 * K) : 0);
}
// Grids that cover three quarters of the 256 compute units keep the larger of the small tiles.
constexpr int64_t kSmallEnoughBlocks = 192;

}  // namespace fff
