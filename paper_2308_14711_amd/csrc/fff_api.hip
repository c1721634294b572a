// C ABI of the FFF library: argument checks (host only, before any HIP call),
// per-device workspace, and the sequence of kernel launches of Forward_I
// (Algorithm 1): descent -> bucketing -> leaf networks with fused output rows.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fff.h"
#include "fff_internal.h"

// Scratch of fff_forward_hard_static, the entry point for callers that cannot allocate: a fixed
// block in the device image of this library, so every GPU the library runs on holds one copy of it
// (at an address of its own) until the process ends.  The name is a host-side stand-in: host code
// never passes it anywhere, it asks each device for the array's address once (scratch_on_device)
// and uses that pointer.
#define FFF_STATIC_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[FFF_STATIC_SCRATCH_BYTES];

namespace fff {
namespace {

thread_local std::string g_last_error;
// kernels of the last forward call (process-wide, like the "last_*" options), put into text by fff_last_launch
constexpr int kMaxNotes = 8;
LaunchNote g_notes[kMaxNotes];
int g_n_notes = 0;
std::mutex g_notes_mu;   // forward calls of several threads note their kernels in one list

// One workspace per device: the library's own block (grown on demand), or the caller's
// (fff_set_workspace), which takes precedence while it is set.
struct DeviceWs {
    void* base = nullptr;        // library-owned
    size_t bytes = 0;
    void* user_base = nullptr;   // caller-provided
    size_t user_bytes = 0;
};
constexpr int kMaxDevices = 64;
DeviceWs g_ws[kMaxDevices];
std::mutex g_mu;

struct Options {
    int64_t path = 0;            // 0 auto, 1 fused walk, 2 staged, 3 generic one-wave-per-token, ..., 6 grouped walk, 7 wave a token
    int64_t leaf_path = 0;       // 0 auto, 1 gather kernel only, 2 MFMA tiles whenever the shape allows
    int64_t bucketing = 1;       // 0: leaf kernel visits tokens in token order
    int64_t stage_timing = 0;    // 1: bracket the stages of fff_forward_hard with events
    int64_t bucket_kernel = 0;   // 0 auto, 1 leaf-range kernel, 2 chunk-matrix kernels, 3 token-chunk kernel, 4 segment kernels
    int64_t last_path = 0;       // read-only: the path the last fff_forward_hard call took
    int64_t last_leaf_path = 0;  // read-only: leaf stage of the last staged call (1 gather kernel, 2 tile kernels, 3 both)
    int64_t leaf_split = 0;      // 1..16: tiles of 16 slots with that many runs of equal leaf go to the gather kernel
    int64_t last_block_kernel = 0; // read-only: 1 = fff_forward_block ran a vector kernel, 2 = the element-wise one
    int64_t token_max_T = 512;   // batches up to this many tokens (6x where no fused launch fits) go one block per token
} g_opt;

// the vector L1 of a compute unit (not reported by the runtime)
constexpr int64_t kVectorL1Bytes = 32 * 1024;

// Events recorded around the stages of fff_forward_hard while "stage_timing" is on:
// five per call (start, after descent, after bucketing, after the leaf stage's first kernel, after
// its second; a path with fewer kernels records the later marks back to back).
std::vector<hipEvent_t> g_stage_events;

void stage_mark(hipStream_t s) {
    if (!g_opt.stage_timing) return;
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return;
    if (hipEventRecord(e, s) != hipSuccess) {
        (void)hipEventDestroy(e);
        return;
    }
    std::lock_guard<std::mutex> lock(g_mu);
    g_stage_events.push_back(e);
}

constexpr int64_t kAlignWords = 64;            // 256-byte regions
constexpr int64_t kMaxMatrixWords = 8 << 20;   // per-chunk histogram budget (32 MiB)
constexpr int64_t kCtrlWords = 64;

int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

struct Layout {
    int64_t n_chunks;
    int64_t o_ctrl, o_leaf, o_rank, o_sleaf, o_perm, o_count, o_offset, o_tileoff, o_matrix, o_fold, o_hidden, o_extra, total;
};

// extra_words: room for a caller-specific scratch region (the gating candidates of the mixture of experts)
Layout layout_for(int64_t T, int depth, int64_t extra_words = 0) {
    Layout l;
    const int64_t NL = (int64_t)1 << depth;
    const int64_t per_round = (T + kChunkTokens - 1) / kChunkTokens;
    int64_t c = kMaxMatrixWords / NL;
    if (c < 1) c = 1;
    if (c > per_round) c = per_round;
    if (c < 1) c = 1;
    l.n_chunks = c;
    int64_t o = 0;
    auto take = [&](int64_t words) { int64_t at = o; o += round_up(words, kAlignWords); return at; };
    l.o_ctrl = take(kCtrlWords);
    l.o_leaf = take(T);
    l.o_rank = take(T);
    l.o_sleaf = take(T);
    l.o_perm = take(T);
    l.o_count = take(NL);
    l.o_offset = take(NL + 1);
    l.o_tileoff = take(NL + 1);
    l.o_matrix = take(c * NL);
    l.o_fold = take(T > 0 && depth <= 10 ? kFoldWords : 0);   // per-block leaf counts of the descent
    l.o_hidden = take((int64_t)(kTilesMaxLeafWidth / 2) * T);   // T * L bf16 values, L up to the tile path's limit
    l.o_extra = take(extra_words);
    l.total = o;
    return l;
}

// Called once the host-side checks have passed: forgets the message of an earlier failure and
// any error another user of the HIP runtime left in this thread's last-error slot, so that the
// launch checks below report this call's errors only.
void begin_device_call() {
    g_last_error.clear();
    {
        std::lock_guard<std::mutex> lock(g_notes_mu);
        g_n_notes = 0;
    }
    (void)hipGetLastError();
}

int set_device_error(hipError_t e, const char* what) {
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return FFF_ERR_DEVICE;
}

int current_device(int* dev) {
    hipError_t e = hipGetDevice(dev);
    if (e != hipSuccess) return set_device_error(e, "hipGetDevice");
    if (*dev < 0 || *dev >= kMaxDevices) {
        g_last_error = "device ordinal out of range";
        return FFF_ERR_DEVICE;
    }
    return FFF_OK;
}

int64_t g_fail_growths = 0;   // debug option "fail_workspace_growth": how many of the next growths fail

// Makes the current device's library-owned block at least `need` bytes (g_mu held).  Growing frees
// the old block (which waits for the device) and cannot be done while `s` is being captured.
int grow_owned(DeviceWs& d, size_t need, hipStream_t s, bool check_capture) {
    if (d.bytes >= need) return FFF_OK;
    if (check_capture) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &st) != hipSuccess) (void)hipGetLastError();
        if (st != hipStreamCaptureStatusNone) {
            g_last_error = "workspace must grow to " + std::to_string(need) +
                           " bytes, which cannot happen during stream capture: reserve or set it first";
            return FFF_ERR_WORKSPACE;
        }
    }
    hipError_t e;
    if (d.base) {
        e = hipFree(d.base);   // waits for work that may still use it
        d.base = nullptr;
        d.bytes = 0;
        if (e != hipSuccess) return set_device_error(e, "hipFree(workspace)");
    }
    void* p = nullptr;
    if (g_fail_growths > 0) {          // test hook: this growth fails the way an exhausted device would
        --g_fail_growths;
        e = hipErrorOutOfMemory;
    } else {
        e = hipMalloc(&p, need);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        g_last_error = std::string("hipMalloc(workspace): ") + hipGetErrorString(e);
        return FFF_ERR_WORKSPACE;
    }
    e = hipMemset(p, 0, kCtrlWords * sizeof(int32_t));   // ticket counters start at zero
    if (e != hipSuccess) {
        (void)hipFree(p);
        return set_device_error(e, "hipMemset(workspace)");
    }
    d.base = p;
    d.bytes = need;
    return FFF_OK;
}

void carve(void* base, const Layout& lay, Workspace* ws) {
    int32_t* b = (int32_t*)base;
    ws->ctrl = b + lay.o_ctrl;
    ws->leaf_idx = b + lay.o_leaf;
    ws->rank = b + lay.o_rank;
    ws->slot_leaf = b + lay.o_sleaf;
    ws->perm = b + lay.o_perm;
    ws->count = b + lay.o_count;
    ws->offset = b + lay.o_offset;
    ws->tile_off = b + lay.o_tileoff;
    ws->chunk_cnt = b + lay.o_matrix;
    ws->fold = b + lay.o_fold;
    ws->hidden = b + lay.o_hidden;
    ws->extra = b + lay.o_extra;
    ws->n_chunks = lay.n_chunks;
}

// The current device's workspace carved for (T, depth): the caller's if one is set (too small is
// an error, nothing is allocated), else the library's own, grown if needed.
int get_workspace(int64_t T, int depth, Workspace* ws, Layout* lay, hipStream_t s, int64_t extra_words = 0) {
    *lay = layout_for(T, depth, extra_words);
    const size_t need = (size_t)lay->total * sizeof(int32_t);
    int dev = 0;
    int rc = current_device(&dev);
    if (rc != FFF_OK) return rc;
    std::lock_guard<std::mutex> lock(g_mu);
    DeviceWs& d = g_ws[dev];
    if (d.user_base) {
        if (d.user_bytes < need) {
            g_last_error = "the caller's workspace holds " + std::to_string(d.user_bytes) + " bytes, this call needs " +
                           std::to_string(need);
            return FFF_ERR_WORKSPACE;
        }
        carve(d.user_base, *lay, ws);
        return FFF_OK;
    }
    if ((rc = grow_owned(d, need, s, true)) != FFF_OK) return rc;
    carve(d.base, *lay, ws);
    return FFF_OK;
}

constexpr int64_t kMaxElems = (int64_t)1 << 40;
constexpr int64_t kMaxTokens = ((int64_t)1 << 31) - 1024;
constexpr int kMaxLeafWidth = 4096;

int check_common(int depth, int64_t T, int64_t D, int dtype) {
    if (dtype != FFF_F32 && dtype != FFF_BF16) return FFF_ERR_DTYPE;
    if (depth < 0 || depth > FFF_MAX_DEPTH) return FFF_ERR_RANGE;
    if (T < 0 || T > kMaxTokens) return FFF_ERR_RANGE;
    if (D < 1 || D > kMaxElems) return FFF_ERR_SHAPE;
    if (T * D > kMaxElems || ((int64_t)1 << depth) * D > kMaxElems) return FFF_ERR_SHAPE;
    return FFF_OK;
}

int check_leaf(int depth, int leaf_width, int act, int64_t T, int64_t D, int64_t O) {
    if (leaf_width < 1 || leaf_width > kMaxLeafWidth) return FFF_ERR_RANGE;
    if (O < 1 || O > kMaxElems) return FFF_ERR_SHAPE;
    const int64_t m = D > O ? D : O;
    if (T * O > kMaxElems || ((int64_t)1 << depth) * leaf_width > kMaxElems / m) return FFF_ERR_SHAPE;
    if (act != FFF_ACT_RELU && act != FFF_ACT_GELU) return FFF_ERR_UNSUPPORTED;
    return FFF_OK;
}

bool overlaps(const void* a, int64_t abytes, const void* b, int64_t bbytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + (uintptr_t)bbytes && b0 < a0 + (uintptr_t)abytes;
}

// Shapes the staged path's 16-byte vector kernels take.
bool staged_shape_ok(const Problem& p) {
    return walk_shape_ok(p) && vec_ok(p.leaf_w1, p.D, p.bf16) && p.L <= 64;
}

int64_t g_subtree = 0;   // debug option "subtree"

// Whether no option picks among the launches of the staged path, the walk kernels or the block-a-token kernels: one that does asks for
// these launches, and what takes calls from them by itself (a wave a token, the grouped walk) stands aside.
bool launches_by_default() {
    const WalkTuning& w = g_walk_tuning;
    return g_opt.path == 0 && g_opt.leaf_path == 0 && g_opt.leaf_split == 0 && g_opt.bucketing && g_opt.bucket_kernel == 0 && g_subtree == 0 &&
           g_token_kernel == 0 && !w.tpg && !w.block && !w.top && !w.bpc && !w.prefetch && !w.plain_x;
}

bool grouped_shape_ok(const Problem& p) {
    return fused_shape_ok(p) && p.depth >= 2 && p.T >= 1 && p.T <= 131072 && vec_ok(p.out, p.O, p.bf16) && vec_ok(p.leaf_w2, p.O, p.bf16) &&
           vec_ok(p.leaf_b2, p.O, p.bf16);
}

enum { kPathAuto = 0, kPathFused = 1, kPathStaged = 2, kPathGeneric = 3, kPathToken = 4, kPathSplit = 5, kPathGrouped = 6, kPathWave = 7 };

// One launch that keeps the token row in registers from the root to the output
// row wins while a leaf is narrow (its weights are a few rows per token, like a
// few more tree levels); wider leaves want tokens grouped so that a leaf's
// weights are read once per group.
int choose_path(const Problem& p) {
    const bool fused_ok = fused_shape_ok(p), staged_ok = staged_shape_ok(p), token_ok = token_shape_ok(p);
    const bool split_ok = fused_ok && slices_shape_ok(p);
    if (g_opt.path == kPathToken && token_ok) return kPathToken;
    if (g_opt.path == kPathSplit && split_ok) return kPathSplit;
    if (g_opt.path == kPathWave && wave_shape_ok(p)) return kPathWave;
    if (g_opt.path == kPathGrouped && grouped_shape_ok(p)) return kPathGrouped;
    if (g_opt.path == kPathFused && fused_ok) return kPathFused;
    if (g_opt.path == kPathStaged && staged_ok) return kPathStaged;
    if (g_opt.path == kPathGeneric) return kPathGeneric;
    // a small batch cannot fill the chip with streaming work: one block per token, built for latency
    // (measured crossovers on 768-wide rows: the fused launch, with its smallest tiles, takes 9-12 us
    // from 256 to 2048 tokens, this one 9 us up to 512 tokens and 13-16 at 1024; leaves too wide for
    // the fused launch leave only the staged path, which overtakes between 2048 and 4096 tokens)
    // Rows that are not whole pieces leave fused_rows_kernel, whose time hardly grows with the batch but with every neuron
    // (token block / rows, us a launch: 301 bf16 features, 8 neurons, 512 tokens 7.6/10.4, 768 10.7/10.4; 999, 32 neurons, 1024
    // 23.4/29.1, 1536 33.6/30.2; 599 fp32, 2 neurons, 256 6.1/6.4, 512 8.0/6.6; 77, 4 neurons, 512 6.6/4.2).
    int64_t token_limit = fused_ok ? g_opt.token_max_T : 6 * g_opt.token_max_T;
    if (!fused_ok && !staged_ok && rows_shape_ok(p)) {
        const int64_t limit = g_opt.token_max_T / 2 + 36 * (int64_t)p.L;
        if (limit < token_limit) token_limit = limit;
    } else if (!fused_ok && !staged_ok && p.D <= 64 && !token_rows_ok(p)) {
        // such rows with wider leaves leave the element-wise kernel, a wave a token, which takes a row of up to 64 features at a time
        // (token block / element-wise: 2181 tokens of 9 bf16 features, 168 neurons 94 / 62; 1161 of 11, 116 neurons 39 / 43)
        token_limit = 3 * g_opt.token_max_T;
    }
    if (p.T > g_opt.token_max_T && launches_by_default() && wave_better(p)) return kPathWave;
    if (g_opt.path == kPathAuto && token_ok && p.T <= token_limit) return kPathToken;
    // Whole rows of leaves wider than the staged path takes go one block a token at any batch size: their alternative is the
    // element-wise kernel (4312 tokens of 464 bf16 features, 240 neurons: 391 us against 168).  Not so rows of other
    // lengths (30616 tokens of 9 features, 385 neurons: 706 against 2571).
    if (!fused_ok && !staged_ok)
        return token_ok && (p.T <= token_limit || (p.L > 64 && token_rows_ok(p))) ? kPathToken : kPathGeneric;
    // The fused launch gathers, per token, the leaf's output-weight and bias rows from a table of
    // 2^depth (leaf_width + 1) rows.  Once that table outgrows the L2 of an XCD most of those rows
    // come back from memory; the launch cut in two (walk and hidden neurons per token, then the
    // output rows by column slices, one slice of all rows per XCD) keeps each slice in its L2.
    // Measured on 768-wide rows, 65536 tokens, one neuron a leaf: depth 11 (6 MB of output rows)
    // 80 -> 70 us, depth 12 93 -> 82, depth 13 106 -> 101; two neurons, depth 11: 99 -> 86;
    // 4096-wide rows, 16384 tokens, depth 10: 140 -> 108.  With one neuron a leaf and a full batch
    // (256 tokens per compute unit and more) it is ahead for smaller tables too (depth 8: 57 -> 53),
    // since the walk then runs in the descent's leaner tile shape.  Rows shorter than 1 KB and
    // batches of up to 32 tokens per compute unit stay on the single launch (two launches cost
    // more than they save: 16384 tokens, depth 10: 20.6 against 21.4 us).
    const auto fused_or_split = [&]() {
        if (!split_ok || g_opt.path == kPathFused) return (int)kPathFused;
        const DeviceInfo di = device_info();
        const int64_t es = p.bf16 ? 2 : 4;
        const int64_t out_table = ((int64_t)(p.L + 1) * p.O * es) << p.depth;
        const bool full_rows = p.O * es >= 1024 && p.D * es >= 1024;
        const bool big_batch = p.T > 32 * (int64_t)di.cus;
        // (from 128 tokens per compute unit on, three quarters of an L2 are enough: 100000 tokens, 512-wide
        // rows, two neurons, depth 10 -- 3.1 MB of output rows -- 94 us fused, 78 split)
        const int64_t table_min = p.T >= 128 * (int64_t)di.cus ? di.l2_bytes * 3 / 4 : di.l2_bytes;
        const bool split = full_rows && big_batch &&
                           out_table <= 64 * di.l2_bytes &&     // beyond that no slice of it stays in an L2 either
                           (out_table >= table_min || (p.L == 1 && p.T >= 256 * (int64_t)di.cus));
        return split ? (int)kPathSplit : (int)kPathFused;
    };
    if (!staged_ok) return fused_or_split();
    if (!fused_ok) return kPathStaged;
    // one or two neurons a leaf are "three more tree levels" whatever the row length: never worth
    // the passes of the staged path (9000 tokens, 3072 inputs, 768 outputs, two neurons, depth 9:
    // 71 us staged, 62 fused, 55 split; 768-wide rows, two neurons, depth 13: 133 / 132 / 128)
    if (p.L <= 2) return fused_or_split();
    // Grouping pays once the leaf rows a token meets are many bytes -- 24 KB (8 neurons on 768-wide
    // bf16 rows), or 12 KB (4 neurons) where the leaf weights together (8 MB) outgrow the 4 MB L2 of one XCD,
    // which the fused launch relies on for its per-token row fetches, or 8 KB (3 neurons) from 16 MB
    // on (measured on 768-wide rows: depth 8 ties at 6 neurons, depth 10 at 4, depth 4 only at 8;
    // 128-wide rows stay on the fused launch at 8 neurons, 256-wide ones leave it at depth 12) --
    // and a leaf is visited by a few tokens on average: in bucket order the tokens of a leaf find
    // its rows in cache, so the staged path stays ahead down to 3 tokens a leaf (50432 tokens,
    // 768-wide rows, 8 neurons, depth 13 and 14: 151 and 218 us against 224 and 260 fused; 16384
    // tokens, 4096-wide rows, 4 neurons, depth 12: 233 against 285); below that (the skewed workload:
    // half a token a leaf) the single launch wins again.  Up to 8192 tokens the fused launch, cut
    // into tiles of 32 tokens, is ahead for every leaf it takes (2048-8192 tokens, 8 neurons, depth
    // 9: 17-22 us against 25-31 staged; 16384 tokens: 42 against 34).
    // In the device's own units: a token's leaf rows against the vector L1 of a compute unit
    // (3/4, 3/8, 1/4 of its 32 KB), all leaf weights against the L2 of one XCD (2x, 4x its 4 MB),
    // the batch against 32 tokens per compute unit.
    const DeviceInfo di = device_info();
    const int64_t es = p.bf16 ? 2 : 4;
    const int64_t token_leaf_bytes = (p.L * (p.D + p.O) + p.O) * es;
    const int64_t leaf_bytes = token_leaf_bytes << p.depth;
    const bool wide = token_leaf_bytes * 4 >= 3 * kVectorL1Bytes ||
                      (token_leaf_bytes * 8 >= 3 * kVectorL1Bytes && leaf_bytes >= 2 * di.l2_bytes) ||
                      (token_leaf_bytes * 4 >= kVectorL1Bytes && leaf_bytes >= 4 * di.l2_bytes);
    const bool visited = p.T > 32 * (int64_t)di.cus && p.depth < 40 && p.T >= ((int64_t)3 << p.depth);
    return (wide && visited) ? (int)kPathStaged : fused_or_split();
}

// K2 with whichever kernel set takes the sizes; outputs may be null (then workspace arrays are used).
// dc (optional): per-block leaf counts the descent left behind; then one fold launch finishes the job.
int run_bucket(const int32_t* leaf_idx, int64_t T, int depth, const Workspace& ws, int32_t* count,
               int32_t* offset, int32_t* perm, int32_t* slot_leaf, hipStream_t s, const DescentCounts* dc = nullptr) {
    hipError_t e;
    if (dc && dc->blocks > 0 && (g_opt.bucket_kernel == 0 || g_opt.bucket_kernel == 5)) {
        e = launch_bucket_fold(leaf_idx, T, depth, *dc, count, offset, perm, slot_leaf, s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "bucket kernel launch");
    }
    if (g_opt.bucket_kernel == 5 && T > 0 && depth <= 10) {   // the same kernel fed by a counting launch of its own
        DescentCounts own;
        own.M = ws.fold;
        own.capacity = kFoldWords;
        if ((e = launch_chunk_counts(leaf_idx, T, depth, &own, s)) != hipSuccess)
            return set_device_error(e, "bucket kernel launch");
        if (own.blocks > 0) {
            e = launch_bucket_fold(leaf_idx, T, depth, own, count, offset, perm, slot_leaf, s);
            return e == hipSuccess ? FFF_OK : set_device_error(e, "bucket kernel launch");
        }
    }
    if ((g_opt.bucket_kernel == 0 || g_opt.bucket_kernel == 3) && bucket_hist_ok(T, depth)) {
        e = launch_bucket_hist(leaf_idx, T, depth, count, offset, perm, slot_leaf, s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "bucket kernel launch");
    }
    // beyond the token-chunk kernel's sizes: the leaf-range kernel reads leaf_idx once per block of
    // leaves, which pays for many leaves; for few leaves (up to 4096) and many tokens the segment
    // kernels (count / scan / scatter over segments of 1024 tokens) are faster, and so are the
    // chunk-matrix kernels (806912 tokens over 256 leaves: 102 against 224 us; 201728: 47 against 72 us)
    const bool few_leaves = g_opt.bucket_kernel == 0 && depth <= 12;
    if ((few_leaves || g_opt.bucket_kernel == 4) && bucket_segments_ok(T, depth, ws)) {
        e = launch_bucket_segments(leaf_idx, T, depth, ws, count, offset, perm, slot_leaf, s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "bucket kernel launch");
    }
    if (g_opt.bucket_kernel != 2 && !few_leaves && bucket_onepass_ok(T, depth)) {
        e = launch_bucket_onepass(leaf_idx, T, depth, count, offset, perm, slot_leaf, s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "bucket kernel launch");
    }
    const int64_t NL = (int64_t)1 << depth;
    if ((e = launch_zero(ws.chunk_cnt, round_up(ws.n_chunks * NL, 4), s)) != hipSuccess)
        return set_device_error(e, "zero kernel launch");
    if ((e = launch_bucket(leaf_idx, T, depth, ws, count, offset, perm, slot_leaf, s)) != hipSuccess)
        return set_device_error(e, "bucket kernel launch");
    return FFF_OK;
}

// How many of the last levels the subtree launch takes; -1: whole descent and leaf kernels.
//
// Where tokens are grouped the subtree launch is mostly ahead of the leaf kernels (25216 tokens, 768-wide, depth 8, 8 neurons, fp32: leaf
// kernels 103 us, subtree launch 80; 50432 bf16 71 / 66; 12000 1024-wide, 16 neurons 41 / 31).  Not so, in the same order, where
//   - there are fewer tiles of 64 tokens than compute units and rows of more than 4 KB, whose pieces a tile walks in turn (14315 tokens,
//     3168-wide 93 / 99), fp32 on half as many (3521 tokens of 856, 12 neurons 38 / 48), or bf16 leaves of up to 8 neurons, where little is
//     to be had (16384 tokens of 768, depth 8 34 / 30 us),
//   - output rows are three times as long as input rows and more (34782 tokens, 88 to 584 features, 16 neurons 37 / 45),
//   - leaves see few tokens (19686 of fp32, depth 11 41 / 44; 5679 of bf16, depth 11, 16 neurons 19 / 29),
//   - leaves are small, while the launch computes 16 columns of whatever a tile holds: fewer than 3 neurons, in fp32 4 (26448 bf16 tokens
//     of 128, depth 8, one neuron 15 / 21; 12168 fp32 ones of 656 to 912, depth 9, one neuron 22 / 38), or fp32 and less than 8 KB of rows for a token (30567 of 136, depth 10, 9 neurons 28 / 40),
//   - the leaves are given, so that small groups cannot be merged: fewer than 64 tokens a leaf (fp32: and fewer tiles than compute units), or
//     1024 leaves of less than 8 KB of rows for a token (bf16, 42600 tokens of 112, 8 neurons 24 / 32; fp32 16386 of 176, 6 neurons 18 / 35).
// Of 6000 random calls in whose place these lines put 3000 here, 1.27 times as fast on average, 39 are more than 5 % slower for it.
// A tile wants whole groups: k grows until a group has 128 tokens on average, while the columns computed for all of a group stay few (48;
// one block of 16 for fp32, whose matrix instructions run at a sixteenth of the rate): 50432 tokens, 8 neurons, depth 10, k = 0, 1, 2: 93, 91,
// 83 us; fp32, 12000 tokens, depth 8, 4 neurons 53, 47, 50.
int subtree_levels(const Problem& p, bool leaves_given) {
    if (g_subtree == 1 || g_opt.leaf_path != 0 || g_opt.leaf_split != 0 || !g_opt.bucketing) return -1;
    if (g_subtree >= 2) {
        const int k = leaves_given ? 0 : (int)g_subtree - 2;
        return subtree_shape_ok(p, k) ? k : -1;
    }
    const int64_t es = p.bf16 ? 2 : 4, row_bytes = p.D * es, leaf_bytes = p.L * (p.D + p.O) * es;
    const int64_t cus = device_info().cus;
    const bool filled = p.T >= 64 * cus || (row_bytes <= 4096 && (p.bf16 ? p.L > 8 : !leaves_given && p.T > 32 * cus));
    if (!filled || p.O > 3 * p.D || p.T >> p.depth < (leaves_given ? 64 : p.bf16 ? 8 : 16)) return -1;
    if (p.L < (p.bf16 ? 3 : 4) || (!p.bf16 && leaf_bytes < 8192) || (leaves_given && p.depth >= 10 && leaf_bytes < 8192)) return -1;
    int pick = -1;
    for (int k = 0; k <= (leaves_given ? 0 : 3); ++k) {
        if (!subtree_shape_ok(p, k)) continue;
        if (pick >= 0 && subtree_columns(k, 1, p.L) > (p.bf16 ? 48 : 16)) break;
        pick = k;
        if (p.T >> (p.depth - k) >= 128) break;
    }
    return pick >= 0 && !p.bf16 && p.T >> (p.depth - pick) < 32 ? -1 : pick;
}

// Which of the two leaf stages is ahead: the MFMA tile path (hidden activations rounded to bf16), or the gather kernel (fp32
// ones, which the subtree launch in its place keeps).
//
// The tile path pays once a leaf has a few neurons (for 1-2 the VALU gather kernel is leaner)
// and a tile of 16 slots holds few different leaves: from 8 tokens a leaf on average (measured
// on 768-wide rows, 50432 tokens, 8 neurons: 12 tokens a leaf 118 us tiles against 128 gather,
// 6 tokens a leaf 168 against 151; leaves of more than 8 neurons always, the gather kernel
// needs twice the time there); up to 8192 tokens only from 32 tokens a leaf (4096 tokens, 8
// neurons, 8 tokens a leaf: 40 us against 32)
bool leaf_tiles_pay(const Problem& p) {
    const int64_t per_leaf = p.depth < 40 ? p.T >> p.depth : 0;
    const bool filled = (p.T > 32 * (int64_t)device_info().cus && (p.L > 8 || per_leaf >= 8)) || per_leaf >= 32;
    return tiles_shape_ok(p) && p.L >= 3 && filled;
}

// subtree: whether the subtree launch takes the leaves
int run_leaf_stage(const Problem& p, const int32_t* leaf_idx, const Workspace& ws, hipStream_t s, bool subtree,
                   bool timed = false, const DescentCounts* dc = nullptr) {
    hipError_t e;
    if (subtree) {
        const int rc = run_bucket(leaf_idx, p.T, p.depth, ws, nullptr, ws.offset, ws.perm, ws.slot_leaf, s, dc);
        if (rc != FFF_OK) return rc;
        if (timed) stage_mark(s);
        g_opt.last_leaf_path = 4;
        e = launch_subtree(p, 0, ws.perm, ws.offset, nullptr, s, !leaf_tiles_pay(p));
        for (int i = 0; timed && i < 2; ++i) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "subtree kernel launch");
    }
    if (!g_opt.bucketing) {
        if (timed) stage_mark(s);
        g_opt.last_leaf_path = 1;
        e = launch_leaf_gather(p, leaf_idx, nullptr, s);
        if (timed) stage_mark(s);
        if (timed) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "leaf kernel launch");
    }
    const int rc = run_bucket(leaf_idx, p.T, p.depth, ws, nullptr, nullptr, ws.perm, ws.slot_leaf, s, dc);
    if (rc != FFF_OK) return rc;
    if (timed) stage_mark(s);
    const bool tiles = g_opt.leaf_path != 1 && tiles_shape_ok(p) && (g_opt.leaf_path == 2 || leaf_tiles_pay(p));
    // On request ("leaf_split"), tiles whose 16 slots hold that many different leaves or more are
    // left to the gather kernel, one lane group per token, and the tile kernels keep the tiles of
    // well-filled buckets.  Not the default: on every shape measured one of the two kernels alone
    // was at least as fast as the pair.
    const int split = tiles && gather_takes_split(p) && g_opt.leaf_split >= 1 && g_opt.leaf_split <= 16
                          ? (int)g_opt.leaf_split : 0;
    g_opt.last_leaf_path = tiles ? (split ? 3 : 2) : 1;
    if (tiles) {
        e = launch_leaf_tiles(p, ws.slot_leaf, ws.perm, ws.hidden, s, timed ? stage_mark : nullptr, split);
        if (e == hipSuccess && split) e = launch_leaf_gather(p, leaf_idx, ws.perm, s, ws.slot_leaf, split);
    } else {
        e = launch_leaf_gather(p, leaf_idx, ws.perm, s);
        if (timed) stage_mark(s);
    }
    if (e != hipSuccess) return set_device_error(e, "leaf kernel launch");
    if (timed) stage_mark(s);
    return FFF_OK;
}

// The leaf networks at given leaves: small batches go one block per token, larger ones are bucketed.
int run_leaf_any(const Problem& p, const int32_t* leaf_idx, hipStream_t s) {
    if (g_opt.path != kPathStaged && token_shape_ok(p) && p.T <= 6 * g_opt.token_max_T) {
        hipError_t e = token_rows_better(p) ? launch_token_rows(p, nullptr, s, leaf_idx) : launch_token_block(p, nullptr, s, leaf_idx);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "token-block kernel launch");
    }
    Workspace ws;
    Layout lay;
    const int rc = get_workspace(p.T, p.depth, &ws, &lay, s);
    if (rc != FFF_OK) return rc;
    return run_leaf_stage(p, leaf_idx, ws, s, subtree_levels(p, true) == 0);   // falls back per shape inside
}

// How fff_forward_block's tree is cut for the grouped launches: levels from the root in one or two launches, `leaf` levels with the leaves.
struct BlockCut {
    int first = 0, second = 0, leaf = 0;
};
bool cut_at(const Problem& p, const WideNodes& wide, int leaf, BlockCut* cut) {
    const auto fits = [&](int k) { return subtree_columns(k, wide.n, 0) <= kSubtreeMaxColumns; };
    if (leaf >= p.depth || !subtree_shape_ok(p, leaf, &wide)) return false;
    const int above = p.depth - leaf;
    cut->leaf = leaf;
    cut->second = fits(above) ? 0 : above / 2;
    cut->first = above - cut->second;
    return fits(cut->first) && bucket_hist_ok(p.T, above);
}

// Estimates of both sides' time in us: sums of terms, their weights fitted to random calls of 600 to 131072 tokens that take more than 25 us
// (profiles/grouped_block_estimates.csv: 1200 calls, all cuts).  Half of the estimates are within 5 % (grouped) and 7 % (one launch).
template <int N> double weighted(const double (&weight)[N], const double (&term)[N]) {
    double t = 0;
    for (int i = 0; i < N; ++i) t += weight[i] * term[i];
    return t;
}

// The grouped launches' time goes with the tiles of each launch (a partly filled one ends every group; 512 run at a time), times the
// row's pieces of 128 bytes (more where rows do not start on lines), and the columns computed for them in blocks of 16, and the output
// row's ranges of 64 columns and their steps.
double grouped_estimate(const Problem& p, const WideNodes& wide, const BlockCut& c) {
    const auto blocks = [](int64_t cols) {
        const int64_t b = (cols + 15) / 16;
        return (double)(b <= 2 ? b : b <= 4 ? 4 : b <= 6 ? 6 : 8);
    };
    const double T = (double)p.T;
    const auto tiles = [&](int level) {         // in thousands
        const double groups = (double)((int64_t)1 << level), a_group = T / groups;
        const double t = level == 0 ? T / 64 : T / 64 + groups * (a_group < 0.5 ? a_group : 0.5);
        return 1e-3 * (t < 256 ? 256 : 0.7 * t + 0.3 * 512 * ceil(t / 512));
    };
    const double second = c.second ? 1 : 0, norm = wide.gamma ? 1 : 0, residual = p.D == p.O ? 1 : 0;   // (if it can have one)
    const double pieces = (double)((p.D * (p.bf16 ? 2 : 4) + 127) / 128), ranges = (double)((p.O + 63) / 64);
    const double parts = !wide.gamma || !p.bf16 ? 1 : subtree_row_parts(p);
    const double steps = (double)(((p.L + 1) * (1 << c.leaf) + 15) / 16);
    const double first_cols = blocks(subtree_columns(c.first, wide.n, 0)), second_cols = blocks(subtree_columns(c.second, wide.n, 0));
    const double leaf_cols = blocks(subtree_columns(c.leaf, wide.n, p.L));
    const double t1 = tiles(0), t2 = second * tiles(c.first), t3 = tiles(c.first + c.second);
    const double off_lines = p.D * (p.bf16 ? 2 : 4) % 128 ? 1 : 0, out_off_lines = p.O * (p.bf16 ? 2 : 4) % 128 ? 1 : 0;
    const double term[15] = {1, second, t1 * pieces, t1 * pieces * norm, t1 * pieces * first_cols * parts, t2 * pieces, t2 * pieces * norm,
                             t2 * pieces * second_cols * parts, t3 * pieces * leaf_cols * parts, t3 * ranges, t3 * ranges * steps,
                             t3 * ranges * residual, t1 + t2 + t3, (t1 + t2 + t3) * pieces * off_lines, t3 * ranges * out_off_lines};
    constexpr double bf16[15] = {16, 10.2, 1.32, 3.65, 0.156, 0.487, 1.84, 0.151, 0.162, 0.572, 0.488, 0.571, 8.83, 0.037, 0.491};
    constexpr double f32[15] = {19, 8.68, 0, 1.93, 1.01, 0.429, 1.09, 1.04, 1.08, 2.13, 0.324, 1.64, 7.95, 0.208, 0};
    return weighted(p.bf16 ? bf16 : f32, term);
}

// One launch a token's time goes with the pieces a lane holds of each weight row that a token meets (rows in flight together: batches), and
// with these rows' bytes, the more where all rows together outgrow an L2.  Lanes with eight pieces are the slowest.
double ungrouped_estimate(const Problem& p, const WideNodes& wide) {
    const int64_t longest = ((p.D > p.O ? p.D : p.O) * (p.bf16 ? 2 : 4) + 15) / 16;
    const bool lane_groups = longest <= 128;
    const int64_t held = (longest + (lane_groups ? 15 : 63)) / (lane_groups ? 16 : 64);
    const int64_t nv = held <= 2 ? (lane_groups ? 2 : held) : held <= 4 ? 4 : held <= 6 && lane_groups ? 6 : 8;
    const int64_t together = lane_groups ? (nv >= 6 ? 2 : 4) : nv >= 8 ? 1 : nv >= 4 ? 2 : 4;
    const bool narrow = wide.n == 1 && lane_groups;
    const int64_t node_batches = narrow ? 1 : (wide.n + together - 1) / together, node_rows = narrow ? 1 : node_batches * together;
    const int64_t leaf_rows = (p.L + together - 1) / together * together;
    const double es = p.bf16 ? 2e-6 : 4e-6, T = 1e-3 * (double)p.T, D = (double)p.D, O = (double)p.O, v = T * (double)nv, eight = nv == 8 ? 1 : 0;
    const double nodes = (double)(p.depth * node_rows), leaf = (double)leaf_rows;
    const double table = es * (wide.n * D + p.L * (D + O)) * (double)((int64_t)1 << p.depth) / 4;
    const double met = 1e3 * es * T * (p.depth * wide.n * D + p.L * (D + O));
    const double term[12] = {1, 1e3 * es * T * O, v * nodes, T * (double)(p.depth * node_batches), v * leaf, met,
                             met * (table < 4 ? table : 4), v, v * eight, v * nodes * eight, v * leaf * eight, wide.gamma ? v : 0};
    constexpr double bf16_lanes[12] = {12, 0.0931, 0.00724, 0.0115, 0.013, 0.00333, 0.0064, 0, 0.0335, 0.00328, 0.00967, 0.0703};
    constexpr double bf16_waves[12] = {12.2, 0.143, 0.0471, 0, 0.0542, 0.00712, 0.00665, 0.00999, 0.162, 0.0228, 0.0545, 0.103};
    constexpr double f32_lanes[12] = {14.5, 0.0699, 0.00321, 0.0235, 0.00777, 0.00797, 0.00538, 0, 0.0159, 0.00105, 0.00151, 0.0277};
    constexpr double f32_waves[12] = {12.4, 0.0827, 0.0362, 0, 0.0482, 0.00321, 0.00653, 0, 0.143, 0.0104, 0.0172, 0.0802};
    return p.bf16 ? weighted(lane_groups ? bf16_lanes : bf16_waves, term) : weighted(lane_groups ? f32_lanes : f32_waves, term);
}

// The grouped launches are taken where they are estimated to be 1.15 times as fast: 1199 of 6360 further random calls, 1.86 times as fast on
// average, 7 of them more than 5 % slower (50432 tokens, 768-wide, depth 8, 4 neurons a node, 8 a leaf: 219 us in one launch, 141 grouped;
// 20000 of 512 to 1600 features 209 and 72).  The cut that is estimated fastest takes 0.7 % longer than the fastest on average.
bool block_cut(const Problem& p, const WideNodes& wide, BlockCut* cut) {
    if (g_subtree == 1) return false;
    if (g_subtree >= 2) return cut_at(p, wide, (int)g_subtree - 2, cut);
    double best = ungrouped_estimate(p, wide) / 1.15;
    bool found = false;
    for (int leaf = 0; leaf <= 4; ++leaf) {
        BlockCut c;
        if (!cut_at(p, wide, leaf, &c)) continue;
        const double t = grouped_estimate(p, wide, c);
        if (t < best) best = t, *cut = c, found = true;
    }
    return found;
}

// How many levels the grouped walk goes through before it groups (of 5 .. 9 the best on average for every row length, +- 1 %).
constexpr int kGroupLevel = 6;

// The sizes whose time the estimates below were fitted to.
bool walk_grouped_range(const Problem& p) {
    const int64_t row = p.D * (p.bf16 ? 2 : 4);
    return p.depth >= 8 && p.depth <= 16 && row >= 512 && p.O <= 2 * p.D && 4 * p.O >= p.D && p.T > 32 * (int64_t)device_info().cus && grouped_shape_ok(p);
}

// Whether a call that `path` would take goes to the grouped walk instead.
//
// Below the top levels every token of the fused launch wants rows of its own, and once the tables outgrow an L2 most of them come from
// memory (16384 tokens, 4096-wide, depth 15, 4 neurons, skewed: 1636 MB moved, 236 us).  Tokens of one subtree that run on one XCD at
// the same time find them in its L2, and a row that both tokens of a wave want is fetched once (861 MB, 217 us); the price is a second
// read of the token rows and two launches more.  In the place of the split launch (65536 tokens, 768-wide, one neuron, depth 13) 101
// -> 86 us; of the staged path with more leaves than its fast bucketing takes (58703 fp32 tokens, 360-wide, depth 13, 4 neurons,
// skewed) 213 -> 100.  Not so while the tables are small against the rows (the split launch at depth 11: 69 and 71).
// By estimates in us of the grouped walk and of what the call would take, terms and weights below, fitted to 4300 random calls with
// uniform and with skewed leaves (8200 to 131072 tokens, rows of 512 bytes to 16 KB, depth 8 to 16; half of the estimates are within
// 9 % for the grouped walk and 13 % for the others).  The lines are from 7759 further calls of both sides (profiles/grouped_walk_calls.csv): where
// they lie the two take the same time on average (rows that fill their lanes badly: tiles 1.0 below the line, the others 0.97 to 1.08).  The fused launch keeps
// less than 40 MB of token rows with fewer than 0.8 tokens a leaf (0.97), the gather kernel rows that fill less than 61 % of the lanes (0.96).  Of the
// 7110 that the lines leave here, 1.17 times as fast, 218 are more than 5 % slower and 62 more than 10 %, most of them with skewed leaves, which
// spare the others' caches and which sizes do not tell.  Where the subtree launch has the lower end of the tree it stays ahead.
bool walk_grouped(const Problem& p, int path) {
    if (!launches_by_default() || (path != kPathFused && path != kPathSplit && path != kPathStaged)) return false;
    if (!walk_grouped_range(p) || (path == kPathStaged && subtree_levels(p, false) >= 0)) return false;
    const int64_t es = p.bf16 ? 2 : 4;
    const double T = (double)p.T, node = 1e-6 * (double)(p.D * es), leaf = 1e-6 * (double)((p.L * (p.D + p.O) + p.O) * es);    // MB
    const double leaves = (double)((int64_t)1 << p.depth);
    // rows that some token meets, if all leaves are as likely
    double met = leaf * leaves * (1 - exp(-T / leaves));
    for (int m = 0; m < p.depth; ++m) met += node * (double)(1 << m) * (1 - exp(-T / (double)(1 << m)));
    const double x = T * node, out = T * 1e-6 * (double)(p.O * es), leaf_rows = T * leaf;
    const bool wide = p.D * es > 2048;
    const double grouped_term[5] = {1, x, out, x * (p.depth - 6) + leaf_rows, met};
    constexpr double grouped_short[5] = {17.1, 0.348, 0.0207, 0.0493, 0.0599}, grouped_wide[5] = {19.9, 0.414, 0.0257, 0.0402, 0.0864};
    // lanes past the end of a row wait with the others (rows of 2056 bf16 features, 257 of 512 pieces: 1.23 times the fitted time)
    const int64_t pieces = p.D * es / 16;
    int64_t held = 1024;
    for (const int64_t h : {512, 256, 192, 128, 96, 64}) held = pieces <= h ? h : held;
    const double filled = (double)pieces / (double)held, waiting = 1 + 0.45 * (1 - filled), least = 0.9 * waiting > 1.05 ? 0.9 * waiting : 1.05;
    const double grouped = weighted(wide ? grouped_wide : grouped_short, grouped_term);
    if (path == kPathStaged) {
        const double term[6] = {1, x, out, x * (p.depth - 5), leaf_rows, met};
        constexpr double gather_short[6] = {16.4, 0, 0.0349, 0.143, 0.0257, 0.187}, gather_wide[6] = {14.1, 0.457, 0.0178, 0.0634, 0.0324, 0.163};
        constexpr double tiles_short[6] = {25, 0.146, 0, 0.0608, 0, 1.04}, tiles_wide[6] = {29.8, 0.671, 0.184, 0, 0.0018, 0.599};
        if (leaf_tiles_pay(p)) return weighted(wide ? tiles_wide : tiles_short, term) > (10 * p.O < 7 * p.D ? 1.12 : 1.05) * waiting * grouped;
        return !(p.depth <= 12 && filled <= 0.61 && p.L > 3) && weighted(wide ? gather_wide : gather_short, term) > least * grouped;
    }
    const double rows = x * (p.depth - 5) + leaf_rows, beyond = log2(met / 4);
    const double term[6] = {1, x, out, rows, rows * (beyond < 0 ? 0 : beyond > 4 ? 4 : beyond), met};
    constexpr double fused_short[6] = {7.56, 0.176, 0, 0.0615, 0.0037, 0.0551}, fused_wide[6] = {9.35, 0.148, 0.0916, 0.0699, 0.0023, 0.0606};
    constexpr double split_short[6] = {9.06, 0.159, 0.0822, 0.0589, 0.0029, 0.0503}, split_wide[6] = {14.8, 0.153, 0.0887, 0.0527, 0.0036, 0.0723};
    if (path == kPathSplit) return weighted(wide ? split_wide : split_short, term) > least * grouped;
    return !(x < 40 && T < 0.8 * leaves) && weighted(wide ? fused_wide : fused_short, term) > least * grouped;
}

// Scratch of the grouped launches, in words: node reached (twice), grouped order, mean and deviation of T tokens, group offsets, counts.
struct BlockScratch {
    int64_t row, groups, total;
};
BlockScratch block_scratch(int64_t T, const BlockCut& cut) {
    BlockScratch b;
    b.row = round_up(T, kAlignWords);
    b.groups = round_up(((int64_t)1 << (cut.first + cut.second)) + 1, kAlignWords);
    b.total = 5 * b.row + b.groups + kFoldWords;
    return b;
}

int run_block_grouped(const Problem& p, const WideNodes& wide, const BlockCut& cut, void* scratch, int32_t* leaf_idx, hipStream_t s) {
    const int above = cut.first + cut.second;
    const BlockScratch b = block_scratch(p.T, cut);
    Workspace ws = {};
    int32_t* const idx = (int32_t*)scratch;
    int32_t* const node = idx + b.row;                // (of the second launch from the root)
    ws.perm = node + b.row;
    float* const stats = (float*)(ws.perm + b.row);   // [T] mean and deviation
    ws.offset = (int32_t*)stats + 2 * b.row;
    DescentCounts dc;
    dc.M = ws.offset + b.groups;
    dc.capacity = kFoldWords;
    const auto bucket = [&](const int32_t* at, int depth, const DescentCounts* counts) -> hipError_t {
        return counts && counts->blocks > 0 ? launch_bucket_fold(at, p.T, depth, *counts, nullptr, ws.offset, ws.perm, nullptr, s)
                                            : launch_bucket_hist(at, p.T, depth, nullptr, ws.offset, ws.perm, nullptr, s);
    };
    hipError_t e = launch_subtree_levels(p, 0, cut.first, nullptr, nullptr, idx, s, wide, stats, &dc);
    if (e == hipSuccess) e = bucket(idx, cut.first, &dc);
    if (e == hipSuccess && cut.second) {
        e = launch_subtree_levels(p, cut.first, cut.second, ws.perm, ws.offset, node, s, wide, stats, nullptr);
        if (e == hipSuccess) e = bucket(node, above, nullptr);
    }
    if (e == hipSuccess) e = launch_subtree(p, cut.leaf, ws.perm, ws.offset, leaf_idx, s, true, &wide, stats);
    return e == hipSuccess ? FFF_OK : set_device_error(e, "block kernel launch");
}

// Whether one block a token takes a call of fff_forward_block: by estimate of what its tokens meet.
bool block_by_token(const Problem& p, int node_size, bool vector_rows) {
    // Any batch whose rows are not whole pieces when its tokens meet much: the element-wise kernel's time goes with the rows a
    // token meets times their chunks of 64 elements (generic / token block, us, 24000 tokens: 20 chunks 126/256,
    // 56 265/270, 200 955/423, 640 3940/538).
    const int64_t chunks = ((int64_t)p.depth * node_size + p.L) * ((p.D + 63) / 64);
    const bool far_rows = !vector_rows && chunks >= 80;
    // Small batches, from 480 calls of both sides: up to 256 tokens always (a token a compute unit), up to 512 unless the rows are
    // short and few (313 tokens of 112 fp32 features, 7 rows met: 5.6 / 4.5 us of the kernels below), up to 1024 where a
    // token meets enough of them: 50 short ones (932 tokens of 96, 7 rows 9.0 / 4.1; 1019 of 48 bf16, 16 rows 11.3 / 6.6),
    // 12 long ones or ones that are not whole pieces (998 of 23, 8 rows 11.4 / 7.7).
    const int64_t met = (int64_t)p.depth * node_size + p.L, small = g_opt.token_max_T;
    const bool short_rows = (p.D > p.O ? p.D : p.O) * (p.bf16 ? 2 : 4) <= 64 * 16;
    const int64_t enough = p.T <= small / 2 ? 0 : p.T <= small ? (vector_rows && short_rows ? 12 : 0)
                           : vector_rows ? (short_rows ? 50 : 12) : short_rows ? 12 : 0;
    return ((p.T <= 2 * small && met > enough) || far_rows) && token_wide_ok(p, node_size);
}

// Host-side argument checks of fff_forward_hard (no HIP call).  FFF_OK with *empty set: nothing to do.
int check_forward_hard(const void* x, const void* node_w, const void* node_b, const void* leaf_w1,
                       const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int depth, int leaf_width,
                       int act, const void* out, int64_t T, int64_t D, int64_t O, int dtype, bool* empty) {
    *empty = false;
    int rc = check_common(depth, T, D, dtype);
    if (rc == FFF_OK) rc = check_leaf(depth, leaf_width, act, T, D, O);
    if (rc != FFF_OK) return rc;
    if (T == 0) {
        *empty = true;
        return FFF_OK;
    }
    if (!x || !leaf_w1 || !leaf_b1 || !leaf_w2 || !leaf_b2 || !out) return FFF_ERR_NULL;
    if (depth > 0 && (!node_w || !node_b)) return FFF_ERR_NULL;
    const int64_t es = dtype == FFF_BF16 ? 2 : 4;
    if (overlaps(x, T * D * es, out, T * O * es)) return FFF_ERR_ALIAS;
    return FFF_OK;
}

// The address of `scratch` on the current device, asked for once per device with that device
// current (each device has its own copy of the array).
void* g_scratch_ptr[kMaxDevices];

int scratch_on_device(void** ptr) {
    int dev = 0;
    const int rc = current_device(&dev);
    if (rc != FFF_OK) return rc;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return set_device_error(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return FFF_OK;
}

// Scratch of the grouped walk, in words: the node every token reaches, the tokens in their order, the descent's counts.
int64_t walk_scratch_words(int64_t T) { return 2 * round_up(T, kAlignWords) + kFoldWords; }

// The first kGroupLevel levels for every token, the tokens grouped by the node they reach, then the rest of the fused launch in that
// order: the same bits as the fused launch.
int run_walk_grouped(const Problem& p, int32_t* leaf_idx, hipStream_t s, int32_t* node, int32_t* perm, int32_t* counts, int64_t capacity,
                     bool marks) {
    const int level = p.depth <= kGroupLevel ? p.depth - 1 : kGroupLevel;
    g_opt.last_path = kPathGrouped;
    Problem top = p;
    top.depth = level;
    DescentCounts dc;
    dc.M = counts;
    dc.capacity = capacity;
    if (marks) stage_mark(s);
    hipError_t e = launch_descend(top, node, s, &dc);
    if (e != hipSuccess) return set_device_error(e, "descent kernel launch");
    if (marks) stage_mark(s);
    e = dc.blocks > 0 ? launch_bucket_fold(node, p.T, level, dc, nullptr, nullptr, perm, nullptr, s)
                      : launch_bucket_hist(node, p.T, level, nullptr, nullptr, perm, nullptr, s);
    if (e != hipSuccess) return set_device_error(e, "bucket kernel launch");
    if (marks) stage_mark(s);
    e = launch_walk_grouped(p, level, perm, node, leaf_idx, s);
    for (int i = 0; marks && i < 2; ++i) stage_mark(s);
    return e == hipSuccess ? FFF_OK : set_device_error(e, "grouped walk kernel launch");
}

int run_walk_grouped(const Problem& p, int32_t* leaf_idx, hipStream_t s, const Workspace& ws, bool marks) {
    const int64_t words = kTilesMaxLeafWidth / 2 * p.T;
    return run_walk_grouped(p, leaf_idx, s, ws.leaf_idx, ws.perm, ws.hidden, words < kFoldWords ? words : kFoldWords, marks);
}

// The launches of Forward_I.  fixed_scratch == nullptr: the staged path works in the device's
// workspace and the stages are bracketed by events when "stage_timing" is on.  Otherwise that block
// of device memory (large enough for layout_for(T, depth): the caller has checked) is carved
// instead, its control words are cleared by a kernel first, and no event is created.
// walk_scratch: the grouped walk in this memory (walk_scratch_words) in the place of the fused launch.  Memory of this call alone: the fused
// launch needs none, and what takes its place may not allocate, fail or leave an address in a captured graph where that did not.
int run_forward_hard(const Problem& p, int32_t* leaf_idx, hipStream_t s, void* fixed_scratch, void* walk_scratch = nullptr) {
    const bool marks = fixed_scratch == nullptr;
    g_walk_tuning.last_top = 0;         // (of this call; a launch that keeps levels in LDS says so)
    int path = choose_path(p);
    if (path == kPathGrouped) {                                        // (asked for: the fused launch where there is no workspace to be had)
        Workspace ws;
        Layout lay;
        int rc = FFF_OK;
        if (fixed_scratch) carve(fixed_scratch, layout_for(p.T, p.depth), &ws);
        else rc = get_workspace(p.T, p.depth, &ws, &lay, s);
        if (rc == FFF_OK) return run_walk_grouped(p, leaf_idx, s, ws, marks);
        if (rc != FFF_ERR_WORKSPACE) return rc;
        g_last_error.clear();
        path = kPathFused;
    }
    g_opt.last_path = path == kPathWave ? (int)kPathFused : path;      // (one fused launch, whichever kernel)
    if (path == kPathGeneric) {
        // rows of at least one piece by 16-byte pieces at any element (20011 tokens of 77 features: 7.5 us against 19.8 element by
        // element); option path = 3 asks for the element-wise kernel
        hipError_t e = g_opt.path != kPathGeneric && rows_shape_ok(p) ? launch_fused_rows(p, leaf_idx, s)
                                                                   : launch_fused_generic(p, leaf_idx, s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "generic kernel launch");
    }
    if (path == kPathToken) {
        if (marks) stage_mark(s);
        hipError_t e = token_rows_better(p) ? launch_token_rows(p, leaf_idx, s) : launch_token_block(p, leaf_idx, s);
        for (int k = 0; marks && k < 4; ++k) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "token-block kernel launch");
    }
    if (walk_scratch) {
        int32_t *const node = (int32_t*)walk_scratch, *const perm = node + round_up(p.T, kAlignWords);
        return run_walk_grouped(p, leaf_idx, s, node, perm, perm + round_up(p.T, kAlignWords), kFoldWords, marks);
    }
    if (path == kPathWave) {
        if (marks) stage_mark(s);
        hipError_t e = launch_walk_wave(p, leaf_idx, s);
        for (int k = 0; marks && k < 4; ++k) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "wave kernel launch");
    }
    if (path == kPathFused) {
        if (marks) stage_mark(s);
        hipError_t e = launch_walk_fused(p, leaf_idx, s);
        for (int k = 0; marks && k < 4; ++k) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "fused walk kernel launch");
    }
    Workspace ws;
    Layout lay;
    hipError_t e;
    const bool grouped = walk_grouped(p, path);
    if (fixed_scratch) {
        lay = layout_for(p.T, p.depth);
        carve(fixed_scratch, lay, &ws);
        if (path == kPathStaged && !grouped && (e = launch_zero(ws.ctrl, kCtrlWords, s)) != hipSuccess)
            return set_device_error(e, "zero kernel launch");
    } else {
        const int rc = get_workspace(p.T, p.depth, &ws, &lay, s);
        if (rc != FFF_OK) return rc;
    }
    if (grouped) return run_walk_grouped(p, leaf_idx, s, ws, marks);
    int32_t* li = leaf_idx ? leaf_idx : ws.leaf_idx;
    if (path == kPathSplit) {
        // walk and hidden neurons per token, then the output rows by column slices; the hidden
        // activations (fp32, at most 8 a token) use the workspace's hidden-activation region
        float* hid = (float*)ws.hidden;
        if (marks) stage_mark(s);
        if ((e = launch_walk_hidden(p, li, hid, s)) != hipSuccess) return set_device_error(e, "walk kernel launch");
        for (int k = 0; marks && k < 2; ++k) stage_mark(s);
        if ((e = launch_leaf_slices(p, li, hid, s)) != hipSuccess) return set_device_error(e, "slice kernel launch");
        for (int k = 0; marks && k < 2; ++k) stage_mark(s);
        return FFF_OK;
    }
    // the descent leaves per-block leaf counts for the bucketing stage where the sizes allow it
    DescentCounts dc;
    const bool fold = g_opt.bucketing && p.depth <= 10 && (g_opt.bucket_kernel == 0 || g_opt.bucket_kernel == 5);
    dc.M = fold ? ws.fold : nullptr;
    dc.capacity = kFoldWords;
    if (marks) stage_mark(s);
    const int k = subtree_levels(p, false);
    if (k > 0) {
        Problem top = p;
        top.depth = p.depth - k;
        if ((e = launch_descend(top, ws.leaf_idx, s, &dc)) != hipSuccess) return set_device_error(e, "descent kernel launch");
        if (marks) stage_mark(s);
        const int rc = run_bucket(ws.leaf_idx, p.T, top.depth, ws, nullptr, ws.offset, ws.perm, ws.slot_leaf, s, &dc);
        if (rc != FFF_OK) return rc;
        if (marks) stage_mark(s);
        g_opt.last_leaf_path = 4;
        e = launch_subtree(p, k, ws.perm, ws.offset, leaf_idx, s, !leaf_tiles_pay(p));
        for (int i = 0; marks && i < 2; ++i) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "subtree kernel launch");
    }
    e = launch_descend(p, li, s, &dc);
    if (e != hipSuccess) return set_device_error(e, "descent kernel launch");
    if (marks) stage_mark(s);
    return run_leaf_stage(p, li, ws, s, k == 0, marks, &dc);
}

}  // namespace

void add_launch_note(const LaunchNote& note) {
    std::lock_guard<std::mutex> lock(g_notes_mu);
    if (g_n_notes == kMaxNotes) --g_n_notes;
    g_notes[g_n_notes++] = note;
}

}  // namespace fff

using namespace fff;

extern "C" {

int fff_forward_hard_scratch(const void* x, const void* node_w, const void* node_b, const void* leaf_w1,
                             const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int depth,
                             int leaf_width, int act, void* out, int32_t* leaf_idx, void* stream, int64_t T,
                             int64_t D, int64_t O, int dtype, void* scratch, size_t scratch_bytes) {
    bool empty = false;
    const int rc = check_forward_hard(x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act,
                                      out, T, D, O, dtype, &empty);
    if (rc != FFF_OK || empty) return rc;
    if (scratch) {
        const int64_t es = dtype == FFF_BF16 ? 2 : 4;
        if ((reinterpret_cast<uintptr_t>(scratch) & 255u) != 0) return FFF_ERR_WORKSPACE;
        if (overlaps(scratch, (int64_t)scratch_bytes, x, T * D * es) || overlaps(scratch, (int64_t)scratch_bytes, out, T * O * es) ||
            (leaf_idx && overlaps(scratch, (int64_t)scratch_bytes, leaf_idx, T * 4)))
            return FFF_ERR_ALIAS;
    }
    Problem p{x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, leaf_idx,
              T, D, O, depth, leaf_width, act, dtype == FFF_BF16};
    const bool grouped = scratch && choose_path(p) == kPathFused && walk_grouped(p, kPathFused);
    const size_t need = (size_t)walk_scratch_words(T) * sizeof(int32_t);
    if (grouped && scratch_bytes < need) {
        g_last_error = "the scratch holds " + std::to_string(scratch_bytes) + " bytes, this call needs " + std::to_string(need);
        return FFF_ERR_WORKSPACE;
    }
    begin_device_call();
    return run_forward_hard(p, leaf_idx, (hipStream_t)stream, nullptr, grouped ? scratch : nullptr);
}

int fff_forward_hard(const void* x, const void* node_w, const void* node_b, const void* leaf_w1,
                     const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int depth,
                     int leaf_width, int act, void* out, int32_t* leaf_idx, void* stream, int64_t T,
                     int64_t D, int64_t O, int dtype) {
    return fff_forward_hard_scratch(x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act, out, leaf_idx, stream, T,
                                    D, O, dtype, nullptr, 0);
}

size_t fff_hard_scratch_bytes(int64_t T, int64_t D, int64_t O, int depth, int leaf_width, int dtype) {
    if (check_common(depth, T, D, dtype) != FFF_OK || check_leaf(depth, leaf_width, 0, T, D, O) != FFF_OK || T == 0) return 0;
    Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
              T, D, O, depth, leaf_width, 0, dtype == FFF_BF16};
    return walk_grouped_range(p) && choose_path(p) == kPathFused && walk_grouped(p, kPathFused)
               ? (size_t)walk_scratch_words(T) * sizeof(int32_t) : 0;
}

int fff_forward_hard_static(const void* x, const void* node_w, const void* node_b, const void* leaf_w1,
                            const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int depth,
                            int leaf_width, int act, void* out, int32_t* leaf_idx, void* stream, int64_t T,
                            int64_t D, int64_t O, int dtype) {
    bool empty = false;
    const int rc = check_forward_hard(x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act,
                                      out, T, D, O, dtype, &empty);
    if (rc != FFF_OK || empty) return rc;
    const size_t need = (size_t)layout_for(T, depth).total * sizeof(int32_t);
    if (need > FFF_STATIC_SCRATCH_BYTES) {
        g_last_error = "fff_forward_hard_static: T = " + std::to_string(T) + ", depth = " + std::to_string(depth) +
                       " need " + std::to_string(need) + " bytes of scratch, the static array holds " +
                       std::to_string((size_t)FFF_STATIC_SCRATCH_BYTES);
        return FFF_ERR_WORKSPACE;
    }
    Problem p{x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, leaf_idx,
              T, D, O, depth, leaf_width, act, dtype == FFF_BF16};
    begin_device_call();
    void* ptr = nullptr;
    const int rs = scratch_on_device(&ptr);
    if (rs != FFF_OK) return rs;
    return run_forward_hard(p, leaf_idx, (hipStream_t)stream, ptr);
}

size_t fff_static_scratch_bytes(void) { return FFF_STATIC_SCRATCH_BYTES; }

int fff_descend(const void* x, const void* node_w, const void* node_b, int depth, int32_t* leaf_idx,
                void* stream, int64_t T, int64_t D, int dtype) {
    int rc = check_common(depth, T, D, dtype);
    if (rc != FFF_OK) return rc;
    if (T == 0) return FFF_OK;
    if (!x || !leaf_idx) return FFF_ERR_NULL;
    if (depth > 0 && (!node_w || !node_b)) return FFF_ERR_NULL;
    Problem p{x, node_w, node_b, nullptr, nullptr, nullptr, nullptr, nullptr, leaf_idx,
              T, D, 1, depth, 1, 0, dtype == FFF_BF16};
    begin_device_call();
    hipError_t e = launch_descend(p, leaf_idx, (hipStream_t)stream);
    return e == hipSuccess ? FFF_OK : set_device_error(e, "descent kernel launch");
}

int fff_bucket(const int32_t* leaf_idx, int64_t T, int depth, int32_t* count, int32_t* offset,
               int32_t* perm, void* stream) {
    if (depth < 0 || depth > FFF_MAX_DEPTH || T < 0 || T > kMaxTokens) return FFF_ERR_RANGE;
    if (T > 0 && !leaf_idx) return FFF_ERR_NULL;
    begin_device_call();
    Workspace ws;
    Layout lay;
    int rc = get_workspace(T, depth, &ws, &lay, (hipStream_t)stream);
    if (rc != FFF_OK) return rc;
    return run_bucket(leaf_idx, T, depth, ws, count, offset, perm, nullptr, (hipStream_t)stream);
}

int fff_leaf_forward(const void* x, const void* leaf_w1, const void* leaf_b1, const void* leaf_w2,
                     const void* leaf_b2, const int32_t* leaf_idx, int depth, int leaf_width, int act,
                     void* out, void* stream, int64_t T, int64_t D, int64_t O, int dtype) {
    int rc = check_common(depth, T, D, dtype);
    if (rc == FFF_OK) rc = check_leaf(depth, leaf_width, act, T, D, O);
    if (rc != FFF_OK) return rc;
    if (T == 0) return FFF_OK;
    if (!x || !leaf_w1 || !leaf_b1 || !leaf_w2 || !leaf_b2 || !out || !leaf_idx) return FFF_ERR_NULL;
    const int64_t es = dtype == FFF_BF16 ? 2 : 4;
    if (overlaps(x, T * D * es, out, T * O * es)) return FFF_ERR_ALIAS;
    Problem p{x, nullptr, nullptr, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, nullptr,
              T, D, O, depth, leaf_width, act, dtype == FFF_BF16};
    begin_device_call();
    return run_leaf_any(p, leaf_idx, (hipStream_t)stream);
}

int fff_moe_top1_forward(const void* x, const void* gate_w, const void* gate_b, const void* leaf_w1,
                         const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int log2_experts,
                         int leaf_width, int act, void* out, int32_t* expert_idx, void* stream, int64_t T,
                         int64_t D, int64_t O, int dtype) {
    int rc = check_common(log2_experts, T, D, dtype);
    if (rc == FFF_OK) rc = check_leaf(log2_experts, leaf_width, act, T, D, O);
    if (rc != FFF_OK) return rc;
    if (T == 0) return FFF_OK;
    if (!x || !gate_w || !leaf_w1 || !leaf_b1 || !leaf_w2 || !leaf_b2 || !out) return FFF_ERR_NULL;
    const int64_t es = dtype == FFF_BF16 ? 2 : 4;
    if (overlaps(x, T * D * es, out, T * O * es)) return FFF_ERR_ALIAS;
    if (!moe_gate_shape_ok(x, gate_w, D, dtype == FFF_BF16)) return FFF_ERR_UNSUPPORTED;
    const int64_t G = (int64_t)1 << log2_experts;
    Problem p{x, nullptr, nullptr, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, nullptr,
              T, D, O, log2_experts, leaf_width, act, dtype == FFF_BF16};
    begin_device_call();
    hipStream_t s = (hipStream_t)stream;
    Workspace ws;
    Layout lay;
    if ((rc = get_workspace(T, log2_experts, &ws, &lay, s, moe_gate_words(T, G))) != FFF_OK) return rc;
    int32_t* ei = expert_idx ? expert_idx : ws.leaf_idx;
    stage_mark(s);
    GateCandidates gate;
    hipError_t e = launch_moe_gate(x, gate_w, gate_b, T, D, G, ws.extra, &gate, s);
    if (e != hipSuccess) return set_device_error(e, "gating kernel launch");
    // the experts are leaves: small batches one block per token (token_block_kernel picks the expert by itself), larger ones bucketed
    const bool small = g_opt.path != kPathStaged && token_shape_ok(p) && T <= 6 * g_opt.token_max_T;
    const bool picks = small && !token_rows_better(p, true);
    if (!picks && (e = launch_moe_pick(gate, T, ei, s)) != hipSuccess) return set_device_error(e, "gating kernel launch");
    stage_mark(s);
    if (small) {
        g_opt.last_path = kPathToken;
        e = picks ? launch_token_block(p, expert_idx, s, nullptr, &gate) : launch_token_rows(p, nullptr, s, ei);
        for (int k = 0; k < 3; ++k) stage_mark(s);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "token-block kernel launch");
    }
    g_opt.last_path = kPathStaged;
    return run_leaf_stage(p, ei, ws, s, subtree_levels(p, true) == 0, true);
}

int fff_forward_soft(const void* x, const void* node_w, const void* node_b, const void* leaf_w1,
                     const void* leaf_b1, const void* leaf_w2, const void* leaf_b2, int depth, int leaf_width,
                     int act, void* out, float* mix, float* entropy, void* stream, int64_t T, int64_t D,
                     int64_t O, int dtype) {
    int rc = check_common(depth, T, D, dtype);
    if (rc == FFF_OK) rc = check_leaf(depth, leaf_width, act, T, D, O);
    if (rc != FFF_OK) return rc;
    if (T == 0) return FFF_OK;
    if (!x || !leaf_w1 || !leaf_b1 || !leaf_w2 || !leaf_b2 || !out) return FFF_ERR_NULL;
    if (depth > 0 && (!node_w || !node_b)) return FFF_ERR_NULL;
    const int64_t es = dtype == FFF_BF16 ? 2 : 4;
    if (overlaps(x, T * D * es, out, T * O * es)) return FFF_ERR_ALIAS;
    Problem p{x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, nullptr,
              T, D, O, depth, leaf_width, act, dtype == FFF_BF16};
    if (!soft_shape_ok(p)) return FFF_ERR_UNSUPPORTED;
    // every token meets every leaf: the intermediate matrices are T x 2^depth x (leaf_width + 1) wide
    const int64_t words = soft_scratch_words(p);
    if (words > kMaxElems / 4) return FFF_ERR_SHAPE;
    begin_device_call();
    Workspace ws;
    Layout lay;
    if ((rc = get_workspace(0, 0, &ws, &lay, (hipStream_t)stream, words)) != FFF_OK) return rc;
    hipError_t e = launch_forward_soft(p, ws.extra, mix, entropy, (hipStream_t)stream);
    return e == hipSuccess ? FFF_OK : set_device_error(e, "soft forward kernel launch");
}

int fff_forward_block_scratch(const void* x, const void* ln_gamma, const void* ln_beta, float ln_eps,
                              const void* node_w1, const void* node_b1, const void* node_w2, const void* node_b2,
                              const void* leaf_w1, const void* leaf_b1, const void* leaf_w2, const void* leaf_b2,
                              int depth, int node_size, int leaf_width, int act, int residual, void* out,
                              int32_t* leaf_idx, void* stream, int64_t T, int64_t D, int64_t O, int dtype,
                              void* scratch, size_t scratch_bytes) {
    int rc = check_common(depth, T, D, dtype);
    if (rc == FFF_OK) rc = check_leaf(depth, leaf_width, act, T, D, O);
    if (rc != FFF_OK) return rc;
    if (node_size < 1 || node_size > kMaxLeafWidth) return FFF_ERR_RANGE;
    if ((((int64_t)1 << depth) - 1) * node_size > kMaxElems / D) return FFF_ERR_SHAPE;
    if (residual && O != D) return FFF_ERR_SHAPE;
    if ((ln_gamma != nullptr) != (ln_beta != nullptr)) return FFF_ERR_NULL;
    if (ln_gamma && !(ln_eps >= 0.0f)) return FFF_ERR_RANGE;
    if (T == 0) return FFF_OK;
    if (!x || !leaf_w1 || !leaf_b1 || !leaf_w2 || !leaf_b2 || !out) return FFF_ERR_NULL;
    if (depth > 0 && (!node_w1 || !node_b1 || !node_w2 || !node_b2)) return FFF_ERR_NULL;
    const int64_t es = dtype == FFF_BF16 ? 2 : 4;
    // in place (out == x with rows of one width) is fine: a wave reads its token before it writes it
    if (!(out == x && O == D) && overlaps(x, T * D * es, out, T * O * es)) return FFF_ERR_ALIAS;
    if (leaf_idx && overlaps(leaf_idx, T * 4, out, T * O * es)) return FFF_ERR_ALIAS;
    if (scratch) {
        if ((reinterpret_cast<uintptr_t>(scratch) & 255u) != 0) return FFF_ERR_WORKSPACE;
        if (overlaps(scratch, (int64_t)scratch_bytes, x, T * D * es) || overlaps(scratch, (int64_t)scratch_bytes, out, T * O * es) ||
            (leaf_idx && overlaps(scratch, (int64_t)scratch_bytes, leaf_idx, T * 4)))
            return FFF_ERR_ALIAS;
    }
    Problem p{x, nullptr, nullptr, leaf_w1, leaf_b1, leaf_w2, leaf_b2, out, leaf_idx,
              T, D, O, depth, leaf_width, act, dtype == FFF_BF16};
    WideNodes wide;
    wide.gamma = ln_gamma;
    wide.beta = ln_beta;
    wide.w1 = node_w1;
    wide.b1 = node_b1;
    wide.w2 = node_w2;
    wide.b2 = node_b2;
    wide.n = node_size;
    wide.residual = residual != 0;
    wide.eps = ln_eps;
    // rows of whole 16-byte pieces, short enough for a lane group or a wave to hold, take the vector
    // kernels; everything else the element-wise one
    const bool vector_rows = block_shape_ok(x, out, leaf_w1, leaf_w2, D, O, p.bf16) &&
                             (depth == 0 || vec_ok(node_w1, D, p.bf16)) &&
                             (!ln_gamma || (vec_ok(ln_gamma, D, p.bf16) && vec_ok(ln_beta, D, p.bf16))) &&
                             vec_ok(leaf_b2, O, p.bf16);
    const bool by_token = block_by_token(p, node_size, vector_rows);
    BlockCut cut;
    const bool grouped = scratch && vector_rows && !by_token && block_cut(p, wide, &cut);
    if (grouped && scratch_bytes < (size_t)block_scratch(T, cut).total * sizeof(int32_t)) {
        g_last_error = "the scratch holds " + std::to_string(scratch_bytes) + " bytes, this call needs " +
                       std::to_string((size_t)block_scratch(T, cut).total * sizeof(int32_t));
        return FFF_ERR_WORKSPACE;
    }
    begin_device_call();
    g_opt.last_block_kernel = vector_rows ? 1 : 2;
    g_block_tuning.last_top = 0;        // (of this call; the lane groups say what they keep)
    if (by_token) {
        hipError_t e = launch_token_block(p, leaf_idx, (hipStream_t)stream, nullptr, nullptr, &wide);
        return e == hipSuccess ? FFF_OK : set_device_error(e, "token-block kernel launch");
    }
    if (grouped) return run_block_grouped(p, wide, cut, scratch, leaf_idx, (hipStream_t)stream);
    hipError_t e = launch_forward_block(p, ln_gamma, ln_beta, ln_eps, node_w1, node_b1, node_w2, node_b2,
                                        node_size, residual != 0, leaf_idx, (hipStream_t)stream, vector_rows);
    return e == hipSuccess ? FFF_OK : set_device_error(e, "block kernel launch");
}

int fff_forward_block(const void* x, const void* ln_gamma, const void* ln_beta, float ln_eps,
                      const void* node_w1, const void* node_b1, const void* node_w2, const void* node_b2,
                      const void* leaf_w1, const void* leaf_b1, const void* leaf_w2, const void* leaf_b2,
                      int depth, int node_size, int leaf_width, int act, int residual, void* out,
                      int32_t* leaf_idx, void* stream, int64_t T, int64_t D, int64_t O, int dtype) {
    return fff_forward_block_scratch(x, ln_gamma, ln_beta, ln_eps, node_w1, node_b1, node_w2, node_b2, leaf_w1, leaf_b1, leaf_w2, leaf_b2,
                                     depth, node_size, leaf_width, act, residual, out, leaf_idx, stream, T, D, O, dtype, nullptr, 0);
}

size_t fff_block_scratch_bytes(int64_t T, int64_t D, int64_t O, int depth, int node_size, int leaf_width, int norm, int dtype) {
    if (check_common(depth, T, D, dtype) != FFF_OK || check_leaf(depth, leaf_width, 0, T, D, O) != FFF_OK || T == 0 || depth == 0 ||
        node_size < 1 || node_size > kMaxLeafWidth)
        return 0;
    Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
              T, D, O, depth, leaf_width, 0, dtype == FFF_BF16};
    alignas(16) static const char some[16] = {};       // (asked for alignment only)
    WideNodes wide;
    wide.gamma = wide.beta = norm ? some : nullptr;
    wide.n = node_size;
    BlockCut cut;
    if (!block_shape_ok(nullptr, nullptr, nullptr, nullptr, D, O, p.bf16) || block_by_token(p, node_size, true) || !block_cut(p, wide, &cut))
        return 0;
    return (size_t)block_scratch(T, cut).total * sizeof(int32_t);
}

size_t fff_workspace_bytes(int64_t T, int depth) {
    if (T < 0 || T > kMaxTokens || depth < 0 || depth > FFF_MAX_DEPTH) return 0;
    return (size_t)layout_for(T, depth).total * sizeof(int32_t);
}

size_t fff_workspace_bytes_moe(int64_t T, int log2_experts) {
    if (T < 0 || T > kMaxTokens || log2_experts < 0 || log2_experts > FFF_MAX_DEPTH) return 0;
    const int64_t G = (int64_t)1 << log2_experts;
    return (size_t)layout_for(T, log2_experts, moe_gate_words(T, G)).total * sizeof(int32_t);
}

size_t fff_workspace_bytes_soft(int64_t T, int64_t O, int depth, int leaf_width) {
    if (T < 0 || T > kMaxTokens || depth < 0 || depth > FFF_MAX_DEPTH || O < 1 || O > kMaxElems ||
        leaf_width < 1 || leaf_width > kMaxLeafWidth)
        return 0;
    Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
              T, 8, O, depth, leaf_width, 0, true};
    const int64_t words = soft_scratch_words(p);
    if (words > kMaxElems / 4) return 0;
    return (size_t)layout_for(0, 0, words).total * sizeof(int32_t);
}

int fff_set_workspace(void* dev_ptr, size_t bytes, void* stream) {
    if (dev_ptr && ((reinterpret_cast<uintptr_t>(dev_ptr) & 255u) != 0 || bytes < kCtrlWords * sizeof(int32_t)))
        return FFF_ERR_WORKSPACE;
    begin_device_call();
    int dev = 0;
    int rc = current_device(&dev);
    if (rc != FFF_OK) return rc;
    if (dev_ptr) {   // ticket counters start at zero (a fill kernel: a memset node does not belong in a graph)
        hipError_t e = launch_zero((int32_t*)dev_ptr, kCtrlWords, (hipStream_t)stream);
        if (e != hipSuccess) return set_device_error(e, "zero kernel launch");
    }
    std::lock_guard<std::mutex> lock(g_mu);
    g_ws[dev].user_base = dev_ptr;
    g_ws[dev].user_bytes = dev_ptr ? bytes : 0;
    return FFF_OK;
}

int fff_reserve_workspace_bytes(size_t bytes) {
    begin_device_call();
    int dev = 0;
    int rc = current_device(&dev);
    if (rc != FFF_OK) return rc;
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_ws[dev].user_base) {
        g_last_error = "a caller-provided workspace is set on this device";
        return FFF_ERR_WORKSPACE;
    }
    return grow_owned(g_ws[dev], bytes, nullptr, false);
}

int fff_reserve_workspace(int64_t T, int depth) {
    if (T < 0 || T > kMaxTokens || depth < 0 || depth > FFF_MAX_DEPTH) return FFF_ERR_RANGE;
    return fff_reserve_workspace_bytes(fff_workspace_bytes(T, depth));
}

int fff_release_workspace(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess) return FFF_ERR_DEVICE;
    int rc = FFF_OK;
    for (int d = 0; d < kMaxDevices; ++d) {
        if (!g_ws[d].base) continue;
        if (hipSetDevice(d) != hipSuccess || hipFree(g_ws[d].base) != hipSuccess) rc = FFF_ERR_DEVICE;
        g_ws[d].base = nullptr;
        g_ws[d].bytes = 0;
    }
    (void)hipSetDevice(cur);
    return rc;
}

static int64_t* option_slot(const char* name) {
    if (!name) return nullptr;
    if (!std::strcmp(name, "path")) return &g_opt.path;
    if (!std::strcmp(name, "leaf_path")) return &g_opt.leaf_path;
    if (!std::strcmp(name, "bucketing")) return &g_opt.bucketing;
    if (!std::strcmp(name, "stage_timing")) return &g_opt.stage_timing;
    if (!std::strcmp(name, "last_path")) return &g_opt.last_path;
    if (!std::strcmp(name, "last_leaf_path")) return &g_opt.last_leaf_path;
    if (!std::strcmp(name, "last_walk_top")) return &g_walk_tuning.last_top;
    if (!std::strcmp(name, "last_block_kernel")) return &g_opt.last_block_kernel;
    if (!std::strcmp(name, "last_block_top")) return &g_block_tuning.last_top;
    return nullptr;
}

// Experiment switches (fff_debug_option); 0 = the built-in choice everywhere.
//   "token_max_T"    batches of up to this many tokens take the one-block-per-token launch (6 times
//                    that where leaf_width > 8 rules out the fused launch, half of it and 36 a
//                    neuron for rows that are not whole pieces); default 512
//   "walk_tpg", "walk_block", "walk_top", "walk_bpc", "walk_prefetch"
//                    descent / fused kernel: tokens per lane group, threads per block, k + 1 = at most
//                    k LDS-staged levels, persistent blocks per compute unit, next-tile prefetch;
//                    combinations the kernel is not built for are ignored
//   "block_top"      fff_forward_block, persistent launch: k + 1 = at most k node levels in LDS
//   "leaf_split"     staged leaf stage on the tile kernels: 1..16 = a tile (16 consecutive slots of the
//                    bucketed order) with at least this many runs of equal leaf goes to the gather
//                    kernel instead; 0 or above 16 = no split
//   "subtree"        the launch that takes the last levels, the leaf and the output rows of grouped tokens (fff_forward_hard's
//                    staged path, fff_forward_block): 0 = by size, 1 = never, k + 2 = with k of the last levels wherever the shape allows it
//   "bucket_kernel"  0 = choose by size (the token-chunk kernel up to 131072 tokens and 4096 leaves;
//                    beyond that the segment kernels for up to 4096 leaves, else the leaf-range kernel
//                    up to 2^21 tokens and 2^19 leaves, else the chunk-matrix kernels), 1 = the
//                    leaf-range kernel, 2 = the chunk-matrix kernels, 3 = the token-chunk kernel,
//                    4 = the segment kernels, 5 = the fold kernel on per-block leaf counts (the
//                    descent's inside fff_forward_hard, a counting launch's otherwise; up to 1024
//                    leaves and 1024 tokens a block), each when the sizes allow it; 0 also takes
//                    the fold kernel whenever the descent has left counts
//   "fail_workspace_growth" n = the next n growths of the library's own workspace fail as if the device
//                    were out of memory (FFF_ERR_WORKSPACE; the call after them allocates again)
//   "soft_small_tiles" fff_forward_soft: 1 = the 64 x 128 MFMA tile for every contraction (from 2048 tokens on, up to
//                    255 nodes, the 128-row nodes + mixture launch), 2 = the small-batch kernels (slices of K) wherever
//                    they fit, 0 = by estimated time
//   "token_kernel"   one block per token: 1 = token_block_kernel, 2 = token_rows_kernel (for the rows it takes)
//   "walk_plain_x"   the descent reads token rows 1 = without the streaming hint, 2 = with it,
//                    0 = without it while the batch fits half the last-level cache
static int64_t* debug_slot(const char* name) {
    if (!name) return nullptr;
    if (!std::strcmp(name, "token_max_T")) return &g_opt.token_max_T;
    if (!std::strcmp(name, "token_kernel")) return &g_token_kernel;
    if (!std::strcmp(name, "walk_tpg")) return &g_walk_tuning.tpg;
    if (!std::strcmp(name, "walk_block")) return &g_walk_tuning.block;
    if (!std::strcmp(name, "walk_top")) return &g_walk_tuning.top;
    if (!std::strcmp(name, "walk_bpc")) return &g_walk_tuning.bpc;
    if (!std::strcmp(name, "walk_prefetch")) return &g_walk_tuning.prefetch;
    if (!std::strcmp(name, "walk_plain_x")) return &g_walk_tuning.plain_x;
    if (!std::strcmp(name, "block_top")) return &g_block_tuning.top;
    if (!std::strcmp(name, "leaf_split")) return &g_opt.leaf_split;
    if (!std::strcmp(name, "subtree")) return &g_subtree;
    if (!std::strcmp(name, "bucket_kernel")) return &g_opt.bucket_kernel;
    if (!std::strcmp(name, "soft_small_tiles")) return &g_soft_small_tiles;
    if (!std::strcmp(name, "fail_workspace_growth")) return &g_fail_growths;
    return nullptr;
}

int fff_set_option(const char* name, int64_t value) {
    int64_t* s = option_slot(name);
    if (!s || value < 0) return FFF_ERR_UNSUPPORTED;
    if (s == &g_opt.last_path || s == &g_opt.last_leaf_path || s == &g_walk_tuning.last_top ||
        s == &g_opt.last_block_kernel || s == &g_block_tuning.last_top)
        return FFF_ERR_UNSUPPORTED;   // read-only
    *s = value;
    return FFF_OK;
}

int fff_get_option(const char* name, int64_t* value) {
    int64_t* s = option_slot(name);
    if (!s) return FFF_ERR_UNSUPPORTED;
    if (!value) return FFF_ERR_NULL;
    *value = *s;
    return FFF_OK;
}

int fff_debug_option(const char* name, int64_t value, int64_t* current) {
    int64_t* s = debug_slot(name);
    if (!s) return FFF_ERR_UNSUPPORTED;
    if (value >= 0) *s = value;
    if (current) *current = *s;
    return FFF_OK;
}

int fff_stage_times(double* ms, int64_t* calls) {
    if (!ms || !calls) return FFF_ERR_NULL;
    std::vector<hipEvent_t> ev;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        ev.swap(g_stage_events);
    }
    for (int k = 0; k < 4; ++k) ms[k] = 0.0;
    *calls = 0;
    int rc = FFF_OK;
    for (size_t i = 0; i + 4 < ev.size(); i += 5) {
        if (hipEventSynchronize(ev[i + 4]) != hipSuccess) { rc = FFF_ERR_DEVICE; break; }
        float d[4];
        bool ok = true;
        for (int k = 0; k < 4; ++k) ok = ok && hipEventElapsedTime(&d[k], ev[i + k], ev[i + k + 1]) == hipSuccess;
        if (!ok) { rc = FFF_ERR_DEVICE; break; }
        for (int k = 0; k < 4; ++k) ms[k] += d[k];
        *calls += 1;
    }
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    return rc;
}

const char* fff_status_string(int status) {
    switch (status) {
        case FFF_OK: return "ok";
        case FFF_ERR_NULL: return "a required pointer is NULL";
        case FFF_ERR_SHAPE: return "sizes are inconsistent or out of the supported range";
        case FFF_ERR_DTYPE: return "unknown dtype";
        case FFF_ERR_RANGE: return "depth, leaf_width or T out of range";
        case FFF_ERR_UNSUPPORTED: return "unknown activation or option";
        case FFF_ERR_WORKSPACE: return "workspace too small, misaligned or not allocatable";
        case FFF_ERR_DEVICE: return "a HIP call failed";
        case FFF_ERR_ALIAS: return "out overlaps x";
        default: return "unknown status";
    }
}

const char* fff_last_device_error(void) { return g_last_error.c_str(); }

const char* fff_last_launch(void) {
    static thread_local std::string text;   // each caller its own: the pointer stays good while others ask
    text.clear();
    std::lock_guard<std::mutex> lock(g_notes_mu);
    for (int i = 0; i < g_n_notes; ++i) {
        if (i) text += " + ";
        int arg = 0;
        for (const char* c = g_notes[i].fmt; *c; ++c) {
            if (c[0] != '%') {
                text += *c;
            } else if (*++c == 's') {
                text += (const char*)g_notes[i].args[arg++];
            } else {
                text += std::to_string((long long)g_notes[i].args[arg++]);
            }
        }
    }
    return text.c_str();
}

int fff_version(void) { return 300; }

}  // extern "C"
