// A wave a token, for batches between the block-a-token launches and the streaming ones (up to 48 tokens a compute unit).
//
// Such a batch is a chain of dependent trips to L2, one a level in walk_kernel, whose tiles of 32 tokens also leave most compute
// units idle.  Here a block holds few tokens (4 at least: a block for every compute unit from four tokens a unit on), and a trip
// takes as much of the chain as the registers hold:
//   - where more than eight tokens a compute unit share them, the rows of the first levels travel to LDS beside the token's own row, one trip for both;
//   - below them (or from the root) a trip takes two levels: a node's row and those of both its children, which lie side by side in heap order;
//   - the leaf's first neurons, its biases and its first output weights are requested together.
// A token's sums are taken over 64 lanes; the activations of a leaf are kept one a lane and evaluated once for all.
//
// What bounds it: the trips (2048 bf16 tokens of 768, depth 11, one neuron: 10.4 us in walk_kernel, 8.4 here), and with wider leaves the
// rows of each token through the L1s (4096 fp32 tokens of 784, depth 6, 4 neurons: 14.7 -> 9.9 us, 0.5 MB of rows a compute unit).
#include "fff_device.h"
#include "fff_internal.h"

namespace fff {
namespace {

struct WaveArgs {
    const uint4* x;
    const uint4* node_w;
    const void* node_b;
    const uint4* w1;
    const void* b1;
    const void* w2;
    const void* b2;
    void* out;
    int32_t* leaf_idx;    // may be null
    int64_t T, O;
    int depth, top, nvec, L, act;
};

// waves (tokens) of a block: what leaves the registers for two levels of rows of NV pieces a lane
constexpr int max_waves(int nv) { return nv <= 4 ? 16 : 8; }
constexpr int kMaxNeurons = 64;        // a lane each
constexpr int kAhead = 4;              // output weight rows requested together

// this lane's part of x . row (zero past the row in x and in row)
template <bool BF16, int NV> __device__ __forceinline__ float part_dot(const uint4 (&x)[NV], const uint4 (&w)[NV]) {
    float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (i & 1) acc1 = Elem<BF16>::dot(x[i], w[i], acc1);
        else acc0 = Elem<BF16>::dot(x[i], w[i], acc0);
    }
    return acc0 + acc1;
}

// What a lane holds of an output row at a time: a piece of 16 bytes, or (rows that are not whole pieces) one element.
template <bool BF16, bool PIECES> struct OutUnit;
template <bool BF16> struct OutUnit<BF16, true> {
    static constexpr int kElems = Elem<BF16>::kPerVec;
    uint4 v;
    __device__ __forceinline__ void load(const void* p, int64_t unit) { v = ((const uint4*)p)[unit]; }
    __device__ __forceinline__ void get(float* f) const { widen<BF16>(v, f); }
    static __device__ __forceinline__ void store(void* p, int64_t unit, const float* f) { store_stream((uint4*)p + unit, narrow<BF16>(f)); }
};
template <bool BF16> struct OutUnit<BF16, false> {
    static constexpr int kElems = 1;
    typename Elem<BF16>::type v;
    __device__ __forceinline__ void load(const void* p, int64_t unit) { v = ((const typename Elem<BF16>::type*)p)[unit]; }
    __device__ __forceinline__ void get(float* f) const { f[0] = Elem<BF16>::load(&v, 0); }
    static __device__ __forceinline__ void store(void* p, int64_t unit, const float* f) { Elem<BF16>::store(p, unit, f[0]); }
};

// NV: 16-byte pieces of a row a lane holds.  PIECES: output rows are whole pieces.
template <bool BF16, int NV, bool PIECES>
__global__ __launch_bounds__(max_waves(NV) * kWave) void walk_wave_kernel(const WaveArgs a) {
    extern __shared__ uint4 lds[];                  // [(2^top - 1) * nvec] rows, then as many biases
    constexpr int kRows = NV == 1 ? 8 : NV == 4 && PIECES ? 3 : 4;      // neurons of a trip
    typedef OutUnit<BF16, PIECES> Unit;
    const int lane = threadIdx.x & (kWave - 1), nvec = a.nvec, n_top = (1 << a.top) - 1;
    const int64_t mine = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    const bool live = mine < a.T;
    const int64_t t = live ? mine : a.T - 1;
    const auto request = [&](const uint4* row, uint4 (&v)[NV]) {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = row[lane + i * kWave < nvec ? lane + i * kWave : nvec - 1];
    };
    const auto trim = [&](uint4 (&v)[NV]) {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = keep_if(lane + i * kWave < nvec, v[i]);
    };
    uint4 xv[NV];
    request(a.x + t * nvec, xv);
    {
        const int n = n_top * nvec, step = blockDim.x;
        for (int i0 = threadIdx.x; i0 < n; i0 += 4 * step) {
            uint4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = a.node_w[i0 + i * step < n ? i0 + i * step : n - 1];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i0 + i * step < n) lds[i0 + i * step] = v[i];
        }
    }
    float* const lds_bias = (float*)(lds + (int64_t)n_top * nvec);
    for (int i = threadIdx.x; i < n_top; i += blockDim.x) lds_bias[i] = Elem<BF16>::load(a.node_b, i);
    __syncthreads();
    trim(xv);

    int node = 0;
    for (int m = 0; m < a.top; ++m) {
        uint4 w[NV];
        request(lds + node * nvec, w);
        const float bias = lds_bias[node];
        trim(w);
        const float logit = wave_sum(part_dot<BF16, NV>(xv, w)) + bias;
        node = __builtin_amdgcn_readfirstlane(2 * node + 1 + (logit >= 0.0f ? 1 : 0));
    }
    int m = a.top;
    if ((a.depth - m) & 1) {
        uint4 w[NV];
        request(a.node_w + (int64_t)node * nvec, w);
        const float bias = Elem<BF16>::load(a.node_b, node);
        trim(w);
        const float logit = wave_sum(part_dot<BF16, NV>(xv, w)) + bias;
        node = __builtin_amdgcn_readfirstlane(2 * node + 1 + (logit >= 0.0f ? 1 : 0));
        ++m;
    }
    for (; m < a.depth; m += 2) {
        const int64_t child = 2 * (int64_t)node + 1;
        uint4 w0[NV], w1[NV], w2[NV];
        request(a.node_w + (int64_t)node * nvec, w0);
        request(a.node_w + child * nvec, w1);
        request(a.node_w + (child + 1) * nvec, w2);
        const float b0 = Elem<BF16>::load(a.node_b, node), b1 = Elem<BF16>::load(a.node_b, child), b2 = Elem<BF16>::load(a.node_b, child + 1);
        trim(w0);
        trim(w1);
        trim(w2);
        const float s0 = wave_sum(part_dot<BF16, NV>(xv, w0)) + b0;
        const float s1 = wave_sum(part_dot<BF16, NV>(xv, w1)) + b1;
        const float s2 = wave_sum(part_dot<BF16, NV>(xv, w2)) + b2;
        const bool right = s0 >= 0.0f;
        const int next = (int)child + (right ? 1 : 0);
        node = __builtin_amdgcn_readfirstlane(2 * next + 1 + ((right ? s2 : s1) >= 0.0f ? 1 : 0));
    }
    const int64_t leaf = node - ((1 << a.depth) - 1);
    if (a.leaf_idx && live && lane == 0) a.leaf_idx[t] = (int32_t)leaf;

    const int L = a.L, units = (int)(a.O / Unit::kElems);
    const auto row_of = [&](int r) { return (leaf * L + (r < L ? r : L - 1)) * units; };
    // the leaf's first output weights and everything of its first neurons
    Unit bias, out_w[kAhead];
    const auto request_bias = [&](int u) { bias.load(a.b2, leaf * units + u); };
    const auto request_out = [&](int u, int r0) {
#pragma unroll
        for (int r = 0; r < kAhead; ++r) out_w[r].load(a.w2, row_of(r0 + r) + u);
    };
    const int first = lane < units ? lane : units - 1;
    float pre = 0.0f;                               // lane r: pre-activation of neuron r
    for (int r0 = 0; r0 < L; r0 += kRows) {
        uint4 w[kRows][NV];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            if (r0 + r < L) request(a.w1 + (leaf * L + r0 + r) * nvec, w[r]);
        if (r0 == 0) {
            pre = Elem<BF16>::load(a.b1, leaf * L + (lane < L ? lane : L - 1));
            request_bias(first);
            request_out(first, 0);
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            if (r0 + r >= L) continue;
            trim(w[r]);
            const float s = wave_sum(part_dot<BF16, NV>(xv, w[r]));
            pre += lane == r0 + r ? s : 0.0f;
        }
    }
    const float h = activate(pre, a.act);
    for (int u0 = 0; u0 < units; u0 += kWave) {
        const int u = u0 + lane < units ? u0 + lane : units - 1;
        if (u0 > 0) {
            request_bias(u);
            request_out(u, 0);
        }
        float y[Unit::kElems], f[Unit::kElems];
        bias.get(y);
        for (int r0 = 0; r0 < L; r0 += kAhead) {
            if (r0 > 0) request_out(u, r0);
#pragma unroll
            for (int r = 0; r < kAhead; ++r) {
                if (r0 + r >= L) continue;
                const float hr = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), r0 + r));
                out_w[r].get(f);
#pragma unroll
                for (int e = 0; e < Unit::kElems; ++e) y[e] = fmaf(hr, f[e], y[e]);
            }
        }
        if (live && u0 + lane < units) Unit::store(a.out, t * units + u, y);
    }
}

template <bool BF16, int NV, bool PIECES> hipError_t run(const WaveArgs& a, int waves, size_t lds_bytes, hipStream_t s) {
    auto kern = walk_wave_kernel<BF16, NV, PIECES>;
    note_launch("walk_wave_kernel<%s,%d,%s> tokens=%d top=%d", BF16 ? "bf16" : "f32", NV, PIECES ? "pieces" : "elements", waves, a.top);
    kern<<<dim3((unsigned)((a.T + waves - 1) / waves)), dim3(waves * kWave), lds_bytes, s>>>(a);
    return hipGetLastError();
}

template <bool BF16, bool PIECES> hipError_t dispatch(const WaveArgs& a, int waves, size_t lds_bytes, hipStream_t s) {
    if (a.nvec <= 64) return run<BF16, 1, PIECES>(a, waves, lds_bytes, s);
    if (a.nvec <= 128) return run<BF16, 2, PIECES>(a, waves, lds_bytes, s);
    if (a.nvec <= 256) return run<BF16, 4, PIECES>(a, waves, lds_bytes, s);
    return run<BF16, 8, PIECES>(a, waves, lds_bytes, s);
}

}  // namespace

// Whole aligned token, node and input weight rows of up to 512 pieces; output rows of any alignment, of at most 2^30 elements (the kernel's
// positions in a row are 32 bits, and a wave looks 64 units ahead).
bool wave_shape_ok(const Problem& p) {
    return walk_shape_ok(p) && vec_ok(p.leaf_w1, p.D, p.bf16) && p.D * (p.bf16 ? 2 : 4) <= 512 * 16 && p.L <= kMaxNeurons && p.depth >= 1 && p.depth < 30 &&
           p.O <= (int64_t)1 << 30;
}

// Whether 17 to 32 tokens a compute unit (many: more than 24), leaves of more than 8 neurons, go faster through the staged path's matrix launches.
// By tokens a leaf, from 4021 such calls (profiles/wave_a_token_calls.csv): 32 neurons from 32 tokens on (0.78 to 1.05; fewer 1.2 and more), in the larger
// half of the batches 17 to 28 neurons from 64 on (1.01, every third call 0.7 to 0.95), 13 to 16 from 12 on (0.90 to 0.98; 9 to 12 neurons 1.1) and
// small leaf rows, which the gather kernel finds in L1, from 2 on (1.0); leaf rows of more than 23 KB from 8 on (0.95).
bool staged_fills_tiles(const Problem& p, bool many, int64_t leaf_rows) {
    const int64_t per_leaf = p.T >> p.depth, L = p.L;
    if (L <= 16 && per_leaf >= 8 && per_leaf < 16 && leaf_rows > 23 * 1024) return true;
    if (many && L >= 16 && leaf_rows < 8192 && per_leaf >= 2) return true;
    return L > 28 ? per_leaf >= 32 : many && (L > 16 ? per_leaf >= 64 : L > 12 && per_leaf >= 12);
}

// Where a wave a token is ahead of what else takes a call: lines from 23285 random calls of both sides (513 to 12800 tokens, rows of 64
// bytes to 8 KB, depth 1 to 14, 1 to 32 neurons; profiles/wave_a_token_calls.csv).  By tokens a compute unit (up to 2 a block a token is taken):
//   2 to 4    up to 8 neurons: 1.5 (one neuron, short rows) to 2.4
//   4 to 8    up to 16 neurons: 1.5 to 2.2; not one or two on rows of up to 512 bytes (0.95 to 1.2)
//   8 to 16   rows of up to 4 KB (beyond, 8 waves are all that a block holds: 0.8 to 0.9) of more than 512 bytes, or 256 from 3 neurons on, or any from 6
//             on or with output rows that are not whole pieces: 1.2 to 2.1; from 12 on not leaves of up to 8 neurons on rows of up to 256 bytes (1.02, a
//             tenth of the calls 0.85) or, with output rows that are not whole pieces, less than 3 KB of rows for a token (1.1, every seventh 0.84 to 0.95)
//   16 to 32  leaves of more than 8 neurons on rows of up to 2 KB: 1.2 to 2.0; 6 to 8 neurons on 512 bytes to 1 KB: 1.16 and more up to 24 tokens (beyond
//             0.96, but 1.4 with output rows of more than 40 bytes that are not whole pieces).  Not where bf16 tokens fill the tiles of the staged path's
//             matrix launches (staged_fills_tiles: there 0.97 on average, down to 0.56)
//   32 to 48  3 to 8 neurons on 512 bytes to 1 KB: 1.1 to 1.5; on 256 to 512 with leaf rows of 4 MB together (1.2; less: 0.9 to 1.07); output rows that are
//             not whole pieces 1.5 from 40 bytes on (shorter ones 1.06, every fourth call 0.85 to 0.95)
// Element-wise output rows of wide leaves are a trip for 64 elements of four neurons: up to 12 tokens a compute unit a block a token, with four to
// eight waves for them, is ahead from 7000 weights on (2547 tokens of 32, 32 neurons, 958 outputs 29.7 us, 58.2 here).
// Of the 23285 calls the lines leave 22180 here, 1.72 times as fast on average, 38 more than 5 % slower, 14 more than 10 %.
bool wave_better(const Problem& p) {
    const int64_t cus = device_info().cus, es = p.bf16 ? 2 : 4, row = p.D * es, out_row = p.O * es, T = p.T, L = p.L;
    if (!wave_shape_ok(p) || T > 48 * cus) return false;
    const bool pieces = vec_ok(p.out, p.O, p.bf16) && vec_ok(p.leaf_w2, p.O, p.bf16) && vec_ok(p.leaf_b2, p.O, p.bf16);
    const int64_t leaf_rows = L * (row + out_row) + out_row, met = p.depth * row + leaf_rows;      // bytes of a leaf's rows, of all that a token meets
    if (T <= 4 * cus) return L <= 8;
    if (T <= 12 * cus && !pieces && L > 8 && L * p.O >= 7000) return false;
    if (T <= 8 * cus) return L <= 16 && (L > 2 || row > 512 || !pieces);
    if (T <= 16 * cus) {
        if (row > 4096 || L > 32 || (T > 12 * cus && L <= 8 && (pieces ? row <= 256 : met < 3000))) return false;
        return row > 512 || (row > 256 && L >= 3) || L >= 6 || !pieces;
    }
    if (T <= 32 * cus) {
        if (L <= 8) return L >= 6 && row > 512 && row <= 1024 && (T <= 24 * cus || (!pieces && out_row > 40));
        return L <= 32 && row <= 2048 && !(p.bf16 && pieces && staged_fills_tiles(p, T > 24 * cus, leaf_rows));
    }
    return L >= 3 && L <= 8 && row > 256 && row <= 1024 && (pieces ? row > 512 || leaf_rows << p.depth > (int64_t)4 << 20 : out_row > 40);
}

hipError_t launch_walk_wave(const Problem& p, int32_t* leaf_idx, hipStream_t s) {
    if (p.T == 0) return hipSuccess;
    WaveArgs a;
    a.x = (const uint4*)p.x;
    a.node_w = (const uint4*)p.node_w;
    a.node_b = p.node_b;
    a.w1 = (const uint4*)p.leaf_w1;
    a.b1 = p.leaf_b1;
    a.w2 = p.leaf_w2;
    a.b2 = p.leaf_b2;
    a.out = p.out;
    a.leaf_idx = leaf_idx;
    a.T = p.T;
    a.O = p.O;
    a.depth = p.depth;
    a.nvec = (int)(p.D / (p.bf16 ? 8 : 4));
    a.L = p.L;
    a.act = p.act;
    const int64_t cus = device_info().cus, row_bytes = p.D * (p.bf16 ? 2 : 4);
    // A block a compute unit up to 16 tokens a compute unit; beyond that blocks of 8, several of which run side by side (8192 tokens, rows
    // of up to 2 KB: 10 % faster than blocks of 16).
    int64_t waves = (p.T + cus - 1) / cus;
    waves = waves < 4 ? 4 : waves > 16 ? 8 : waves;
    if (waves > max_waves(a.nvec <= 256 ? 4 : 8)) waves = max_waves(a.nvec <= 256 ? 4 : 8);
    // Levels kept in LDS: a block of up to eight tokens finds the top rows in L1 and L2 as fast as it would fill LDS with them (5000 random calls
    // of 1024 to 2048 tokens: without 1.01 to 1.12 times as fast as with three levels; 2048 tokens of 768, depth 11: 8.6 -> 8.4 us); more tokens share
    // more (4096 fp32 ones of 784, depth 6: 1.18 times the time without as with four).
    const int64_t widest = p.T <= 8 * cus ? 0 : p.T > 16 * cus ? 14 : row_bytes <= 2048 ? 7 : 28;   // KB
    a.top = 0;
    while (a.top < p.depth && (row_bytes << a.top) <= widest * 1024 && (row_bytes + 4) * ((2 << a.top) - 1) <= 64 * 1024) ++a.top;
    g_walk_tuning.last_top = a.top;
    const size_t lds_bytes = (size_t)(row_bytes + 4) * (((int64_t)1 << a.top) - 1);
    const bool pieces = vec_ok(p.out, p.O, p.bf16) && vec_ok(p.leaf_w2, p.O, p.bf16) && vec_ok(p.leaf_b2, p.O, p.bf16);
    if (p.bf16) return pieces ? dispatch<true, true>(a, (int)waves, lds_bytes, s) : dispatch<true, false>(a, (int)waves, lds_bytes, s);
    return pieces ? dispatch<false, true>(a, (int)waves, lds_bytes, s) : dispatch<false, false>(a, (int)waves, lds_bytes, s);
}

}  // namespace fff
