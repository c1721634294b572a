// Small-batch launch: one block per token -- hard-routed FFF inference (Algorithm 1, Forward_I), the experts of a
// mixture, and the transformer block with wide nodes between layer norm and residual sum.
//
// With a few hundred tokens the call is a chain of dependent steps: a node's row cannot be requested before the
// decision above it is known, so the time is the number of memory round trips plus the instructions between
// them.  This kernel shortens both instead of streaming.
//   - The eight waves form row slots of H waves; a slot holds the token row in registers, a 16-byte piece a
//     lane (H = 1, 2, 4 or 8 by the row's length).
//   - A round trip takes S levels: the rows of the whole S-level subtree below the current node (2^S - 1 nodes,
//     contiguous level by level in heap order) are dealt to the slots, eight rows a wave, the sums meet in LDS
//     (one barrier, two buffers), and every wave takes the S decisions for itself from a ballot.  S is as large as the
//     block can request at once (64 KB), and the levels are spread evenly over the round trips.
//   - Leaf: the hidden neurons are dealt to the slots in the same way (the same code runs); the output weights, of
//     which every thread owns one piece of every G-th neuron, and the output biases are requested before the
//     hidden activations are known.
// (figures: at launch_token_block)
#include <type_traits>

#include "fff_device.h"
#include "fff_internal.h"

namespace fff {
namespace {

constexpr int kTokenBlock = 512;
constexpr int kTokenWaves = kTokenBlock / kWave;
constexpr int kTokenPieces = 8;         // 16-byte pieces of weight rows a lane has in flight
constexpr int kMaxLevels = 6;           // of a round trip: its decisions come out of one ballot
constexpr int kOutGroups = 4;           // partial output rows that meet in LDS, at most
constexpr int kTokenMaxPieces = 1024;
constexpr int64_t kTokenMaxBlocks = 1 << 22;    // of a launch, which ends at 2^32 threads

struct TokenArgs {
    const char* x;
    const char* node_w;      // [nodes, n, D]
    const void* node_b;      // [nodes, n] biases of the nodes' hidden neurons (without wide nodes: of the nodes)
    const char* w1;
    const void* b1;
    const char* w2;
    const char* b2;
    char* out;
    int32_t* leaf_idx;
    int xbytes, obytes, opieces;
    int depth, levels;           // levels per round trip
    int L, act, slots;           // slots: sums of a round trip kept in LDS
    int group_shift, groups;     // output rows: the 2^group_shift threads of a group own one piece each, groups take turns over the neurons
    int O, out_vec;
    const int32_t* given_leaf;   // kFromList: the leaf of every token
    GateCandidates gate;         // kFromGate
    WideNodes wide;              // block kernels only
    uint32_t per_n;              // 65536 / n + 1: divides the row numbers of a round trip
    int D;
    int64_t T;
};

// where the leaf comes from: the tree, the gating candidates of a mixture of experts, or a list
enum { kFromTree = 0, kFromGate = 1, kFromList = 2 };

// One element, widened only where it is used: the conversion would wait for the load, and with it for all loads before it.
template <bool BF16> __device__ __forceinline__ uint32_t load_raw(const void* p, int64_t i) {
    return BF16 ? ((const uint16_t*)p)[i] : ((const uint32_t*)p)[i];
}
template <bool BF16> __device__ __forceinline__ float raw_value(uint32_t v) { return __uint_as_float(BF16 ? v << 16 : v); }

// Sums of eight values over the wave, in 24 instructions instead of 96: halves of the wave, then quarters, are exchanged
// between two values at a time, so that 16-lane row r of out[j] ends up with the sum of value 4 j + r / 2 + 2 (r % 2).
__device__ __forceinline__ void wave_sums_of_8(const float (&v)[8], float (&out)[2]) {
    float h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {       // lower half of the wave: value 2 i, upper half: value 2 i + 1
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * i]), __float_as_uint(v[2 * i + 1]), false, false);
        h[i] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(h[2 * j]), __float_as_uint(h[2 * j + 1]), false, false);
        out[j] = group_sum<16>(__uint_as_float(x[0]) + __uint_as_float(x[1]));
    }
}

// SPLIT: log2 H; NV: pieces of a row per lane; BLOCK: wide nodes on the normalised token, which is kept in fp32;
// ODD: rows that are not whole pieces.
//
// No load is predicated by lane (that compiles to guarded loads and a wait each): lanes past the end of a row read
// its last window; whole waves skip the rows that are not there.  What such lanes and windows repeat must not count even where it
// is infinite (0 * inf is NaN): of whole pieces a lane past the row drops its sum, of odd rows the weights are cleared like the
// token.  (The clearing behind a branch cost every launch a wait: 64 tokens of 768 features, depth 11 5.7 -> 6.3 us.)
// With two waves a SIMD every instruction of a wave costs 4 to 8 cycles, as much in all as the memory round trips: row addresses are made
// by the lanes at once (lane q: row q), sums reduced eight at a time, the cases told apart by templates.
template <bool BF16, int SPLIT, int NV, int SRC, bool BLOCK, bool ODD>
__global__ __launch_bounds__(kTokenBlock, 4) void token_block_kernel(const TokenArgs a) {
    constexpr int E = Elem<BF16>::kPerVec;
    constexpr int H = 1 << SPLIT, kSlots = kTokenWaves >> SPLIT;
    constexpr int kRows = kTokenPieces / NV;    // rows a wave has in flight
    constexpr int kOutAhead = BLOCK ? 4 : 8;    // output-weight pieces a thread requests ahead
    // LDS: two buffers of a round trip's sums (also the layer norm's partial sums), [L] hidden activations,
    // [groups][opieces * E] partial output rows
    extern __shared__ float lds_all[];
    float* const hidden = lds_all + 2 * a.slots;
    float* const rows_lds = hidden + (a.L + 3) / 4 * 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int part = wv % H, slot = wv / H;
    const int nn = BLOCK ? a.wide.n : 1;
    const int c0 = part * (NV * kWave) + lane;      // this lane's first piece of an input row
    const int64_t t = blockIdx.x;
    int off[NV];
    bool past[NV];      // the piece lies past the row's end
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        off[v] = piece_offset(c0 + v * kWave, a.xbytes);
        past[v] = 16 * (c0 + v * kWave) >= a.xbytes;
    }
    // what a piece of a row holds that the pieces before it do not
    uint4 held[ODD ? NV : 1];
    if constexpr (ODD) {
#pragma unroll
        for (int v = 0; v < NV; ++v) held[v] = drop_first<BF16>(make_uint4(~0u, ~0u, ~0u, ~0u), c0 + v * kWave, a.xbytes);
    }

    // the token row as loaded, and in fp32 where it is normalised
    uint4 xv[NV], w[kRows][NV];
    float z[BLOCK ? NV : 1][E];
#pragma unroll
    for (int v = 0; v < NV; ++v) xv[v] = load_any(a.x + t * a.xbytes + off[v]);

    // Requests the rows q0, q0 + kSlots, ... below `rows` (at most 64) of `weights`; lane q holds where row q starts.
    const auto fetch = [&](const char* weights, uint64_t start, int rows, int q0) {
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int q = q0 + i * kSlots;
            if (q >= rows) continue;
            const char* const row = weights + ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(start >> 32), q) << 32 |
                                               (uint32_t)__builtin_amdgcn_readlane((int)start, q));
#pragma unroll
            for (int v = 0; v < NV; ++v) w[i][v] = load_any(row + off[v]);
        }
    };
    // ... and their dot products with the token go to `sums` (a row's H parts side by side)
    const auto reduce = [&](float* sums, int rows, int q0) {
        float p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = 0.0f;
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            if (q0 + i * kSlots >= rows) continue;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                float d = 0.0f;
                if constexpr (ODD)
                    w[i][v] = make_uint4(w[i][v].x & held[v].x, w[i][v].y & held[v].y, w[i][v].z & held[v].z, w[i][v].w & held[v].w);
                if constexpr (BLOCK) {
                    float f[E], d1 = 0.0f;
                    widen<BF16>(w[i][v], f);
#pragma unroll
                    for (int e = 0; e < E; e += 2) {
                        d = fmaf(f[e], z[v][e], d);
                        d1 = fmaf(f[e + 1], z[v][e + 1], d1);
                    }
                    d += d1;
                } else {
                    d = Elem<BF16>::dot(xv[v], w[i][v], d);
                }
                d = !ODD && past[v] ? 0.0f : d;
                p[i] = v > 0 ? p[i] + d : d;
            }
        }
        float sum[2];
        wave_sums_of_8(p, sum);
#pragma unroll
        for (int j = 0; j < (kRows > 4 ? 2 : 1); ++j) {
            const int q = q0 + (4 * j + lane / 32 + 2 * (lane / 16 & 1)) * kSlots;      // the row of this 16-lane row's sum
            if ((lane & 15) == 0 && q < rows) sums[q * H + part] = sum[j];
        }
    };
    const auto parts_of = [&](const float* sums, int q) {     // the sum of row q over its slot's waves
        float s[H];
        if constexpr (H >= 4) {
#pragma unroll
            for (int h = 0; h < H; h += 4) *(float4*)(s + h) = *(const float4*)(sums + q * H + h);
        } else {
#pragma unroll
            for (int h = 0; h < H; ++h) s[h] = sums[q * H + h];
        }
#pragma unroll
        for (int d = H / 2; d > 0; d /= 2)
#pragma unroll
            for (int h = 0; h < d; ++h) s[h] += s[h + d];
        return s[0];
    };

    // ---- descent (Algorithm 1: logit >= 0 takes the right child)
    int n = 0, buf = 0;      // position within the current level; buffer of sums
    // of the round trip from level m on: its levels, rows, and this lane's row, its start, bias ...
    int m = 0, s = 0, nodes = 0, rows = 0;
    uint64_t start = 0;
    uint32_t bias = 0, scale = 0, out_bias = 0;
    const auto plan = [&]() {
        s = a.depth - m < a.levels ? a.depth - m : a.levels;
        nodes = (1 << s) - 1;
        rows = nodes * nn;
        const uint32_t root = (1u << m) - 1 + n;        // heap row of the subtree's root; node j at depth k of it: (root << k) + j
        const int mine = lane < rows ? lane : rows - 1, node = BLOCK ? (int)(mine * a.per_n >> 16) : mine;
        const uint32_t row = ((root << (31 - __clz(node + 1))) + node) * (uint32_t)nn + (BLOCK ? mine - node * nn : 0);
        start = (uint64_t)row * (uint32_t)a.xbytes;
        bias = load_raw<BF16>(a.node_b, row);
        if (BLOCK) {
            const int my = lane < nodes ? lane : nodes - 1;
            scale = load_raw<BF16>(a.wide.w2, row);
            out_bias = load_raw<BF16>(a.wide.b2, (root << (31 - __clz(my + 1))) + my);
        }
    };
    if (SRC == kFromTree && a.depth > 0) {
        plan();
        fetch(a.node_w, start, rows, slot);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) xv[v] = drop_first<BF16>(xv[v], c0 + v * kWave, a.xbytes);
    if constexpr (BLOCK) {
#pragma unroll
        for (int v = 0; v < NV; ++v) widen<BF16>(xv[v], z[v]);
        if (a.wide.gamma) {
            // mean, then the mean of squared deviations (divisor D), over the waves of the slot
            float* partial = lds_all;
            const auto slot_sum = [&](float v) {
                v = wave_sum(v);
                if (H == 1) return v;
                if (lane == 0) partial[wv] = v;
                __syncthreads();
                v = parts_of(partial, slot);
                partial += kTokenWaves;
                return v;
            };
            float g[NV][E], b[NV][E];
            int dropped[NV];        // elements that belong to the piece before
            float sum = 0.0f, sq = 0.0f;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                widen<BF16>(load_any((const char*)a.wide.gamma + off[v]), g[v]);
                widen<BF16>(load_any((const char*)a.wide.beta + off[v]), b[v]);
                dropped[v] = (16 * (c0 + v * kWave) - off[v]) * E / 16;
#pragma unroll
                for (int e = 0; e < E; ++e) sum += z[v][e];
            }
            const float mean = slot_sum(sum) / (float)a.D;
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    z[v][e] = e >= dropped[v] ? z[v][e] - mean : 0.0f;
                    sq = fmaf(z[v][e], z[v][e], sq);
                }
            const float rstd = 1.0f / sqrtf(slot_sum(sq) / (float)a.D + a.wide.eps);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int e = 0; e < E; ++e) z[v][e] = e >= dropped[v] ? fmaf(z[v][e] * rstd, g[v][e], b[v][e]) : 0.0f;
            if (H > 1) buf = 1;     // (buffer 0 holds the partial sums, which the slowest wave may still read)
        }
    }
    if constexpr (SRC == kFromTree) {
        while (m < a.depth) {
            float* const sums = lds_all + buf * a.slots;
            for (int q0 = slot; q0 < rows; q0 += kSlots * kRows) {
                if (m > 0 || q0 != slot) fetch(a.node_w, start, rows, q0);
                reduce(sums, rows, q0);
            }
            __syncthreads();
            float logit = parts_of(sums, lane < rows ? lane : rows - 1) + raw_value<BF16>(bias);
            if constexpr (BLOCK) {
                const float v = lane < rows ? raw_value<BF16>(scale) * activate(logit, a.act) : 0.0f;    // one hidden neuron a lane
                if (s == 1) {
                    logit = wave_sum(v) + raw_value<BF16>(out_bias);
                } else {
                    const int my = lane < nodes ? lane : nodes - 1;
                    logit = raw_value<BF16>(out_bias);
                    for (int j = 0; j < nn; ++j) logit += __shfl(v, my * nn + j, kWave);
                }
            }
            const uint64_t right = __ballot(logit >= 0.0f);
            int j = 0;
#pragma unroll
            for (int k = 0; k < kMaxLevels; ++k) j = k < s ? 2 * j + (int)(right >> ((1 << k) - 1 + j) & 1) : j;
            n = __builtin_amdgcn_readfirstlane((n << s) + j);
            m += s;
            buf ^= 1;
            if (m < a.depth) plan();
        }
    } else if constexpr (SRC == kFromGate) {
        n = __builtin_amdgcn_readfirstlane(best_candidate(a.gate.val + t * a.gate.n, a.gate.idx + t * a.gate.n, a.gate.n));
    } else {
        n = a.given_leaf[t];
    }

    // ---- leaf: hidden neurons, 64 at a time (lane q: neuron q); behind the first ones, what the output row needs
    const char* const w1 = a.w1 + (int64_t)n * a.L * a.xbytes;
    const char* const w2 = a.w2 + (int64_t)n * a.L * a.obytes;
    const int grp = wv >> (a.group_shift - 6), c = threadIdx.x - (grp << a.group_shift);     // (a group is whole waves)
    const int ooff = a.out_vec ? piece_offset(c < a.opieces ? c : a.opieces - 1, a.obytes) : 0;
    uint4 ahead[kOutAhead], b2, res;
    const bool few = a.L <= kWave;
    float h_lane = 0.0f;
    const auto hidden_neurons = [&](int base, auto with_output) {
        const int count = a.L - base < kWave ? a.L - base : kWave;
        float* const sums = lds_all + buf * a.slots;
        const uint64_t first = (uint64_t)(uint32_t)(base + (lane < count ? lane : count - 1)) * (uint32_t)a.xbytes;
        if (slot < count) fetch(w1, first, count, slot);
        const uint32_t b1 = load_raw<BF16>(a.b1, (int64_t)n * a.L + base + (lane < count ? lane : count - 1));
        if (with_output.value && a.out_vec) {
#pragma unroll
            for (int i = 0; i < kOutAhead; ++i) {
                const int r = grp + i * a.groups;
                if (r < a.L) ahead[i] = load_any(w2 + (int64_t)r * a.obytes + ooff);
            }
            b2 = load_any(a.b2 + (int64_t)n * a.obytes + ooff);
            if (BLOCK && a.wide.residual) res = load_any(a.x + t * a.xbytes + ooff);
        }
        for (int q0 = slot; q0 < count; q0 += kSlots * kRows) {
            if (q0 != slot) fetch(w1, first, count, q0);
            reduce(sums, count, q0);
        }
        __syncthreads();
        // up to 64 neurons every wave takes all the activations, a lane each, and picks the ones it needs from its lanes
        if (few || wv == 0) h_lane = activate(parts_of(sums, lane < count ? lane : count - 1) + raw_value<BF16>(b1), a.act);
        if (!few && wv == 0 && lane < count) hidden[base + lane] = h_lane;
        buf ^= 1;
    };
    // (the usual single chunk stands alone: in a loop its loads would wait for those of the turn before)
    hidden_neurons(0, std::true_type());
    for (int base = kWave; base < a.L; base += kWave) hidden_neurons(base, std::false_type());
    if (threadIdx.x == 0 && a.leaf_idx) a.leaf_idx[t] = n;
    if (!few) __syncthreads();
    const auto hidden_of = [&](int r) {
        return few ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h_lane), r)) : hidden[r];
    };

    // ---- output row: the thread's piece of every groups-th neuron, then the groups' sums
    if (a.out_vec) {
        float y[E], f[E];
        const auto add = [&](const uint4& v, float h) {
            widen<BF16>(v, f);
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = fmaf(h, f[e], y[e]);
        };
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = 0.0f;
#pragma unroll
        for (int i = 0; i < kOutAhead; ++i)
            if (grp + i * a.groups < a.L) add(ahead[i], hidden_of(grp + i * a.groups));
        for (int r = grp + kOutAhead * a.groups; r < a.L; r += a.groups) add(load_any(w2 + (int64_t)r * a.obytes + ooff), hidden_of(r));
        if (a.groups > 1) {
            if (grp < a.groups && c < a.opieces) {
                float4* dst = (float4*)(rows_lds + (grp * a.opieces + c) * E);
                dst[0] = make_float4(y[0], y[1], y[2], y[3]);
                if (E == 8) dst[1] = make_float4(y[4 % E], y[5 % E], y[6 % E], y[7 % E]);
            }
            __syncthreads();
            if (grp == 0 && c < a.opieces) {
#pragma unroll
                for (int g = 1; g < kOutGroups; ++g) {
                    if (g >= a.groups) continue;
                    const float* src = rows_lds + (g * a.opieces + c) * E;
#pragma unroll
                    for (int e = 0; e < E; ++e) y[e] += src[e];
                }
            }
        }
        // In place (out = x) a row's last window, which may overlap the piece before, is read before anything is stored.
        // Rows longer than the block have their second pieces still to read: at most one a thread, as rows of x end at 1024 pieces.
        uint4 res_far;
        const bool far = BLOCK && a.wide.residual && a.opieces > kTokenBlock;
        if (far) {
            const int cf = threadIdx.x + kTokenBlock;
            res_far = load_any(a.x + t * a.xbytes + piece_offset(cf < a.opieces ? cf : a.opieces - 1, a.obytes));
            __syncthreads();
        }
        if (grp == 0 && c < a.opieces) {
            add(b2, 1.0f);
            if (BLOCK && a.wide.residual) add(res, 1.0f);
            store_any(a.out + t * a.obytes + ooff, narrow<BF16>(y));
        }
        // rows longer than the block
        for (int cc = c + kTokenBlock; cc < a.opieces; cc += kTokenBlock) {
            const int at = piece_offset(cc, a.obytes);
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = 0.0f;
            for (int r = 0; r < a.L; ++r) add(load_any(w2 + (int64_t)r * a.obytes + at), hidden_of(r));
            add(load_any(a.b2 + (int64_t)n * a.obytes + at), 1.0f);
            if (far) add(res_far, 1.0f);
            store_any(a.out + t * a.obytes + at, narrow<BF16>(y));
        }
    } else {        // rows shorter than a piece
        for (int o = threadIdx.x; o < a.O; o += kTokenBlock) {
            float y = Elem<BF16>::load(a.b2, (int64_t)n * a.O + o);
            for (int r = 0; r < a.L; ++r) y = fmaf(hidden_of(r), Elem<BF16>::load(a.w2, ((int64_t)n * a.L + r) * a.O + o), y);
            if (BLOCK && a.wide.residual) y += Elem<BF16>::load(a.x, t * a.D + o);
            Elem<BF16>::store(a.out, t * a.O + o, y);
        }
    }
}

template <bool BF16, int SPLIT, int NV, int SRC, bool BLOCK, bool ODD>
hipError_t run_token(TokenArgs a, hipStream_t s) {
    constexpr int E = Elem<BF16>::kPerVec;
    constexpr int H = 1 << SPLIT;
    // Levels per round trip, from an estimate fitted to kernel clocks: a trip costs about 1800 cycles, and every row of its subtree 30 per
    // wave of a slot, a third more once every compute unit has a block (2 tokens
    // of 64 features, depth 11: trips of 6 levels 5.0 us a call, of 4 5.2, of 3 5.9, of 2 7.0; 196 of 664, depth 12: of 4 7.4, of 3 7.6, of 5 8.0, of 2 8.8).
    const int n = BLOCK ? a.wide.n : 1, room = (kTokenWaves >> SPLIT) * kTokenPieces / NV;
    const double row_cost = (30 + 10 * (a.T < 256 ? (double)a.T / 256 : 1)) * (H * NV) * n;
    double best = 0;
    for (int levels = 1; levels <= kMaxLevels && (levels == 1 || ((1 << levels) - 1) * n <= room); ++levels) {
        double cost = 0;
        for (int m = 0; m < a.depth; m += levels) cost += 1800 + row_cost * ((1 << (a.depth - m < levels ? a.depth - m : levels)) - 1);
        if (levels == 1 || cost < best) {
            best = cost;
            a.levels = levels;
        }
    }
    a.per_n = 65536 / n + 1;
    a.slots = kWave << SPLIT;       // sums of a round trip: at most 64 rows, times the waves of a slot
    a.group_shift = 6;
    while (a.group_shift < 9 && (1 << a.group_shift) < a.opieces) ++a.group_shift;
    a.groups = kTokenBlock >> a.group_shift;
    if (a.groups > kOutGroups) a.groups = kOutGroups;
    if (a.groups > (a.L + 1) / 2) a.groups = (a.L + 1) / 2;
    const size_t lds_bytes = sizeof(float) * (2 * (size_t)a.slots + (a.L + 3) / 4 * 4 +
                                              (a.out_vec && a.groups > 1 ? (size_t)a.groups * a.opieces * E : 0));
    note_launch("token_block_kernel<%s,%d,%d,%s> levels=%d %s", BF16 ? "bf16" : "f32", H, NV,
                BLOCK ? "block" : SRC == kFromTree ? "hard" : SRC == kFromGate ? "gate" : "list", a.levels, a.out_vec ? "vec" : "elem");
    token_block_kernel<BF16, SPLIT, NV, SRC, BLOCK, ODD><<<dim3((unsigned)a.T), dim3(kTokenBlock), lds_bytes, s>>>(a);
    return hipGetLastError();
}

template <bool BF16, int SRC, bool BLOCK, bool ODD>
hipError_t pick_rows(const TokenArgs& a, int pieces, hipStream_t s) {
    if (pieces <= 64) return run_token<BF16, 0, 1, SRC, BLOCK, ODD>(a, s);
    if (pieces <= 128) return run_token<BF16, 1, 1, SRC, BLOCK, ODD>(a, s);
    if (pieces <= 256) return run_token<BF16, 2, 1, SRC, BLOCK, ODD>(a, s);
    if (pieces <= 512) return run_token<BF16, 3, 1, SRC, BLOCK, ODD>(a, s);
    return run_token<BF16, 3, 2, SRC, BLOCK, ODD>(a, s);
}
template <bool BF16, int SRC, bool BLOCK>
hipError_t dispatch_token(const TokenArgs& a, int pieces, hipStream_t s) {
    if (SRC != kFromGate && (a.xbytes & 15)) return pick_rows<BF16, SRC, BLOCK, SRC != kFromGate>(a, pieces, s);   // (the gating takes whole pieces)
    return pick_rows<BF16, SRC, BLOCK, false>(a, pieces, s);
}

template <bool BF16> hipError_t pick_token(const TokenArgs& a, int pieces, bool wide, hipStream_t s) {
    if (wide) return dispatch_token<BF16, kFromTree, true>(a, pieces, s);
    if (a.gate.n > 0) return dispatch_token<BF16, kFromGate, false>(a, pieces, s);
    if (a.given_leaf) return dispatch_token<BF16, kFromList, false>(a, pieces, s);
    return dispatch_token<BF16, kFromTree, false>(a, pieces, s);
}

}  // namespace

// Rows of at least one piece and at most 1024 of them, at any alignment; leaves of up to 4096 neurons
bool token_shape_ok(const Problem& p) {
    const int64_t per = p.bf16 ? 8 : 4;
    return p.D >= per && (p.D + per - 1) / per <= kTokenMaxPieces && p.O <= (1 << 24) && p.L <= 4096;
}

// ... and nodes of at most 64 hidden neurons (a lane each)
bool token_wide_ok(const Problem& p, int node_size) { return token_shape_ok(p) && node_size <= kWave; }

// Measured against the kernel before it (wave 0 alone walked three levels a trip, a wave held whole rows), per call back to back:
// 9 tokens of 2256 fp32 features, depth 14 23.3 -> 11.4 us (no kernel of this kind took the row), 174 of 2768 79 -> 14; 1003 of 1416 bf16 features,
// 16 neurons 40.5 -> 26.7; 2 of 64, depth 11 7.0 -> 4.7; 196 of 664, depth 12 8.0 -> 7.7; odd rows, which the element-wise kernels took:
// 3 of 671 fp32 features, 32 neurons 64 -> 7.6, 1361 of 974 74 -> 25; wide nodes: 113 tokens of 712, four neurons a node 22 -> 8.
// What bounds it: the round trips (1800 cycles each).  Where the leaf outweighs the tree, or the batch wants more than two blocks a
// compute unit, token_rows_kernel is ahead (token_rows_better).
hipError_t launch_token_block(const Problem& p, int32_t* leaf_idx, hipStream_t s, const int32_t* given_leaf,
                              const GateCandidates* gate, const WideNodes* wide) {
    const int per = p.bf16 ? 8 : 4, es = p.bf16 ? 2 : 4;
    TokenArgs a;
    a.node_w = (const char*)(wide ? wide->w1 : p.node_w);
    a.node_b = wide ? wide->b1 : p.node_b;
    a.w1 = (const char*)p.leaf_w1;
    a.b1 = p.leaf_b1;
    a.w2 = (const char*)p.leaf_w2;
    a.b2 = (const char*)p.leaf_b2;
    a.wide = wide ? *wide : WideNodes{};
    a.D = (int)p.D;
    a.O = (int)p.O;
    a.depth = p.depth;
    a.xbytes = (int)p.D * es;
    a.obytes = (int)p.O * es;
    a.opieces = (int)((p.O + per - 1) / per);
    a.L = p.L;
    a.act = p.act;
    a.out_vec = p.O >= per;
    const int pieces = (int)((p.D + per - 1) / per);
    hipError_t e = hipSuccess;
    for (int64_t t = 0; t < p.T && e == hipSuccess; t += kTokenMaxBlocks) {
        a.x = (const char*)p.x + t * a.xbytes;
        a.out = (char*)p.out + t * a.obytes;
        a.leaf_idx = leaf_idx ? leaf_idx + t : nullptr;
        a.given_leaf = given_leaf ? given_leaf + t : nullptr;
        a.gate = gate ? GateCandidates{gate->val + t * gate->n, gate->idx + t * gate->n, gate->n} : GateCandidates{};
        a.T = p.T - t < kTokenMaxBlocks ? p.T - t : kTokenMaxBlocks;
        e = p.bf16 ? pick_token<true>(a, pieces, wide != nullptr, s) : pick_token<false>(a, pieces, wide != nullptr, s);
    }
    return e;
}

}  // namespace fff
