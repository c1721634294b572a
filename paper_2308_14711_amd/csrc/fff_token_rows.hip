// Hard-routed FFF inference (Algorithm 1, Forward_I), one block per token, for leaves of many neurons and for batches of short
// rows: a wave holds whole rows.
//
// Where a leaf is hundreds of rows, the call is the stream of those rows through one block, not the chain of decisions.  Wave 0
// walks the tree S levels a round trip (the whole S-level subtree below the current node requested at once); the leaf it
// reaches goes through LDS to the other waves, which deal the hidden neurons among themselves and request a
// neuron's input and output weights together, so that a neuron costs no barrier and no trip of its own; the waves' partial
// output rows meet in LDS once.  Every wave keeps its own token row, which ends at 512 pieces.
// (which of this kernel and token_block_kernel runs, and what both measured: token_rows_better)
#include "fff_device.h"
#include "fff_internal.h"

namespace fff {
int64_t g_token_kernel = 0;
namespace {

constexpr int kTokenBlock = 512;
constexpr int kTokenWaves = kTokenBlock / kWave;
constexpr size_t kRowsMaxLds = 144 * 1024;
constexpr int64_t kRowsMaxBlocks = 8192;      // blocks stride over larger batches

struct TokenRowsArgs {
    const uint4* x;
    const uint4* node_w;
    const void* node_b;
    const uint4* w1;
    const void* b1;
    const void* w2;
    const void* b2;
    void* out;
    int32_t* leaf_idx;
    const int32_t* given_leaf;   // non-null: the leaf of every token is given, nothing is descended
    int64_t T, O;
    int depth, nvec, ovec, L, act;
};

// Sum over the wave as a wave-uniform value: DPP rotations inside each 16-lane row, then the four row sums are read
// out as scalars.
__device__ __forceinline__ float uniform_sum(float v) {
    v = group_sum<16>(v);
    const int b = __float_as_int(v);
    const float s0 = __int_as_float(__builtin_amdgcn_readlane(b, 0));
    const float s1 = __int_as_float(__builtin_amdgcn_readlane(b, 16));
    const float s2 = __int_as_float(__builtin_amdgcn_readlane(b, 32));
    const float s3 = __int_as_float(__builtin_amdgcn_readlane(b, 48));
    return (s0 + s1) + (s2 + s3);
}

// NV: 16-byte vectors of a row per lane (rows of up to 64 * NV vectors); S: tree levels per round trip; OUTVEC: output rows are
// whole aligned vectors (else element-wise output, its hidden activations in LDS).
//
// Every load is unconditional (a predicated 16-byte load compiles to four guarded dword loads
// and a wait each): lanes past the end of a row re-read its last vector, subtree rows past the last level and neurons
// past the leaf width re-read a valid row, and their results are dropped (not multiplied by zero: the weights may be infinite).
template <bool BF16, int NV, int S, bool OUTVEC>
__global__ __launch_bounds__(kTokenBlock) void token_rows_kernel(TokenRowsArgs a) {
    constexpr int kPer = Elem<BF16>::kPerVec;
    constexpr int kSub = (1 << S) - 1;
    constexpr int kBatch = NV >= 8 ? 2 : 4;   // leaf neurons in flight per wave
    // LDS: the leaf found by wave 0 (one 16-byte slot), then OUTVEC: [waves][O] partial output rows; else [L] hidden activations
    extern __shared__ float lds_all[];
    int* const lds_leaf = (int*)lds_all;
    float* const lds = lds_all + 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int col[NV], ocol[NV];   // this lane's vectors of an input row / an output row, clamped
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int c = v * kWave + lane;
        col[v] = c < a.nvec ? c : a.nvec - 1;
        ocol[v] = OUTVEC ? (c < a.ovec ? c : a.ovec - 1) : 0;
    }
    const int64_t last_node = (((int64_t)1 << a.depth) - 1) - 1;

    for (int64_t t = blockIdx.x; t < a.T; t += gridDim.x) {
        uint4 xv[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) xv[v] = a.x[t * a.nvec + col[v]];
        const auto dot_row = [&](const uint4 (&w)[NV]) {
            float p = 0.0f;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const float q = Elem<BF16>::dot(xv[v], w[v], p);
                p = v * kWave + lane < a.nvec ? q : p;
            }
            return uniform_sum(p);
        };

        // ---- descent by wave 0: S levels per round trip (Algorithm 1: logit >= 0 takes the right child)
        int64_t n = 0;   // position within the current level
        for (int m = 0; wv == 0 && !a.given_leaf && m < a.depth; m += S) {
            const int s = a.depth - m < S ? a.depth - m : S;
            const int64_t root = (((int64_t)1 << m) - 1 + n) + 1;   // heap row of the subtree's root, plus one
            uint4 rows[kSub][NV];
            float bias[kSub], acc[kSub];
#pragma unroll
            for (int k = 0; k < S; ++k) {
#pragma unroll
                for (int j = 0; j < (1 << k); ++j) {
                    int64_t row = (root << k) - 1 + j;   // level k below the root, j-th node
                    row = row < last_node ? row : last_node;
                    const int q = (1 << k) - 1 + j;
#pragma unroll
                    for (int v = 0; v < NV; ++v) rows[q][v] = a.node_w[row * a.nvec + col[v]];
                    bias[q] = Elem<BF16>::load(a.node_b, row);
                }
            }
#pragma unroll
            for (int q = 0; q < kSub; ++q) acc[q] = dot_row(rows[q]) + bias[q];
            int j = 0;
#pragma unroll
            for (int k = 0; k < S; ++k) {
                // acc[2^k - 1 + j] as a chain of selects (registers cannot be indexed at run time)
                float logit = acc[(1 << k) - 1];
#pragma unroll
                for (int q = 1; q < (1 << k); ++q) logit = j == q ? acc[(1 << k) - 1 + q] : logit;
                j = k < s ? 2 * j + (logit >= 0.0f ? 1 : 0) : j;
            }
            n = (n << s) + j;
        }
        if (threadIdx.x == 0) {
            if (a.given_leaf) n = a.given_leaf[t];
            lds_leaf[0] = (int)n;
            if (a.leaf_idx) a.leaf_idx[t] = (int32_t)n;
        }
        __syncthreads();
        const int64_t leaf = lds_leaf[0];

        // ---- leaf: wave wv takes neurons wv, wv + waves, ...
        const int64_t nrow0 = leaf * a.L;
        float oacc[OUTVEC ? NV : 1][kPer];
#pragma unroll
        for (int v = 0; v < (OUTVEC ? NV : 1); ++v)
#pragma unroll
            for (int e = 0; e < kPer; ++e) oacc[v][e] = 0.0f;
        for (int r0 = wv; r0 < a.L; r0 += kTokenWaves * kBatch) {
            uint4 w1[kBatch][NV], w2[OUTVEC ? kBatch : 1][NV];
            float b1[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                int r = r0 + i * kTokenWaves;
                r = r < a.L ? r : a.L - 1;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    w1[i][v] = a.w1[(nrow0 + r) * a.nvec + col[v]];
                    if constexpr (OUTVEC) w2[i][v] = ((const uint4*)a.w2)[(nrow0 + r) * a.ovec + ocol[v]];
                }
                b1[i] = Elem<BF16>::load(a.b1, nrow0 + r);
            }
            float hidden[kBatch];       // (all of them before the first branch, so that their chains overlap)
#pragma unroll
            for (int i = 0; i < kBatch; ++i) hidden[i] = activate(dot_row(w1[i]) + b1[i], a.act);
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int r = r0 + i * kTokenWaves;
                if (r >= a.L) continue;
                if constexpr (OUTVEC) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        float w[kPer];
                        widen<BF16>(w2[i][v], w);
#pragma unroll
                        for (int e = 0; e < kPer; ++e) oacc[v][e] = fmaf(hidden[i], w[e], oacc[v][e]);
                    }
                } else if (lane == 0) {
                    lds[r] = hidden[i];
                }
            }
        }

        if constexpr (!OUTVEC) {
            __syncthreads();
            for (int64_t o = threadIdx.x; o < a.O; o += kTokenBlock) {
                float y = Elem<BF16>::load(a.b2, leaf * a.O + o);
                for (int r = 0; r < a.L; ++r) y = fmaf(lds[r], Elem<BF16>::load(a.w2, (nrow0 + r) * a.O + o), y);
                Elem<BF16>::store(a.out, t * a.O + o, y);
            }
            __syncthreads();
            continue;
        }
        // partial rows of the waves meet in LDS; then one thread per output vector
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int c = v * kWave + lane;
            if (c < a.ovec) {
                float* dst = lds + (int64_t)wv * a.O + (int64_t)c * kPer;
#pragma unroll
                for (int e = 0; e < kPer; e += 4)
                    *(float4*)(dst + e) = make_float4(oacc[v][e], oacc[v][e + 1], oacc[v][e + 2], oacc[v][e + 3]);
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < a.ovec; c += kTokenBlock) {
            float y[kPer];
            widen<BF16>(((const uint4*)a.b2)[leaf * a.ovec + c], y);
#pragma unroll
            for (int w = 0; w < kTokenWaves; ++w) {
                const float4* src = (const float4*)(lds + (int64_t)w * a.O + (int64_t)c * kPer);
#pragma unroll
                for (int e = 0; e < kPer; e += 4) {
                    const float4 f = src[e / 4];
                    y[e] += f.x;
                    y[e + 1] += f.y;
                    y[e + 2] += f.z;
                    y[e + 3] += f.w;
                }
            }
            ((uint4*)a.out)[t * a.ovec + c] = narrow<BF16>(y);
        }
        __syncthreads();   // LDS is reused by the block's next token
    }
}

// Whole aligned output rows of at most 512 pieces, whose partial sums fit LDS
bool rows_out_vec(const Problem& p) {
    const int64_t per = p.bf16 ? 8 : 4;
    return vec_ok(p.out, p.O, p.bf16) && vec_ok(p.leaf_w2, p.O, p.bf16) && vec_ok(p.leaf_b2, p.O, p.bf16) && p.O / per <= 8 * kWave &&
           16 + (size_t)kTokenWaves * p.O * sizeof(float) <= kRowsMaxLds;
}

template <bool BF16, int NV, int S, bool OUTVEC>
hipError_t run_rows(const Problem& p, int32_t* leaf_idx, const int32_t* given_leaf, hipStream_t s) {
    constexpr int kPer = Elem<BF16>::kPerVec;
    TokenRowsArgs a;
    a.x = (const uint4*)p.x;
    a.node_w = (const uint4*)p.node_w;
    a.node_b = p.node_b;
    a.w1 = (const uint4*)p.leaf_w1;
    a.b1 = p.leaf_b1;
    a.w2 = p.leaf_w2;
    a.b2 = p.leaf_b2;
    a.out = p.out;
    a.leaf_idx = leaf_idx;
    a.given_leaf = given_leaf;
    a.T = p.T;
    a.O = p.O;
    a.depth = p.depth;
    a.nvec = (int)(p.D / kPer);
    a.ovec = OUTVEC ? (int)(p.O / kPer) : 0;
    a.L = p.L;
    a.act = p.act;
    const size_t lds_bytes = 16 + sizeof(float) * (OUTVEC ? (size_t)kTokenWaves * p.O : (size_t)p.L);
    auto kern = token_rows_kernel<BF16, NV, S, OUTVEC>;
    static bool raised[64];
    if (lds_bytes > 48 * 1024) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        if (!raised[dev]) {
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kRowsMaxLds);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    const int64_t blocks = p.T < kRowsMaxBlocks ? p.T : kRowsMaxBlocks;
    note_launch("token_rows_kernel<%s,%d,%d,%s>", BF16 ? "bf16" : "f32", NV, S, OUTVEC ? "vec" : "elem");
    kern<<<dim3((unsigned)blocks), dim3(kTokenBlock), lds_bytes, s>>>(a);
    return hipGetLastError();
}

template <bool BF16, bool OUTVEC>
hipError_t dispatch_rows(const Problem& p, int32_t* leaf_idx, const int32_t* given_leaf, hipStream_t s) {
    const int64_t vecs = (OUTVEC && p.O > p.D ? p.O : p.D) / Elem<BF16>::kPerVec;
    // (vectors per lane, levels per round trip): 2^S - 1 rows of NV vectors stay under 32 registers x 4
    if (vecs <= 64) return run_rows<BF16, 1, 3, OUTVEC>(p, leaf_idx, given_leaf, s);
    if (vecs <= 128) return run_rows<BF16, 2, 3, OUTVEC>(p, leaf_idx, given_leaf, s);
    if (vecs <= 256) return run_rows<BF16, 4, 3, OUTVEC>(p, leaf_idx, given_leaf, s);
    return run_rows<BF16, 8, 2, OUTVEC>(p, leaf_idx, given_leaf, s);
}

}  // namespace

// Whole aligned input rows of at most 512 pieces
bool token_rows_ok(const Problem& p) {
    return vec_ok(p.x, p.D, p.bf16) && vec_ok(p.leaf_w1, p.D, p.bf16) && (p.depth == 0 || vec_ok(p.node_w, p.D, p.bf16)) &&
           p.D / (p.bf16 ? 8 : 4) <= 8 * kWave;
}

// The line between the two kernels, from 3100 calls of both (us, token_block / this one).
// Leaves of more than 64 neurons are this one's: token_block_kernel takes 64 at a time with a barrier and a trip each, and its
// threads read their output pieces one after the other (107 tokens of 168 bf16 features, 160 neurons 12.8 / 9.4; 40 of 1040, 417
// neurons 98.9 / 36.2).  But batches that fill the chip with long rows next to short ones stay there while the leaf is no wider than
// 192, as this kernel holds both in registers of the longer one's length (2440 tokens of 376 bf16 features and 3328 outputs,
// 85 neurons 94 / 174), and so do output rows that are not whole pieces, which it writes element by element (366 tokens of
// 152 features and 113 outputs, 436 neurons 50 / 138), except those shorter than a piece, element-wise on both sides.
// Below 65 neurons token_block_kernel's trees are the faster ones, this kernel's leaves: up to 256 tokens the line is at 32 neurons
// (256 of 768 bf16 features, depth 9, 32 neurons 7.8 / 7.1, 16 neurons 6.5 / 6.7).  Beyond a token a compute unit this one has
// more blocks on it, while a row is 64 pieces (529 tokens of 144 fp32 features, depth 6, 38 neurons 10.2 / 7.2) and up to 128 for such
// leaves, or trees of more than eight levels while there are two tokens a unit (400 of 768 bf16, depth 9, 4 neurons 7.7 / 6.8, depth
// 4 5.6 / 6.1); longer rows take its registers (two thirds the speed at 256 pieces).  With output rows that are not whole pieces
// only narrow leaves (1502 of 288 bf16 features, 23 outputs, 16 neurons 17.1 / 11.2; 290 of 152 fp32, 55 outputs, 32 neurons
// 5.8 / 7.5).  A mixture's pick is a launch of its own with this kernel: short rows from 1024 tokens on (2825 tokens of 72
// features, 18 neurons 29.8 / 23.5).
bool token_rows_better(const Problem& p, bool picks) {
    if (g_token_kernel == 1 || !token_rows_ok(p)) return false;
    if (g_token_kernel == 2) return true;
    const int64_t per = p.bf16 ? 8 : 4;
    const int64_t longer = (p.D > p.O ? p.D : p.O) / per, shorter = (p.D > p.O ? p.O : p.D) / per;
    const bool full = p.T > 256, whole = rows_out_vec(p);
    if (p.O < per && (p.L > 64 || (full && !picks && longer <= 128))) return true;
    if (p.L > 64) return whole && (!full || longer <= 128 || 2 * shorter > longer || p.L > 192);
    if (picks) return whole && p.T > 1024 && longer <= 64;
    if (!full) return whole && p.L >= 32;
    if (!whole) return (p.L <= 32 && p.T > 512 && longer <= 64) || (p.L <= 16 && longer <= 128);
    return longer <= 64 || (longer <= 128 && (p.L >= 32 || (p.depth > 8 && p.T <= 512)));
}

hipError_t launch_token_rows(const Problem& p, int32_t* leaf_idx, hipStream_t s, const int32_t* given_leaf) {
    const bool ov = rows_out_vec(p);
    if (p.bf16) return ov ? dispatch_rows<true, true>(p, leaf_idx, given_leaf, s) : dispatch_rows<true, false>(p, leaf_idx, given_leaf, s);
    return ov ? dispatch_rows<false, true>(p, leaf_idx, given_leaf, s) : dispatch_rows<false, false>(p, leaf_idx, given_leaf, s);
}

}  // namespace fff
