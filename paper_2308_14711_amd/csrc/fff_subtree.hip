// The lower end of the tree on the matrix cores: tokens arrive grouped by the node they have reached
// (perm and offset of the bucketing stage), and a block takes 64 tokens of one such group through the
// last k levels below that node, the leaf network and the output row.
//
// Per token the last levels and the leaf are k node rows and L input rows that differ from token to
// token; for 64 tokens of one subtree they are (2^k - 1) node rows and 2^k L input rows that all of them
// share, a contraction [64, D] x [D, columns] with at most 128 columns.  So every pre-activation of the
// subtree is computed for every token of the tile, and the walk then only picks among the results:
//
//   1. S[token][column] over K = D: token rows and weight rows stream through a ring of LDS stages, 128
//      bytes of every row a stage, loaded straight to LDS (no registers in between); wave w owns
//      tokens 16 w .. 16 w + 15 against all columns, so that what has to be done to a token's elements
//      (layer norm) is done once.
//   2. every token walks k levels over its own row of S and takes the hidden neurons of its leaf.
//   3. the output rows.  bf16: one contraction over the subtree's (leaf, neuron) pairs, in which a token's activations are zero outside
//      its own leaf; fp32: the tile's tokens in leaf order, four columns a lane, the leaf's weights in registers.
//
// What bounds it: a tile reads its token rows, then writes its output rows, and the tiles of a compute unit do so nearly in step.
// 50432 tokens of 768 bf16 features, 256 leaves of 8 neurons, k = 0: 34 us (77 MB in at 4.5, 77 MB out at 5 TB/s, 3 us until the first
// row arrives) where the two leaf kernels take 18 + 19; fp32, 25216 tokens: 42 us, the gather kernel 65.  Measured and not kept: token
// rows straight to registers in the instruction's layout (64 bytes of 16 rows a load: 47 us), 96 to 128 tokens a block, output rows 16
// tokens at a time (more waves, but a chain of loads each: 36 -> 43 us), a deeper ring (no change).
// Normalised bf16 rows (fff_forward_block; 50432 tokens of 768, 4 neurons a node, 8 a leaf): levels from the root 60 -> 55 us, lower end 84 -> 76
// with the steps of the contraction interleaved, the statistics without masks and the residual rows requested a range ahead; the vector
// unit is busy half of the time.  Measured and not kept there: one round of blocks of 5 to 8 waves, or of 13 on a whole compute unit (131.8
// against 130.6 us for the call), stages in another order in each block (no change).
#include "fff_device.h"
#include "fff_internal.h"

namespace fff {
namespace {

constexpr int kTok = 64;            // tokens of a block
constexpr int kMaxCols = kSubtreeMaxColumns;
constexpr int kMaxL = 16;
constexpr int kFoldTiles = 4;       // tiles of a block of the bucketing launch that follows the levels from the root
constexpr int kMaxNormPieces = 128; // a normalised row: 1024 bf16 or 512 fp32 features

struct SubtreeArgs {
    const char* x;
    const char* node_w;      // linear nodes: [NN, D]; wide ones: [NN, n, D]
    const void* node_b;      // [NN]; [NN, n]
    const void* node_v;      // wide nodes: [NN, n] output weights
    const void* node_c;      // [NN] output biases
    const char* w1;
    const void* b1;
    const char* w2;
    const void* b2;
    const char* gamma;       // layer norm
    const char* beta;
    float2* stats;           // [T] mean and 1 / standard deviation of a token's row
    char* out;
    int32_t* leaf_idx;       // LEAF: the leaf, may be null; else the node reached
    int32_t* counts;         // levels from the root: [tiles, 2^k] tokens of each node
    const int32_t* perm;     // token ids grouped by node of level base_level
    const int32_t* offset;   // [groups + 1]; null: one group of all tokens in their order
    int64_t T;
    int groups, row_bytes, pieces, O, L, act, k, n, base_level, cols, node_cols, residual;
    int hidden_parts;        // bf16 values that make a hidden activation: 2, or 3
    float eps;
};

// the tile of this block: its group, its first slot and how many tokens it holds (0: no work)
struct Tile {
    int group, first, n;
};
// Tiles of 64 slots, group by group; the tiles are dealt to the XCDs in contiguous runs, so that a
// group's weight rows are fetched into one L2.  Every wave finds the tile for itself: a lane sums the tiles of
// `per` consecutive groups, a scan over the lanes says where the wanted tile lies.
__device__ __forceinline__ Tile find_tile(const int32_t* __restrict__ offset, int groups, int64_t T) {
    if (offset == nullptr) {
        const int64_t first = (int64_t)blockIdx.x * kTok;
        return Tile{0, (int)first, T - first < kTok ? (int)(T - first) : kTok};
    }
    const int lane = threadIdx.x & 63;
    const int per = (groups + kWave - 1) / kWave, g0 = lane * per;
    int own = 0;
    for (int i = 0; i < per; ++i) {
        const int g = g0 + i;
        if (g < groups) own += (offset[g + 1] - offset[g] + kTok - 1) / kTok;
    }
    int upto = own;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int v = __shfl_up(upto, d, kWave);
        upto += lane >= d ? v : 0;
    }
    const int total = __shfl(upto, kWave - 1, kWave);
    const int share = (total + kXcds - 1) / kXcds, in = (int)blockIdx.x / kXcds;
    const int tile = ((int)blockIdx.x % kXcds) * share + in;
    if (in >= share || tile >= total) return Tile{0, 0, 0};
    const uint64_t past = __ballot(upto > tile);
    const int at = __ffsll((unsigned long long)past) - 1;
    int g = at * per;
    int left = tile - (__shfl(upto, at, kWave) - __shfl(own, at, kWave));
    for (;; ++g) {                  // (the tile lies in one of this lane's groups)
        const int n = (offset[g + 1] - offset[g] + kTok - 1) / kTok;
        if (left < n) break;
        left -= n;
    }
    const int first = offset[g] + left * kTok, end = offset[g + 1];
    return Tile{g, first, end - first < kTok ? end - first : kTok};
}

// 16 bytes a lane straight to LDS: lane i's land at lds + 16 i.  Written as assembly because the compiler
// waits for every such load before any LDS access that follows it; the waits are wait_loads' below.  (m0 is never allocated
// to a value of the program, and nothing else in these kernels needs it.)
__device__ __forceinline__ void load_to_lds(const char* src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory");
}
// until at most N of this wave's loads are outstanding (they return in order)
template <int N> __device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

template <bool BF16>
__device__ __forceinline__ f32x4_t mfma_piece(const uint4& w, const uint4& x, f32x4_t acc) {
    if (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.x), __uint_as_float(x.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.y), __uint_as_float(x.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.z), __uint_as_float(x.z), acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.w), __uint_as_float(x.w), acc, 0, 0, 0);
}

__device__ __forceinline__ void load4(const float* p, float* f) {
    const float4 v = *(const float4*)p;
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

// s plus the elements of a piece
template <bool BF16> __device__ __forceinline__ float piece_sum(const uint4& v, float s) {
    if (BF16) {
        constexpr uint32_t ones = 0x3f803f80u;
        return dot2_bf16(v.w, ones, dot2_bf16(v.z, ones, dot2_bf16(v.y, ones, dot2_bf16(v.x, ones, s))));
    }
    return s + __uint_as_float(v.x) + __uint_as_float(v.y) + __uint_as_float(v.z) + __uint_as_float(v.w);
}

struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

// The ring: 128 bytes of every row a stage, 64 token rows and NB blocks of 16 columns (whole groups of 32 rows), as deep as
// leaves two blocks a compute unit.
constexpr int stage_rows(int nb) { return kTok + 32 * ((nb + 1) / 2); }
constexpr int ring_stages(int nb) { return nb > 2 ? 3 : 4; }
constexpr int ring_bytes(int nb) { return ring_stages(nb) * stage_rows(nb) * 128; }

// Hidden activations of a tile for the output contraction: a row of `steps` groups of 16 pairs, pair 4 i + e as bf16 values hi and lo at
// elements e and 4 + e of piece i; rows an odd number of pieces apart.
constexpr int hidden_pitch(int steps) { return 4 * steps + 1; }

// nodes: one neuron, n hidden neurons, n hidden neurons on the normalised token (bf16: in two parts, or in three)
enum { kLinear, kWide, kNorm, kNormWhole };

// A piece of a token's row as the matrix instruction takes it.  A normalised bf16 row is the sum of two bf16
// rows, hi = bf16(z) and lo = bf16(z - hi): a relative 2^-17 of each element, as block_group_kernel keeps it; or of three,
// lo2 = z - hi - lo, which is all of the fp32 row, as block_kernel keeps it.
template <bool BF16, bool LN, bool THREE>
__device__ __forceinline__ void token_piece(const uint4& x, const uint4& g, const uint4& b, float mean, float rstd, uint4* hi, uint4* lo,
                                            uint4* lo2) {
    if (!LN) {
        *hi = x;
        return;
    }
    constexpr int E = Elem<BF16>::kPerVec;
    float f[E], gf[E], bf[E];
    widen<BF16>(x, f);
    widen<BF16>(g, gf);
    widen<BF16>(b, bf);
#pragma unroll
    for (int e = 0; e < E; ++e) f[e] = fmaf((f[e] - mean) * rstd, gf[e], bf[e]);
    *hi = narrow<BF16>(f);
    if (BF16) {
        widen<BF16>(*hi, gf);
#pragma unroll
        for (int e = 0; e < E; ++e) f[e] -= gf[e];
        *lo = narrow<BF16>(f);
        if (THREE) {
            widen<BF16>(*lo, gf);
#pragma unroll
            for (int e = 0; e < E; ++e) f[e] -= gf[e];
            *lo2 = narrow<BF16>(f);
        }
    }
}

template <int LB>
__device__ __forceinline__ void write_rows_f32(const SubtreeArgs& a, const float* hid, const int32_t* s_tok, const int32_t* s_sub, int n,
                                               int64_t first_leaf);
template <bool RESIDUAL>
__device__ __forceinline__ void write_rows_mfma(const SubtreeArgs& a, const uint4* hid, const uint2* third, int third_pitch, const int32_t* s_tok,
                                                const int32_t* s_sub, int n, int64_t first_leaf, int steps);

// LEAF: the last k levels, the leaf and the output row; else k levels, the node reached, and (from the root) the tile's counts.
template <bool BF16, int NODES, bool LEAF, int NB>
__global__ __launch_bounds__(256, 2) void subtree_kernel(const SubtreeArgs a) {
    constexpr bool LN = NODES >= kNorm, WIDE = NODES != kLinear, THREE = BF16 && NODES == kNormWhole;
    constexpr int kStages = ring_stages(NB), kRowsW = stage_rows(NB) - kTok;
    constexpr int kLoads = 2 + kRowsW / 32;                 // of a wave, a stage
    constexpr int kStagePieces = stage_rows(NB) * 8;
    constexpr int kPitch = 16 * NB + 4;
    static_assert(kTok * kPitch * 4 + (BF16 ? kTok * hidden_pitch(NB + 1) * 16 : kTok * kMaxL * 4) <= ring_bytes(NB), "the rows of the walk and the leaf fit the ring");
    __shared__ uint4 ring[kStages * kStagePieces];
    __shared__ uint4 s_gamma[LN ? kMaxNormPieces : 1], s_beta[LN ? kMaxNormPieces : 1];
    __shared__ int32_t s_tok[kTok], s_sub[kTok];
    __shared__ float s_bias[kMaxCols], s_v[kMaxCols], s_c[kMaxCols];
    __shared__ int32_t s_count[kMaxCols];
    const Tile at = find_tile(a.offset, a.groups, a.T);
    if (at.n <= 0) return;                                  // (the whole block)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = lane & 15, kg = lane >> 4;
    const int64_t root = ((int64_t)1 << a.base_level) - 1 + at.group;      // heap index
    const int64_t first_leaf = (int64_t)at.group << a.k;                    // (or node, of level base_level + k)
    const int n = WIDE ? a.n : 1;
    const int tok = 16 * wv + j;

    const auto token = [&](int r) -> int64_t {
        r = at.first + (r < at.n ? r : 0);
        return a.perm ? a.perm[r] : r;
    };
    // weight row of a column: node rows level by level, then the subtree's leaves
    const auto subtree_node = [&](int i) {
        const int level = 31 - __clz(i + 1);
        return ((root + 1) << level) - 1 + (i + 1 - (1 << level));
    };
    const auto node_row = [&](int c) { return subtree_node(c / n) * n + c % n; };
    // loader roles: lane l brings row l / 8 of 8 consecutive rows; its 16-byte slot holds piece `pl` of the row (tile_swz)
    const int lrow = lane >> 3, pl = ((lane & 7) - lds_rot(lrow)) & 7;
    const char* src[kLoads];
#pragma unroll
    for (int i = 0; i < 2; ++i) src[i] = a.x + token(16 * wv + 8 * i + lrow) * a.row_bytes;
#pragma unroll
    for (int i = 0; i < kRowsW / 32; ++i) {
        int c = 32 * i + 8 * wv + lrow;
        c = c < a.cols ? c : a.cols - 1;
        src[2 + i] = !LEAF || c < a.node_cols ? a.node_w + node_row(c) * a.row_bytes
                                              : a.w1 + (first_leaf * a.L + (c - a.node_cols)) * a.row_bytes;
    }
    const uint32_t ring_at = lds_address(ring);
    const int chunks = (a.pieces + 7) / 8;
    const auto request = [&](int kc) {
        const int64_t off = 8 * kc + pl < a.pieces ? kc * 128 + pl * 16 : 0;       // (pieces past the row: its first one, masked below)
        const uint32_t to = ring_at + (uint32_t)(kc % kStages) * (kStagePieces * 16);
#pragma unroll
        for (int i = 0; i < 2; ++i) load_to_lds(src[i] + off, __builtin_amdgcn_readfirstlane(to + (16 * wv + 8 * i) * 128));
#pragma unroll
        for (int i = 0; i < kRowsW / 32; ++i)
            load_to_lds(src[2 + i] + off, __builtin_amdgcn_readfirstlane(to + (kTok + 32 * i + 8 * wv) * 128));
    };
    // (what the compiler loads comes before the ring's first requests: it waits for its own loads by waiting for everything)
    if (tid < a.cols) {
        const bool node = !LEAF || tid < a.node_cols;
        s_bias[tid] = node ? Elem<BF16>::load(a.node_b, node_row(tid)) : Elem<BF16>::load(a.b1, first_leaf * a.L + (tid - a.node_cols));
        if (WIDE && node) s_v[tid] = Elem<BF16>::load(a.node_v, node_row(tid));
        if (WIDE && tid < (1 << a.k) - 1) s_c[tid] = Elem<BF16>::load(a.node_c, subtree_node(tid));
    }
    if (!LEAF && tid < kMaxCols) s_count[tid] = 0;

    // ---- mean and deviation of the wave's tokens, 16 lanes a row, all rows requested at once (and left for the later launches)
    float mean = 0.0f, rstd = 0.0f;
    if (LN) {
        for (int i = tid; i < a.pieces; i += 256) {
            s_gamma[i] = ((const uint4*)a.gamma)[i];
            s_beta[i] = ((const uint4*)a.beta)[i];
        }
        if (a.base_level == 0) {
            constexpr int E = Elem<BF16>::kPerVec, NV = kMaxNormPieces / 16;
            const float width = (float)(a.pieces * E);
            uint4 v[4][NV];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint4* const xr = (const uint4*)(a.x + token(16 * wv + 4 * r + kg) * a.row_bytes);
#pragma unroll
                for (int i = 0; i < NV; ++i)
                    if (16 * i < a.pieces) v[r][i] = xr[j + 16 * i < a.pieces ? j + 16 * i : 0];
            }
            float2 st[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // (a vector unit busy half of this launch's time: pieces inside the row need no masks, and two bf16 values are added at once)
                float s = 0.0f, f[E];
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    if (16 * i >= a.pieces) continue;
                    if (16 * i + 16 > a.pieces) v[r][i] = keep_if(j + 16 * i < a.pieces, v[r][i]);
                    s = piece_sum<BF16>(v[r][i], s);
                }
                const float mu = group_sum<16>(s) / width;
                float q = 0.0f;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    if (16 * i >= a.pieces) continue;
                    widen<BF16>(v[r][i], f);
                    float p = 0.0f;
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const float d = f[e] - mu;
                        p = fmaf(d, d, p);
                    }
                    q += 16 * i + 16 <= a.pieces || j + 16 * i < a.pieces ? p : 0.0f;
                }
                const float var = group_sum<16>(q) / width;
                st[r] = make_float2(mu, 1.0f / sqrtf(var + a.eps));
            }
            // token j of the wave is row 4 (j / 4) + j % 4: held by the lanes of group j % 4, as their r = j / 4
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float m = __shfl(st[r].x, 16 * (j & 3), kWave), d = __shfl(st[r].y, 16 * (j & 3), kWave);
                if (j >> 2 == r) mean = m, rstd = d;
            }
            if (kg == 0 && tok < at.n) a.stats[token(tok)] = make_float2(mean, rstd);
        } else {
            const float2 st = a.stats[token(tok)];
            mean = st.x;
            rstd = st.y;
        }
    }

    // fp32 products are added up 16 at a time, from zero, and these sums with what their additions lose kept beside them (mostly in the
    // shadow of the matrix instructions; 78 -> 80 us): one chain over the whole row would round as often as the row is long (25216
    // tokens of 768, 8 neurons: results off by 4.1e-7 in one chain, 0.93e-7 so, 0.99e-7 in the gather kernel, which adds over lanes).
    // The second and third bf16 rows of a normalised token in three parts have sums of their own as well.  Either remainder counts only where
    // it is finite: an infinite product or sum makes inf - inf of it, and the sum beside it is the right result alone.  (Two parts go into
    // one sum, as in block_group_kernel, whose weights have to be finite too.)
    constexpr bool REST = !BF16 || THREE;
    f32x4_t acc[NB], rest[REST ? NB : 1];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = rest[REST ? b : 0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const auto multiply = [&](int kc, auto tail) {
        const uint4* xs = ring + (kc % kStages) * kStagePieces;
        const uint4* ws = xs + kTok * 8;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int piece = 8 * kc + 2 * kg + u;
            const bool in = !decltype(tail)::value || piece < a.pieces;
            const int gp = LN ? (in ? piece : 0) : 0;
            uint4 hi, lo, lo2;
            token_piece<BF16, LN, THREE>(xs[tile_swz(tok, 2 * kg + u)], s_gamma[gp], s_beta[gp], mean, rstd, &hi, &lo, &lo2);
            if (decltype(tail)::value) hi = keep_if(in, hi);
            if (decltype(tail)::value && LN && BF16) lo = keep_if(in, lo);
            uint4 wr[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                uint4 wvv = ws[tile_swz(16 * b + j, 2 * kg + u)];
                if (decltype(tail)::value) wvv = keep_if(in, wvv);
                wr[b] = wvv;
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (BF16) {
                    acc[b] = mfma_piece<BF16>(wr[b], hi, acc[b]);
                } else {
                    const f32x4_t t = mfma_piece<BF16>(wr[b], hi, f32x4_t{0.f, 0.f, 0.f, 0.f}), sum = acc[b] + t, part = sum - acc[b];
                    rest[REST ? b : 0] += (acc[b] - (sum - part)) + (t - part);
                    acc[b] = sum;
                }
            }
            if (LN && BF16 && !THREE) {
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = mfma_piece<BF16>(wr[b], lo, acc[b]);
            }
            if (THREE) {
                if (decltype(tail)::value) lo2 = keep_if(in, lo2);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[REST ? b : 0] = mfma_piece<BF16>(wr[b], lo, rest[REST ? b : 0]);
#pragma unroll
                for (int b = 0; b < NB; ++b) rest[REST ? b : 0] = mfma_piece<BF16>(wr[b], lo2, rest[REST ? b : 0]);
            }
        }
    };
    for (int kc = 0; kc < kStages - 1 && kc < chunks; ++kc) request(kc);
    // stage kc has landed for this wave once no more than the loads requested after it are outstanding, for
    // the block after the barrier; the barrier also says that everyone has read stage kc - 1, which the
    // next request overwrites
    const auto next_stage = [&](int kc) {
        const int ahead = chunks - 1 - kc < kStages - 2 ? chunks - 1 - kc : kStages - 2;
        if (ahead >= 2) wait_loads<2 * kLoads>();
        else if (ahead == 1) wait_loads<kLoads>();
        else wait_loads<0>();
        __syncthreads();
        if (kc + kStages - 1 < chunks) request(kc + kStages - 1);
    };
    int done = 0;
    if (BF16 && LN && !THREE) {
        // Normalising a piece takes the vector unit about as long as the piece's products take the matrix cores, and the waves of a
        // compute unit leave the barrier in step: one after the other they take the sum of both (2800 cycles a stage for two blocks).  So a
        // step of 32 elements is normalised between the matrix instructions of the step before it, and read from LDS ahead of them.
        struct Step {
            uint4 x, g, b, w[NB], hi, lo;
        } even, odd;
        const auto read = [&](int kc, int u, Step& s) {
            const uint4* xs = ring + (kc % kStages) * kStagePieces;
            const int piece = 8 * kc + 2 * kg + u;
            s.x = xs[tile_swz(tok, 2 * kg + u)];
            s.g = s_gamma[LN ? piece : 0];
            s.b = s_beta[LN ? piece : 0];
#pragma unroll
            for (int b = 0; b < NB; ++b) s.w[b] = xs[kTok * 8 + tile_swz(16 * b + j, 2 * kg + u)];
        };
        const auto normalise = [&](Step& s) {
            uint4 lo2;
            token_piece<BF16, LN, THREE>(s.x, s.g, s.b, mean, rstd, &s.hi, &s.lo, &lo2);
        };
        const auto products = [&](const Step& s) {
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = mfma_piece<BF16>(s.w[b], s.hi, acc[b]);
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = mfma_piece<BF16>(s.w[b], s.lo, acc[b]);
        };
        const auto interleave = [&] {
            __builtin_amdgcn_sched_group_barrier(0x100, 3 + NB, 0);                     // LDS reads
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                        // a matrix instruction
                __builtin_amdgcn_sched_group_barrier(0x2, (80 + 2 * NB - 1) / (2 * NB), 0);    // its share of the normalisation
            }
        };
        const int full = a.pieces / 8;
        if (full > 0) {
            next_stage(0);
            read(0, 0, even);
            normalise(even);
            for (; done < full - 1; ++done) {
                read(done, 1, odd);
                products(even);
                normalise(odd);
                interleave();
                next_stage(done + 1);
                read(done + 1, 0, even);
                products(odd);
                normalise(even);
                interleave();
            }
            read(done, 1, odd);
            products(even);
            normalise(odd);
            products(odd);
            ++done;
        }
    }
    for (int kc = done; kc < chunks; ++kc) {
        next_stage(kc);
        if (8 * kc + 8 <= a.pieces) multiply(kc, No());
        else multiply(kc, Yes());
    }
    __syncthreads();

    // ---- the walk: a token's four lanes (j, 0..3) go together
    float* const S = (float*)ring;                          // [kTok][kPitch]
    float* const hid = S + kTok * kPitch;                   // the hidden activations
    if (REST) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float r = rest[REST ? b : 0][q];
                acc[b][q] += fabsf(r) < __builtin_inff() ? r : 0.0f;
            }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) *(f32x4_t*)(S + tok * kPitch + 16 * b + 4 * kg) = acc[b];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const float* const row = S + tok * kPitch;
    int node = 0;
    for (int m = 0; m < a.k; ++m) {
        float logit;
        if (!WIDE) {
            logit = row[node] + s_bias[node];
        } else {
            // each of the token's lanes takes a quarter of the node's hidden neurons; all end with the same bits
            float part = 0.0f;
            for (int i = kg; i < a.n; i += 4) {
                const int c = node * a.n + i;
                part = fmaf(s_v[c], activate(row[c] + s_bias[c], a.act), part);
            }
            part += __shfl_xor(part, 16, kWave);
            part += __shfl_xor(part, 32, kWave);
            logit = part + s_c[node];
        }
        node = 2 * node + 1 + (logit >= 0.0f ? 1 : 0);
    }
    const int sub = node - ((1 << a.k) - 1);
    const bool live = tok < at.n;
    if (!LEAF) {
        if (kg == 0 && live) {
            a.leaf_idx[token(tok)] = (int32_t)(first_leaf + sub);
            if (a.counts) atomicAdd(&s_count[sub], 1);
        }
        if (a.counts) {
            __syncthreads();
            if (tid < 1 << a.k) a.counts[((int64_t)blockIdx.x << a.k) + tid] = s_count[tid];
        }
        return;
    }
    float h[kMaxL / 4];
#pragma unroll
    for (int i = 0; i < kMaxL / 4; ++i) {
        const int r = 4 * i + kg, c = a.node_cols + sub * a.L + r;
        h[i] = r < a.L ? activate(row[c] + s_bias[c], a.act) : 0.0f;
    }
    const int32_t t = (int32_t)token(tok);
    if (kg == 0 && live && a.leaf_idx) a.leaf_idx[t] = (int32_t)(first_leaf + sub);
    if (BF16) {
        const int pairs = a.L << a.k, steps = (pairs + (1 << a.k) + 15) / 16, pitch = hidden_pitch(steps);
        uint4* const hrow = (uint4*)hid + tok * pitch;
        for (int i = kg; i < 4 * steps; i += 4) hrow[i] = make_uint4(0, 0, 0, 0);
        // (the third values go where the token's row of S was, whose readers are this token's lanes, done with it)
        constexpr int kThirdPitch = kPitch / 2;
        static_assert(4 * (NB + 1) + 1 <= kThirdPitch, "the third values of a token fit its row of S");
        uint2* const third = (uint2*)S;
        uint2* const trow = third + tok * kThirdPitch;
        const bool exact = a.hidden_parts == 3;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (exact)
            for (int i = kg; i < 4 * steps; i += 4) trow[i] = make_uint2(0, 0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const auto put = [&](int p, float v) {
            uint16_t* const at = (uint16_t*)(hrow + p / 4) + p % 4;
            const uint16_t near = f32_to_bf16(v);
            const bool whole = !(fabsf(v) < __builtin_inff());                                   // (an infinite value is its hi alone)
            const uint16_t hi = !whole && (near & 0x7fff) == 0x7f80 ? near - 1 : near;           // (a finite one does not round to infinity)
            const float left = whole ? 0.0f : v - bf16_to_f32(hi);
            const uint16_t lo = f32_to_bf16(left);
            at[0] = hi;
            at[4] = lo;
            if (exact) ((uint16_t*)(trow + p / 4))[p % 4] = f32_to_bf16(left - bf16_to_f32(lo));
        };
#pragma unroll
        for (int i = 0; i < kMaxL / 4; ++i)
            if (4 * i + kg < a.L) put(sub * a.L + 4 * i + kg, h[i]);
        if (kg == 0) {
            put(pairs + sub, 1.0f);
            s_tok[tok] = t;
            s_sub[tok] = sub;
        }
        __syncthreads();
        write_rows_mfma<WIDE>(a, (const uint4*)hid, exact ? third : nullptr, kThirdPitch, s_tok, s_sub, at.n, first_leaf, steps);
        return;
    }
    if (kg == 0) s_sub[tok] = live ? sub : 1 << a.k;        // tokens past the tile's end sort last
    __syncthreads();
    // position of every token in leaf order (every wave, all 64 tokens)
    const int of = s_sub[lane];
    int pos = 0, before = 0;
    for (int s = 0; s <= 1 << a.k; ++s) {
        const uint64_t m = __ballot(of == s);
        if (of == s) pos = before + __popcll(m & (((uint64_t)1 << lane) - 1));
        before += __popcll(m);
    }
    const int mine = __shfl(pos, tok, kWave);
    __syncthreads();
    if (kg == 0) {
        s_tok[mine] = t;
        s_sub[mine] = sub;
    }
#pragma unroll
    for (int i = 0; i < kMaxL / 4; ++i) hid[mine * kMaxL + 4 * i + kg] = h[i];
    __syncthreads();
    if (a.L <= 4) write_rows_f32<4>(a, hid, s_tok, s_sub, at.n, first_leaf);
    else if (a.L <= 8) write_rows_f32<8>(a, hid, s_tok, s_sub, at.n, first_leaf);
    else write_rows_f32<16>(a, hid, s_tok, s_sub, at.n, first_leaf);
}

// Output rows of 16 tokens in leaf order, by one wave: four columns a lane, the leaf's weights for
// them in registers (rows past L are zeros against zeros).
template <int LB>
__device__ __forceinline__ void write_rows_f32(const SubtreeArgs& a, const float* hid, const int32_t* s_tok, const int32_t* s_sub,
                                           int n, int64_t first_leaf) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i0 = 16 * wv, cnt = n - i0 < 16 ? n - i0 : 16;
    if (cnt <= 0) return;
    const int toks = s_tok[i0 + (lane & 15)], subs = s_sub[i0 + (lane & 15)];
    const int O = a.O;
    for (int c0 = 0; c0 < O; c0 += 4 * kWave) {
        const int c = c0 + 4 * lane, cc = c < O ? c : O - 4;
        int cur = -1;
        float w[LB][4], bias[4];
        for (int i = 0; i < cnt; ++i) {
            const int sub = __builtin_amdgcn_readlane(subs, i);
            const int64_t t = __builtin_amdgcn_readlane(toks, i);
            if (sub != cur) {
                cur = sub;
                const int64_t leaf = first_leaf + sub;
                load4((const float*)a.b2 + leaf * O + cc, bias);
#pragma unroll
                for (int r = 0; r < LB; ++r) load4((const float*)a.w2 + (leaf * a.L + (r < a.L ? r : 0)) * O + cc, w[r]);
#pragma unroll
                for (int r = 0; r < LB; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[r][e] = r < a.L ? w[r][e] : 0.0f;
            }
            float y[4] = {bias[0], bias[1], bias[2], bias[3]};
#pragma unroll
            for (int r4 = 0; r4 < LB / 4; ++r4) {
                const float4 h = *(const float4*)(hid + (i0 + i) * kMaxL + 4 * r4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[e] = fmaf(h.x, w[4 * r4][e], y[e]);
                    y[e] = fmaf(h.y, w[4 * r4 + 1][e], y[e]);
                    y[e] = fmaf(h.z, w[4 * r4 + 2][e], y[e]);
                    y[e] = fmaf(h.w, w[4 * r4 + 3][e], y[e]);
                }
            }
            if (a.residual) {
                float f[4];
                load4((const float*)a.x + t * O + cc, f);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] += f[e];
            }
            if (c < O) __builtin_nontemporal_store(f32x4_t{y[0], y[1], y[2], y[3]}, (f32x4_t*)((float*)a.out + t * O + c));
        }
    }
}

// The same for bf16 on the matrix cores, for the whole tile at once: out[token][o] over (leaf, neuron) pairs and, for the
// biases, one pair a leaf whose activation is 1.  A token's activations are zero outside its own leaf; they are the sum of two
// bf16 values, so that 16 pairs fill the 32 K slots of an instruction against the same weights, or (third) of three, which is
// all of the fp32 value: 16 more slots (fff_forward_block, 50432 tokens of 768, 4 neurons a node, 8 a leaf: 139.7 -> 141.1 us; two
// steps' third values in one instruction of 32 slots spill: 150).  Each wave takes 64
// columns of all 64 tokens at a time, so that a weight is loaded, and turned around, once a tile: weights are
// contiguous along o while the instruction wants K contiguous, so a lane loads 4 consecutive o of its 4 rows, and
// column j of the c-th instruction stands for o = 64 R + 4 j + c.
__device__ __forceinline__ uint32_t pair_of(uint32_t a, uint32_t b, int hi) {
    return __builtin_amdgcn_perm(b, a, hi ? 0x07060302u : 0x05040100u);
}

// Columns 64 r .. 64 r + 63 of the tile's output rows, a token after the other from its own leaf's weights: for weights that
// are not finite, which against the zeros of another leaf's token, or the lower half of an activation, would make NaN.
__device__ __forceinline__ void write_rows_apart(const SubtreeArgs& a, const uint4* hid, int pitch, const uint2* third, int third_pitch,
                                              const int32_t* s_tok, const int32_t* s_sub, int n, int64_t first_leaf, int r) {
    const int lane = threadIdx.x & 63, O = a.O, o = 64 * r + lane;
    if (o >= O) return;
    for (int i = 0; i < n; ++i) {
        const int64_t t = s_tok[i], leaf = first_leaf + s_sub[i];
        const uint16_t* const h = (const uint16_t*)(hid + i * pitch);
        float y = Elem<true>::load(a.b2, leaf * O + o);
        for (int k = 0; k < a.L; ++k) {
            const int p = s_sub[i] * a.L + k;
            float v = bf16_to_f32(h[8 * (p / 4) + 4 + p % 4]);
            if (third) v += bf16_to_f32(((const uint16_t*)(third + i * third_pitch))[p]);
            v += bf16_to_f32(h[8 * (p / 4) + p % 4]);
            y = fmaf(v, Elem<true>::load(a.w2, (leaf * a.L + k) * O + o), y);
        }
        if (a.residual) y += Elem<true>::load(a.x, t * O + o);
        Elem<true>::store(a.out, t * O + o, y);
    }
}

template <bool RESIDUAL>
__device__ __forceinline__ void write_rows_mfma(const SubtreeArgs& a, const uint4* hid, const uint2* third, int third_pitch, const int32_t* s_tok,
                                                const int32_t* s_sub, int n, int64_t first_leaf, int steps) {
    constexpr int kAhead = 5;                                // steps requested together
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = lane & 15, kg = lane >> 4;
    const int O = a.O, ranges = (O + 63) / 64, pairs = a.L << a.k, rows = pairs + (1 << a.k), pitch = hidden_pitch(steps);
    const bool residual = RESIDUAL && a.residual;
    const uint16_t* const w2 = (const uint16_t*)a.w2 + first_leaf * a.L * O;
    const uint16_t* const b2 = (const uint16_t*)a.b2 + (first_leaf - pairs) * O;
    const auto column = [&](int r) { return 64 * r + 4 * j < O ? 64 * r + 4 * j : O - 4; };
    uint2 w[kAhead][4];
    const auto request_weights = [&](int r, int s0) {
        const int oc = column(r);
#pragma unroll
        for (int s = 0; s < kAhead; ++s) {
            if (s0 + s >= steps) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int p = 16 * (s0 + s) + 4 * kg + q, pc = p < rows ? p : 0;
                w[s][q] = *(const uint2*)((pc < pairs ? w2 : b2) + (int64_t)pc * O + oc);
            }
        }
    };
    const auto request_tokens = [&](int r, uint2 (&x)[4][4]) {
        if (!residual) return;
        const int oc = column(r);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int4 t = *(const int4*)(s_tok + 16 * g + 4 * kg);
            const int32_t tq[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) x[g][q] = *(const uint2*)((const uint16_t*)a.x + (int64_t)tq[q] * O + oc);
        }
    };
    uint2 x[4][4];
    if (wv < ranges) {
        request_weights(wv, 0);
        request_tokens(wv, x);
    }
    for (int r = wv; r < ranges; r += 4) {
        // largest magnitudes (as bit patterns) of the weights met
        u16x2_t most = {0, 0};
        f32x4_t acc[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[g][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < steps; s0 += kAhead) {
            if (s0 > 0) request_weights(r, s0);
#pragma unroll
            for (int s = 0; s < kAhead; ++s) {
                if (s0 + s >= steps) continue;
                uint2 v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool in = 16 * (s0 + s) + 4 * kg + q < rows;
                    v[q] = make_uint2(in ? w[s][q].x : 0u, in ? w[s][q].y : 0u);
                    most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2_t, v[q].x & 0x7fff7fffu));
                    most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2_t, v[q].y & 0x7fff7fffu));
                }
                bf16x8_t fb[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t p01 = pair_of(c < 2 ? v[0].x : v[0].y, c < 2 ? v[1].x : v[1].y, c & 1);
                    const uint32_t p23 = pair_of(c < 2 ? v[2].x : v[2].y, c < 2 ? v[3].x : v[3].y, c & 1);
                    fb[c] = __builtin_bit_cast(bf16x8_t, make_uint4(p01, p23, p01, p23));
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const bf16x8_t fa = __builtin_bit_cast(bf16x8_t, hid[(16 * g + j) * pitch + 4 * (s0 + s) + kg]);
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[c], acc[g][c], 0, 0, 0);
                }
                if (third) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const s16x4_t fa = __builtin_bit_cast(s16x4_t, third[(16 * g + j) * third_pitch + 4 * (s0 + s) + kg]);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint4 w4 = __builtin_bit_cast(uint4, fb[c]);
                            acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa, __builtin_bit_cast(s16x4_t, make_uint2(w4.x, w4.y)), acc[g][c], 0, 0, 0);
                        }
                    }
                }
            }
        }
        if (residual) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[g][0][q] += bf16_lo(x[g][q].x);
                    acc[g][1][q] += bf16_hi(x[g][q].x);
                    acc[g][2][q] += bf16_lo(x[g][q].y);
                    acc[g][3][q] += bf16_hi(x[g][q].y);
                }
        }
        // the next range's weights and tokens before this one's rows leave: a wait for a load is a wait for everything before it
        // (the leaf launch of 50432 tokens of 768, 8 neurons, with residual: 84 -> 79 us)
        if (r + 4 < ranges) {
            request_weights(r + 4, 0);
            request_tokens(r + 4, x);
        }
        if (__ballot(most.x >= 0x7f80 || most.y >= 0x7f80)) {
            write_rows_apart(a, hid, pitch, third, third_pitch, s_tok, s_sub, n, first_leaf, r);
            continue;
        }
        const bool whole = 64 * r + 64 <= O;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (16 * g >= n) continue;
            // rows past the tile's end repeat its first token: the same values to the same place
            const int4 t = *(const int4*)(s_tok + 16 * g + 4 * kg);
            const int32_t tq[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y[4] = {acc[g][0][q], acc[g][1][q], acc[g][2][q], acc[g][3][q]};
                const u32x2_t v = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                u32x2_t* const to = (u32x2_t*)((uint16_t*)a.out + (int64_t)tq[q] * O + 64 * r + 4 * j);
                if (whole) __builtin_nontemporal_store(v, to);
                else if (64 * r + 4 * j < O) __builtin_nontemporal_store(v, to);
            }
        }
    }
}

template <bool BF16, int NODES, bool LEAF, int NB> hipError_t run(const SubtreeArgs& a, int64_t tiles, hipStream_t s) {
    note_launch("subtree_kernel<%s,%s%s,%d> k=%d", BF16 ? "bf16" : "f32", NODES == kNorm ? "norm," : NODES == kNormWhole ? "norm3," : NODES == kWide ? "wide," : "", LEAF ? "leaf" : "levels", NB, a.k);
    subtree_kernel<BF16, NODES, LEAF, NB><<<dim3((unsigned)((tiles + kXcds - 1) / kXcds * kXcds)), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

template <bool BF16, int NODES, bool LEAF> hipError_t dispatch_cols(const SubtreeArgs& a, int64_t tiles, hipStream_t s) {
    const int nb = (a.cols + 15) / 16;
    if (nb <= 1) return run<BF16, NODES, LEAF, 1>(a, tiles, s);
    if (nb <= 2) return run<BF16, NODES, LEAF, 2>(a, tiles, s);
    if (nb <= 4) return run<BF16, NODES, LEAF, 4>(a, tiles, s);
    if (nb <= 6) return run<BF16, NODES, LEAF, 6>(a, tiles, s);
    return run<BF16, NODES, LEAF, 8>(a, tiles, s);
}
template <int NODES, bool LEAF> hipError_t dispatch(const SubtreeArgs& a, bool bf16, int64_t tiles, hipStream_t s) {
    return bf16 ? dispatch_cols<true, NODES, LEAF>(a, tiles, s) : dispatch_cols<false, NODES, LEAF>(a, tiles, s);
}
template <bool LEAF> hipError_t dispatch_wide(const Problem& p, const SubtreeArgs& a, int64_t tiles, hipStream_t s) {
    if (!a.gamma) return dispatch<kWide, LEAF>(a, p.bf16, tiles, s);
    return p.bf16 && subtree_row_parts(p) == 3 ? dispatch_cols<true, kNormWhole, LEAF>(a, tiles, s) : dispatch<kNorm, LEAF>(a, p.bf16, tiles, s);
}

SubtreeArgs make_args(const Problem& p, int base_level, int k, const WideNodes* wide, float* stats, bool fp32_hidden) {
    SubtreeArgs a = {};
    a.x = (const char*)p.x;
    a.node_w = (const char*)(wide ? wide->w1 : p.node_w);
    a.node_b = wide ? wide->b1 : p.node_b;
    if (wide) {
        a.node_v = wide->w2;
        a.node_c = wide->b2;
        a.gamma = (const char*)wide->gamma;
        a.beta = (const char*)wide->beta;
        a.n = wide->n;
        a.residual = wide->residual;
        a.eps = wide->eps;
    }
    a.stats = (float2*)stats;
    a.w1 = (const char*)p.leaf_w1;
    a.b1 = p.leaf_b1;
    a.w2 = (const char*)p.leaf_w2;
    a.b2 = p.leaf_b2;
    a.out = (char*)p.out;
    a.T = p.T;
    a.groups = 1 << base_level;
    a.row_bytes = (int)(p.D * (p.bf16 ? 2 : 4));
    a.pieces = a.row_bytes / 16;
    a.O = (int)p.O;
    a.L = p.L;
    a.act = p.act;
    a.k = k;
    a.base_level = base_level;
    a.node_cols = ((1 << k) - 1) * (wide ? wide->n : 1);
    // as precise as the launch that a call takes otherwise: fff_forward_block's kernels have activations in fp32
    a.hidden_parts = wide || fp32_hidden ? 3 : 2;
    return a;
}

}  // namespace

// Normalised bf16 rows: as precise as the launch that a call takes otherwise, which has pairs where 16 lanes hold the longest
// row of a call, and fp32 beyond.
int subtree_row_parts(const Problem& p) { return p.O * 2 > kMaxNormPieces * 16 ? 3 : 2; }

int64_t subtree_columns(int k, int node_size, int L) { return (((int64_t)1 << k) - 1) * node_size + ((int64_t)L << k); }

// Whole aligned rows, leaves of up to 16 neurons, up to 128 columns under a group's node and 1024 groups.
bool subtree_shape_ok(const Problem& p, int k, const WideNodes* wide) {
    if (k < 0 || k > p.depth || p.depth - k > 10 || k > 4 || p.L > kMaxL) return false;
    const void* const nodes = wide ? wide->w1 : p.node_w;
    const bool norm = wide && wide->gamma;
    return subtree_columns(k, wide ? wide->n : 1, p.L) <= kMaxCols && vec_ok(p.x, p.D, p.bf16) && (k == 0 || vec_ok(nodes, p.D, p.bf16)) &&
           vec_ok(p.leaf_w1, p.D, p.bf16) && vec_ok(p.leaf_w2, p.O, p.bf16) && vec_ok(p.leaf_b2, p.O, p.bf16) &&
           vec_ok(p.out, p.O, p.bf16) && p.D < (1 << 28) && p.O < (1 << 28) &&
           (!norm || (vec_ok(wide->gamma, p.D, p.bf16) && vec_ok(wide->beta, p.D, p.bf16) && p.D * (p.bf16 ? 2 : 4) <= kMaxNormPieces * 16));
}

hipError_t launch_subtree(const Problem& p, int k, const int32_t* perm, const int32_t* offset, int32_t* leaf_idx, hipStream_t s,
                          bool fp32_hidden, const WideNodes* wide, float* stats) {
    if (p.T == 0) return hipSuccess;
    SubtreeArgs a = make_args(p, p.depth - k, k, wide, stats, fp32_hidden);
    a.leaf_idx = leaf_idx;
    a.perm = perm;
    a.offset = offset;
    a.cols = a.node_cols + (p.L << k);
    const int64_t tiles = p.T / kTok + a.groups;             // at most: every group ends in a partly filled tile
    return wide ? dispatch_wide<true>(p, a, tiles, s) : dispatch<kLinear, true>(a, p.bf16, tiles, s);
}

hipError_t launch_subtree_levels(const Problem& p, int base_level, int k, const int32_t* perm, const int32_t* offset, int32_t* node_idx,
                                 hipStream_t s, const WideNodes& wide, float* stats, DescentCounts* dc) {
    if (p.T == 0) return hipSuccess;
    SubtreeArgs a = make_args(p, base_level, k, &wide, stats, false);
    a.leaf_idx = node_idx;
    a.perm = perm;
    a.offset = offset;
    a.cols = a.node_cols;
    const int64_t tiles = offset ? p.T / kTok + a.groups : (p.T + kTok - 1) / kTok;
    if (dc) {
        dc->blocks = 0;
        if (!offset && dc->M && bucket_fold_ok(k, (tiles + kFoldTiles - 1) / kFoldTiles, kTok * kFoldTiles) && (tiles << k) <= dc->capacity) {
            a.counts = dc->M;
            dc->blocks = (int)((tiles + kFoldTiles - 1) / kFoldTiles);
            dc->share = kTok * kFoldTiles;
            dc->rows = kFoldTiles;
            dc->n_rows = (int)tiles;
        }
    }
    return dispatch_wide<false>(p, a, tiles, s);
}

}  // namespace fff
