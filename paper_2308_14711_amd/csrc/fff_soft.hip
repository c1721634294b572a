// The soft forward pass of an FFF -- Forward_T of Algorithm 1: every node gives a choice score
// c = sigmoid(w . x + b), the leaves are mixed with the products of the scores along their paths
// (the stochastic vector over the leaves), out = sum_leaf mix[leaf] * Leaf_leaf(x).  This is the
// pass used in training and for the hardening diagnostics (batch mean entropy of the choice
// scores per node, paragraph "Hardening"); unlike Forward_I it is dense, so it runs on the matrix
// cores as three contractions over the shared 64 x 128 MFMA tile:
//
//   nodes   C[t][n]   = sigmoid(x[t] . node_w[n] + node_b[n])                       fp32, [T, 2^d - 1]
//   mix     M[t][l]   = prod over the path of leaf l of (bit ? c : 1 - c)           fp32, [T, 2^d]
//   hidden  H[t][k]   = act(x[t] . W1[k] + b1[k]) * M[t][k / l]   (k = leaf * l + neuron)   bf16
//           H[t][2^d l + leaf] = M[t][leaf]                          (carries the output bias)
//   out     out[t][o] = H[t] . W2x[o]   with W2x[o] = (W2[.][o], b2[.][o]): W2 and b2 transposed
//                                                                     once per call into [O, K2]
//
// so that the weighting by the mixture and the bias both ride inside the last contraction.
#include "fff_device.h"
#include "fff_internal.h"
#include "fff_mfma_tile.h"

namespace fff {
int64_t g_soft_small_tiles = 0;     // experiment switch: 1 = the 64 x 128 tile for every contraction (the 128-row nodes + mixture launch from 2048 rows on), 2 = the small-batch kernels
namespace {

struct SoftArgs {
    const uint16_t* x;
    const uint16_t* node_w;
    const uint16_t* node_b;
    const uint16_t* w1;
    const uint16_t* b1;
    const uint16_t* w2;
    const uint16_t* b2;
    float* choice;        // [T][NL]: NN scores per row, pitch NL so that rows start 16-byte aligned
    float* mix;           // [T][NL]
    uint16_t* hid;        // [T][K2]
    uint16_t* w2x;        // [O][K2]
    uint16_t* out;        // [T][O]
    int64_t T;
    int D, O, depth, L, act;
    int64_t NN, NL, K2;   // K2 = NL * (L + 1) rounded up to a multiple of 8
};

__device__ __forceinline__ int64_t tile_row0(int64_t n_col_blocks) { return (int64_t)(blockIdx.x / n_col_blocks) * kTileM; }
__device__ __forceinline__ int64_t tile_col0(int64_t n_col_blocks) { return (int64_t)(blockIdx.x % n_col_blocks) * kTileN; }

// nodes: choice scores
__global__ __launch_bounds__(256) void soft_nodes_kernel(const SoftArgs a) {
    __shared__ TileLds tile;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = lane & 15, kg = lane >> 4;
    const int64_t ncb = (a.NN + kTileN - 1) / kTileN;
    const int64_t t0 = tile_row0(ncb), n0 = tile_col0(ncb);
    f32x4_t acc[4][2];
    mfma_tile_64x128<2>(a.x, a.D, a.T, a.node_w, a.D, a.NN, a.D, t0, n0, tile, acc);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int64_t n = n0 + 32 * wv + 16 * nt + j;
        if (n >= a.NN) continue;
        const float b = bf16_to_f32(a.node_b[n]);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t t = t0 + 16 * mt + 4 * kg + q;
                if (t < a.T) a.choice[t * a.NL + n] = 1.0f / (1.0f + __expf(-(acc[mt][nt][q] + b)));
            }
    }
}

// entropy of a Bernoulli variable of parameter c, natural logarithm
__device__ __forceinline__ float bernoulli_entropy(float c) {
    const float h0 = c > 0.0f ? -c * __logf(c) : 0.0f;
    const float h1 = c < 1.0f ? -(1.0f - c) * __logf(1.0f - c) : 0.0f;
    return h0 + h1;
}

// mixture weights: one thread per (token, leaf); also the bias columns of the hidden matrix
__global__ __launch_bounds__(256) void soft_mix_kernel(const SoftArgs a) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.T * a.NL) return;
    const int64_t t = i / a.NL, leaf = i % a.NL;
    const float* c = a.choice + t * a.NL;
    float m = 1.0f;
    for (int lvl = 0; lvl < a.depth; ++lvl) {
        const int64_t pos = leaf >> (a.depth - lvl);                  // the path's node at this level
        const int bit = (int)((leaf >> (a.depth - 1 - lvl)) & 1);
        const float cs = c[(((int64_t)1 << lvl) - 1) + pos];
        m *= bit ? cs : 1.0f - cs;
    }
    a.mix[i] = m;
    a.hid[t * a.K2 + a.NL * a.L + leaf] = f32_to_bf16(m);
    // the padding columns up to K2 (fewer than 8) are cleared by the thread of leaf 0
    if (leaf == 0)
        for (int64_t k = a.NL * (a.L + 1); k < a.K2; ++k) a.hid[t * a.K2 + k] = 0;
}

// The same for trees of up to 2048 leaves, a wave per token: the products grow level by level in a
// wave-private LDS row (entry n of level m = entry n / 2 of level m - 1 times c or 1 - c of that
// node), so a token's scores are read once instead of once per leaf and level; the factors are
// multiplied in the same order as above (root first): same bits.  The scores themselves come in
// through registers, all of a token's loads in flight at once and the next token's requested before
// this token's levels are walked (a load inside the level loop is a trip to memory per iteration),
// and are parked in a third LDS row for the levels to index.  LDS: 3 NL floats per wave; blocks of
// four waves, or of two for 2048 leaves (48 KB either way at most).
constexpr int kMixMaxLeaves = 2048;
constexpr int kMixRegs = kMixMaxLeaves / kWave;          // scores a lane holds for one token
__global__ __launch_bounds__(256) void soft_mix_rows_kernel(const SoftArgs a) {
    extern __shared__ float mix_lds[];                       // per wave: the scores, then two rows of NL products
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int NL = (int)a.NL, NN = (int)a.NN;
    float* sc = mix_lds + (size_t)wv * 3 * NL;
    float* cur = sc + NL;
    float* nxt = cur + NL;
    const int per_lane = (NN + kWave - 1) / kWave;           // <= kMixRegs
    float creg[kMixRegs];
    const auto request = [&](int64_t t) {
        const float* c = a.choice + t * a.NL;
#pragma unroll
        for (int i = 0; i < kMixRegs; ++i)
            if (i < per_lane) creg[i] = lane + kWave * i < NN ? c[lane + kWave * i] : 0.0f;
    };
    const int64_t first = (int64_t)blockIdx.x * waves + wv, step = (int64_t)gridDim.x * waves;
    if (first < a.T) request(first);
    for (int64_t t = first; t < a.T; t += step) {
#pragma unroll
        for (int i = 0; i < kMixRegs; ++i)
            if (i < per_lane && lane + kWave * i < NN) sc[lane + kWave * i] = creg[i];
        if (t + step < a.T) request(t + step);               // travels while this token's levels are walked
        if (lane == 0) cur[0] = 1.0f;
        __builtin_amdgcn_wave_barrier();
        for (int lvl = 0; lvl < a.depth; ++lvl) {
            const int n_nodes = 1 << lvl;                    // nodes of this level; 2 n_nodes entries come out
            const float* cl = sc + (n_nodes - 1);
            for (int e = lane; e < 2 * n_nodes; e += kWave) {
                const float cs = cl[e >> 1];
                nxt[e] = cur[e >> 1] * ((e & 1) ? cs : 1.0f - cs);
            }
            __builtin_amdgcn_wave_barrier();                 // LDS executes a wave's accesses in order
            float* tmp = cur; cur = nxt; nxt = tmp;
        }
        for (int leaf = lane; leaf < NL; leaf += kWave) {
            const float m = cur[leaf];
            __builtin_nontemporal_store(m, a.mix + t * a.NL + leaf);
            __builtin_nontemporal_store(f32_to_bf16(m), a.hid + t * a.K2 + a.NL * a.L + leaf);
        }
        for (int64_t k = a.NL * (a.L + 1) + lane; k < a.K2; k += kWave) a.hid[t * a.K2 + k] = 0;
        __builtin_amdgcn_wave_barrier();
    }
}

// hidden: act(x . W1 + b1) scaled by the mixture weight of the neuron's leaf
__global__ __launch_bounds__(256) void soft_hidden_kernel(const SoftArgs a) {
    __shared__ TileLds tile;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = lane & 15;
    const int64_t NH = a.NL * a.L;
    const int64_t ncb = (NH + kTileN - 1) / kTileN;
    const int64_t t0 = tile_row0(ncb), n0 = tile_col0(ncb);
    f32x4_t acc[4][2];
    mfma_tile_64x128<2>(a.x, a.D, a.T, a.w1, a.D, NH, a.D, t0, n0, tile, acc);
    // the mixture weights this tile needs (64 tokens x the leaves of its 128 columns, at most 128)
    // go through the second tile buffer, read along a row of the weights
    float* mixt = (float*)tile.b;
    const int64_t last = n0 + kTileN - 1 < NH - 1 ? n0 + kTileN - 1 : NH - 1;
    const int64_t leaf_lo = n0 / a.L;
    const int n_leaf = (int)(last / a.L - leaf_lo + 1);
    for (int idx = threadIdx.x; idx < kTileM * n_leaf; idx += 256) {
        const int r = idx / n_leaf, c = idx % n_leaf;
        mixt[idx] = t0 + r < a.T ? a.mix[(t0 + r) * a.NL + leaf_lo + c] : 0.0f;
    }
    float bias[2];
    int lcol[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int64_t n = n0 + 32 * wv + 16 * nt + j;
        bias[nt] = n < NH ? bf16_to_f32(a.b1[n]) : 0.0f;
        lcol[nt] = n < NH ? (int)(n / a.L - leaf_lo) : 0;
    }
    __syncthreads();
    tile_store_bf16(tile, acc, a.hid, a.K2, a.T, NH, t0, n0, [&](int r, int c, float v) {
        const int nt = (c >> 4) & 1;
        return activate_bulk(v + bias[nt], a.act) * mixt[r * n_leaf + lcol[nt]];
    });
}

// The same two contractions over the 128 x 256 tile (batches and widths that fill it).
// Block -> tile so that the column tiles of one row tile run back to back on ONE XCD (blocks are
// dealt to the 8 XCDs round robin): the first of them brings the row tile's A rows into that
// XCD's L2, the others hit there instead of fetching them again from memory.  Row tile
// 8 (i / ncb) + xcd, column tile i % ncb for the i-th block of an XCD; the grid is rounded up to
// whole groups of 8 row tiles and blocks past the last row tile leave at once.
__device__ __forceinline__ bool big_tile_of_block(int64_t ncb, int64_t M, int64_t& m0, int64_t& n0) {
    const int64_t xcd = blockIdx.x & 7, i = blockIdx.x >> 3;
    m0 = (8 * (i / ncb) + xcd) * kBigM;
    n0 = (i % ncb) * kBigN;
    return m0 < M;
}
inline unsigned big_grid(int64_t M, int64_t ncb) {
    const int64_t row_tiles = (M + kBigM - 1) / kBigM;
    return (unsigned)(((row_tiles + 7) / 8) * 8 * ncb);
}

__global__ __launch_bounds__(256, 2) void soft_nodes_big_kernel(const SoftArgs a) {
    __shared__ BigTileLds tile;
    const int64_t ncb = (a.NN + kBigN - 1) / kBigN;
    int64_t t0, n0;
    if (!big_tile_of_block(ncb, a.T, t0, n0)) return;
    f32x4_t acc[4][8];
    mfma_tile_128x256(a.x, a.D, a.T, a.node_w, a.D, a.NN, a.D, t0, n0, tile, acc);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = lane & 15, kg = lane >> 4;
    const int wm = wv >> 1, wn = wv & 1;
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const int64_t n = n0 + 128 * wn + 16 * nt + 4 * kg;          // this lane's nodes n .. n + 3
        if (n >= a.NL) continue;                                     // (the row's last float, past the NN scores, is padding)
        float b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = n + q < a.NN ? bf16_to_f32(a.node_b[n + q]) : 0.0f;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int64_t t = t0 + 64 * wm + 16 * mt + j;
            if (t >= a.T) continue;
            float4 c;
            c.x = 1.0f / (1.0f + __expf(-(acc[mt][nt][0] + b[0])));
            c.y = 1.0f / (1.0f + __expf(-(acc[mt][nt][1] + b[1])));
            c.z = 1.0f / (1.0f + __expf(-(acc[mt][nt][2] + b[2])));
            c.w = 1.0f / (1.0f + __expf(-(acc[mt][nt][3] + b[3])));
            // NL >= 256 here: a multiple of 4, rows 16-byte aligned; read once by the mixture launch
            __builtin_nontemporal_store(f32x4_t{c.x, c.y, c.z, c.w}, (f32x4_t*)(a.choice + t * a.NL + n));
        }
    }
}

// Trees of up to 256 leaves (all nodes in one column tile): the node contraction, the mixture weights and
// the entropy sums in one launch -- the scores never go to memory.  After the contraction the tile's
// scores pass through LDS 64 rows at a time (column n of row r at 256 r + (n xor 4 (r mod 16)): a lane
// stores its four consecutive columns as 16 bytes, the 16 lanes of a group are 16 rows on equal
// columns, and the xor on the 16-byte piece index spreads them over the banks; the readers below run
// along a row).  Then a wave takes 16 of the rows and multiplies
// every leaf's path, root first (the factors and their order are those of soft_mix_kernel: same bits),
// writing the mixture weights and the bias columns of the hidden matrix; thread n adds the entropies
// of node n over the tile's rows in row order into part[row tile][n].
__device__ __forceinline__ int score_slot(int r, int n) { return 256 * r + (n ^ (4 * (r & 15))); }

// (kRows: rows of x per block; 16 is the version for batches that leave a chip of 128-row tiles idle)
template <int kRows> __global__ void soft_nodes_mix_kernel(const SoftArgs a, float* __restrict__ ent_part);
template <> __global__ __launch_bounds__(256, 2) void soft_nodes_mix_kernel<kBigM>(const SoftArgs a, float* __restrict__ ent_part) {
    __shared__ BigTileLds tile;
    int64_t t0, n0;
    if (!big_tile_of_block(1, a.T, t0, n0)) return;
    f32x4_t acc[4][8];
    mfma_tile_128x256(a.x, a.D, a.T, a.node_w, a.D, a.NN, a.D, t0, 0, tile, acc);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = lane & 15, kg = lane >> 4;
    const int wm = wv >> 1, wn = wv & 1;
    const int NL = (int)a.NL, NN = (int)a.NN;
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const int n = 128 * wn + 16 * nt + 4 * kg;                   // this lane's nodes n .. n + 3
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float b = n + q < NN ? bf16_to_f32(a.node_b[n + q]) : 0.0f;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[mt][nt][q] = 1.0f / (1.0f + __expf(-(acc[mt][nt][q] + b)));
        }
    }
    float* const S = (float*)&tile;                     // [64][256] scores of one half of the tile's rows
    const int per_log = NL >= 256 ? 2 : NL >= 128 ? 1 : 0;   // leaves per lane: 4, 2 or 1
    const bool mix_vec = (reinterpret_cast<uintptr_t>(a.mix) & 15u) == 0;
    // a lane takes `per` consecutive leaves (4 for 256 leaves): their paths share all but the last
    // log2(per) levels, so the shared factors are multiplied once, root first, and the product
    // then splits level by level -- every leaf still sees its factors in root-to-leaf order.  Four rows
    // at a time, every score of theirs requested before the first is used: one row after the other the
    // wave waits out an LDS read per level (a tile's epilogue took 40 us so, 128 rows over four waves).
    constexpr int kMixRows = 4, kMaxShared = 6;                        // (at most 256 leaves)
    const int shared = a.depth - per_log, first = lane << per_log;
    const int below = ((1 << shared) - 1) + lane;                      // the lane's node under the shared levels
    float ent = 0.0f;
    for (int h = 0; h < 2; ++h) {
        if (wm == h) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 8; ++nt)
                    *(f32x4_t*)(S + score_slot(16 * mt + j, 128 * wn + 16 * nt + 4 * kg)) = acc[mt][nt];
        }
        __syncthreads();
        for (int rr = 0; rr < 16 && t0 + 64 * h + 16 * wv + rr < a.T; rr += kMixRows) {
            float cs[kMaxShared][kMixRows], c1[kMixRows], c2[kMixRows], c3[kMixRows];
            const auto score = [&](int i, int n) { return S[score_slot(16 * wv + rr + i, n)]; };
            if (first >= NL) continue;
#pragma unroll
            for (int lvl = 0; lvl < kMaxShared; ++lvl) {
                const int l = lvl < shared ? lvl : 0, n = ((1 << l) - 1) + (first >> (a.depth - l));
#pragma unroll
                for (int i = 0; i < kMixRows; ++i) cs[lvl][i] = score(i, n);
            }
#pragma unroll
            for (int i = 0; i < kMixRows; ++i) {
                c1[i] = score(i, per_log > 0 ? below : 0);
                c2[i] = score(i, per_log > 1 ? 2 * below + 1 : 0);
                c3[i] = score(i, per_log > 1 ? 2 * below + 2 : 0);
            }
#pragma unroll
            for (int i = 0; i < kMixRows; ++i) {
                const int64_t t = t0 + 64 * h + 16 * wv + rr + i;
                if (t >= a.T) break;
                float m[4];
                m[0] = 1.0f;
#pragma unroll
                for (int lvl = 0; lvl < kMaxShared; ++lvl) {
                    const int l = lvl < shared ? lvl : 0;
                    const float f = (first >> (a.depth - 1 - l)) & 1 ? cs[lvl][i] : 1.0f - cs[lvl][i];
                    m[0] = lvl < shared ? m[0] * f : m[0];
                }
                float* mp = a.mix + t * a.NL + first;
                uint16_t* hp = a.hid + t * a.K2 + a.NL * a.L + first;
                if (per_log == 2) {
                    const float lo = m[0] * (1.0f - c1[i]), hi = m[0] * c1[i];
                    m[0] = lo * (1.0f - c2[i]); m[1] = lo * c2[i]; m[2] = hi * (1.0f - c3[i]); m[3] = hi * c3[i];
                    // one 16-byte store (a caller's mixture matrix may start anywhere: checked) and one 8-byte store
                    // (the hidden matrix is the library's, K2 a multiple of 8)
                    if (mix_vec) {
                        __builtin_nontemporal_store(f32x4_t{m[0], m[1], m[2], m[3]}, (f32x4_t*)mp);     // written once, read by a later launch
                    } else {
                        mp[0] = m[0]; mp[1] = m[1]; mp[2] = m[2]; mp[3] = m[3];
                    }
                    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
                    const u32x2_t packed = {pack_bf16x2(m[0], m[1]), pack_bf16x2(m[2], m[3])};
                    __builtin_nontemporal_store(packed, (u32x2_t*)hp);
                } else if (per_log == 1) {
                    m[1] = m[0] * c1[i]; m[0] = m[0] * (1.0f - c1[i]);
                    mp[0] = m[0]; mp[1] = m[1];
                    hp[0] = f32_to_bf16(m[0]); hp[1] = f32_to_bf16(m[1]);
                } else {
                    mp[0] = m[0];
                    hp[0] = f32_to_bf16(m[0]);
                }
                for (int64_t k = a.NL * (a.L + 1) + lane; k < a.K2; k += NL < kWave ? NL : kWave) a.hid[t * a.K2 + k] = 0;
            }
        }
        if (ent_part != nullptr && tid < NN) {
            for (int r0 = 0; r0 < 64; r0 += 8) {
                float c[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = S[score_slot(r0 + i, tid)];
#pragma unroll
                for (int i = 0; i < 8; ++i) ent += t0 + 64 * h + r0 + i < a.T ? bernoulli_entropy(c[i]) : 0.0f;
            }
        }
        __syncthreads();
    }
    if (ent_part != nullptr && tid < NN) ent_part[(t0 / kBigM) * a.NN + tid] = ent;
}

typedef uint32_t u32x2_any_t __attribute__((ext_vector_type(2), aligned(2)));       // (the memory system takes it at any address)
// GELU, ONE_LEAF: template parameters -- chosen per element at run time either puts a branch around
// every one of a lane's 128 evaluations, which then run one after the other, each behind its own trip for a
// mixture weight.  ONE_LEAF (leaf widths that are multiples of 4; biases at any element): a lane's four consecutive
// neurons belong to one leaf, and all 32 weights and 8 bias pieces of its tile are requested together (50432 tokens
// of 768, 256 leaves of 8, GELU: the call 485 -> 469 us, the same bits; biases at an odd element 462 -> 443).
template <bool GELU, bool ONE_LEAF>
__global__ __launch_bounds__(256, 2) void soft_hidden_big_kernel(const SoftArgs a) {
    __shared__ BigTileLds tile;
    const int64_t NH = a.NL * a.L;
    const int64_t ncb = (NH + kBigN - 1) / kBigN;
    int64_t t0, n0;
    if (!big_tile_of_block(ncb, a.T, t0, n0)) return;
    f32x4_t acc[4][8];
    mfma_tile_128x256(a.x, a.D, a.T, a.w1, a.D, NH, a.D, t0, n0, tile, acc);
    // bias, activation and the mixture weight of the neuron's leaf.  A lane holds four consecutive
    // neurons of a token per accumulator.
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, j = lane & 15, kg = lane >> 4;
    const int wm = wv >> 1, wn = wv & 1;
    const float* mrow[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        const int64_t t = t0 + 64 * wm + 16 * mt + j;
        mrow[mt] = a.mix + (t < a.T ? t : a.T - 1) * a.NL;
    }
    const bool bias_vec = (reinterpret_cast<uintptr_t>(a.b1) & 7u) == 0;
    const uint32_t L32 = (uint32_t)a.L, last = (uint32_t)(NH - 1);       // the width fits 32 bits (soft_shape_ok)
    if (ONE_LEAF) {
        float m[8][4];
        uint2 b[8];
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            const uint32_t n = (uint32_t)(n0 + 128 * wn + 16 * nt + 4 * kg), nc = n < last ? n : last - 3;     // (a multiple of 4)
            const uint32_t leaf = nc / L32;
            const u32x2_any_t bias = *(const u32x2_any_t*)(a.b1 + nc);
            b[nt] = make_uint2(bias.x, bias.y);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) m[nt][mt] = mrow[mt][leaf];
        }
        __builtin_amdgcn_sched_barrier(0);          // every load is requested before the first is waited for
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            const float bias[4] = {bf16_lo(b[nt].x), bf16_hi(b[nt].x), bf16_lo(b[nt].y), bf16_hi(b[nt].y)};
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                f32x4_t v;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = activate_bulk(acc[mt][nt][q] + bias[q], GELU ? 1 : 0) * m[nt][mt];
                big_tile_stage(tile, mt, nt, v);     // finished, packed and staged at once: nothing is held back
            }
        }
        big_tile_flush(tile, a.hid, a.K2, a.T, NH, t0, n0);
        return;
    }
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const uint32_t n = (uint32_t)(n0 + 128 * wn + 16 * nt + 4 * kg);   // this lane's neurons n .. n + 3
        // columns past the last neuron are dropped by the store: their look-ups are clamped, not skipped
        const uint32_t nc = n < last ? n : last;
        float bias[4];
        if (bias_vec && n + 3 <= last) {
            const uint2 b = *(const uint2*)(a.b1 + n);
            bias[0] = bf16_to_f32((uint16_t)b.x); bias[1] = bf16_to_f32((uint16_t)(b.x >> 16));
            bias[2] = bf16_to_f32((uint16_t)b.y); bias[3] = bf16_to_f32((uint16_t)(b.y >> 16));
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) bias[q] = bf16_to_f32(a.b1[nc + q < last ? nc + q : last]);
        }
        // one division per group of four: the leaf of neuron n + q is that of n plus the number of leaf
        // boundaries crossed, at most three (q <= 3)
        const uint32_t leaf0 = nc / L32, rem = nc - leaf0 * L32;
        uint32_t leaf[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t o = rem + q;
            uint32_t lf = leaf0 + (o >= L32) + (o >= 2 * L32) + (o >= 3 * L32);
            leaf[q] = lf < (uint32_t)a.NL ? lf : (uint32_t)a.NL - 1;
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            float m[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) m[q] = mrow[mt][leaf[q]];
            f32x4_t v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = activate_bulk(acc[mt][nt][q] + bias[q], GELU ? 1 : 0) * m[q];
            big_tile_stage(tile, mt, nt, v);
        }
    }
    big_tile_flush(tile, a.hid, a.K2, a.T, NH, t0, n0);
}

__global__ __launch_bounds__(256, 2) void soft_out_big_kernel(const SoftArgs a) {
    __shared__ BigTileLds tile;
    const int64_t ncb = ((int64_t)a.O + kBigN - 1) / kBigN;
    int64_t t0, n0;
    if (!big_tile_of_block(ncb, a.T, t0, n0)) return;
    f32x4_t acc[4][8];
    mfma_tile_128x256(a.hid, a.K2, a.T, a.w2x, a.K2, a.O, (int)a.K2, t0, n0, tile, acc);
    big_tile_store_bf16(tile, acc, a.out, a.O, a.T, a.O, t0, n0);
}

// W2x[o][k] = W2[k][o] for k < NL * L, b2[k - NL * L][o] for the next NL, zeros up to K2.
// A 32 x 32 tile through LDS: reads run along o, writes along k.
__global__ __launch_bounds__(256) void soft_w2x_kernel(const SoftArgs a) {
    __shared__ uint16_t t32[32][33];
    const int64_t kb = (a.K2 + 31) / 32;
    const int64_t k0 = (int64_t)(blockIdx.x % kb) * 32, o0 = (int64_t)(blockIdx.x / kb) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // 32 x 8
    const int64_t NH = a.NL * a.L;
    for (int r = ty; r < 32; r += 8) {
        const int64_t k = k0 + r, o = o0 + tx;
        uint16_t v = 0;
        if (o < a.O) {
            if (k < NH) v = a.w2[k * a.O + o];
            else if (k < NH + a.NL) v = a.b2[(k - NH) * a.O + o];
        }
        t32[r][tx] = v;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int64_t o = o0 + r, k = k0 + tx;
        if (o < a.O && k < a.K2) a.w2x[o * a.K2 + k] = t32[tx][r];
    }
}

// out: the weighted leaf outputs and biases in one contraction over K2
__global__ __launch_bounds__(256) void soft_out_kernel(const SoftArgs a) {
    __shared__ TileLds tile;
    const int64_t ncb = ((int64_t)a.O + kTileN - 1) / kTileN;
    const int64_t t0 = tile_row0(ncb), n0 = tile_col0(ncb);
    f32x4_t acc[4][2];
    mfma_tile_64x128<2>(a.hid, a.K2, a.T, a.w2x, a.K2, a.O, (int)a.K2, t0, n0, tile, acc);
    tile_store_bf16(tile, acc, a.out, a.O, a.T, a.O, t0, n0, [](int, int, float v) { return v; });
}

// batch mean of the Bernoulli entropy of every node's choice score, in two passes with a fixed
// order of additions (so the result does not depend on scheduling): a block sums kEntTokens
// tokens for every node (thread = node, so the reads run along a row of scores), then one block
// per node adds the partial sums (strided over its threads, then a fixed tree).
constexpr int kEntTokens = 32, kEntPartTokens = 16;     // (tokens of the smallest partial sum of any launch)

__global__ __launch_bounds__(256) void soft_entropy_part_kernel(const float* __restrict__ choice, int64_t T, int64_t NN,
                                                                int64_t pitch, float* __restrict__ part) {
    const int64_t t0 = (int64_t)blockIdx.x * kEntTokens;
    for (int64_t n = threadIdx.x; n < NN; n += 256) {
        float c[kEntTokens], s = 0.0f;
#pragma unroll
        for (int r = 0; r < kEntTokens; ++r) c[r] = choice[(t0 + r < T ? t0 + r : T - 1) * pitch + n];   // all in flight at once
#pragma unroll
        for (int r = 0; r < kEntTokens; ++r) s += t0 + r < T ? bernoulli_entropy(c[r]) : 0.0f;
        part[(int64_t)blockIdx.x * NN + n] = s;
    }
}

__global__ __launch_bounds__(256) void soft_entropy_sum_kernel(const float* __restrict__ part, int64_t n_parts, int64_t T,
                                                               int64_t NN, float* __restrict__ entropy) {
    __shared__ float red[256];
    const int64_t n = blockIdx.x;       // one block per node: strided partial sums, then a fixed tree
    float s = 0.0f;
    for (int64_t b = threadIdx.x; b < n_parts; b += 256) s += part[b * NN + n];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) entropy[n] = red[0] / (float)T;
}

// ---- small batches ---------------------------------------------------------------------------------
//
// The same pass in three launches for batches that cannot fill the chip with tiles: every block's
// waves split K among them (mfma_wave_slice), a hidden block multiplies the mixture weights of its own
// leaves out of the scores, W2 is read where it stands instead of being transposed first, and the
// entropies' sums ride in the second and third launch.  As tiles these batches took five to seven
// launches, each a chain of K / 64 memory round trips.
//
// What bounds a block is how much one compute unit can have in flight (about 80 lines of 128 bytes:
// 10-15 bytes a clock for rows that come from beyond the L2), so tiles shrink until the grid covers the
// chip: 32 x 64, else 16 x 32, else 16 x 16 (64 tokens, K = 3504, 256 columns: 18 us with 32 x 64).
constexpr int kSmallMaxDepth = 9;
struct SmallTile {
    int64_t t0, n0;
};
template <int MT, int NT> __device__ __forceinline__ SmallTile small_tile(int64_t N) {
    const int64_t ncb = (N + 16 * NT - 1) / (16 * NT);
    return SmallTile{(int64_t)(blockIdx.x / ncb) * (16 * MT), (int64_t)(blockIdx.x % ncb) * (16 * NT)};
}
// The block's tile of A B^T: wave w (of the first MT NT) returns, summed over the eight slices in
// order, tile (w / NT, w % NT) with the lane layout of mfma_wave_slice.
template <int MT, int NT>
__device__ __forceinline__ f32x4_t small_contract(const uint16_t* A, int64_t M, const uint16_t* B, int64_t N, int K,
                                                  const SmallTile& at, f32x4_t (&part)[8][MT * NT][kWave]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int k_begin, k_end;
    k_slice(K, 8, wv, &k_begin, &k_end);
    f32x4_t acc[MT][NT];
    mfma_wave_slice<MT, NT, MT * NT == 8 ? 3 : 6>(A, K, M, at.t0, B, K, N, at.n0, k_begin, k_end, acc);
#pragma unroll
    for (int i = 0; i < MT * NT; ++i) part[wv][i][lane] = acc[i / NT][i % NT];
    __syncthreads();
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (wv < MT * NT) {
        v = part[0][wv][lane];
#pragma unroll
        for (int s = 1; s < 8; ++s) v += part[s][wv][lane];
    }
    return v;
}

// nodes: choice scores
template <int MT, int NT>
__global__ __launch_bounds__(512) void soft_small_nodes_kernel(const SoftArgs a) {
    __shared__ f32x4_t part[8][MT * NT][kWave];
    const SmallTile at = small_tile<MT, NT>(a.NN);
    const f32x4_t v = small_contract<MT, NT>(a.x, a.T, a.node_w, a.NN, a.D, at, part);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t t = at.t0 + 16 * (wv / NT) + (lane & 15), n = at.n0 + 16 * (wv % NT) + 4 * (lane >> 4);
    if (wv >= MT * NT || t >= a.T) return;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (n + q < a.NN) a.choice[t * a.NL + n + q] = 1.0f / (1.0f + __expf(-(v[q] + bf16_to_f32(a.node_b[n + q]))));
}

// weight of a leaf from a row of scores, root first
__device__ __forceinline__ float leaf_weight(const float* __restrict__ c, int depth, int leaf) {
    float cs[kSmallMaxDepth];
#pragma unroll
    for (int lvl = 0; lvl < kSmallMaxDepth; ++lvl) {          // all requested before the first is used
        const int l = lvl < depth ? lvl : 0;
        cs[lvl] = c[((1 << l) - 1) + (leaf >> (depth - l))];
    }
    float m = 1.0f;
#pragma unroll
    for (int lvl = 0; lvl < kSmallMaxDepth; ++lvl)
        if (lvl < depth) m *= (leaf >> (depth - 1 - lvl)) & 1 ? cs[lvl] : 1.0f - cs[lvl];
    return m;
}

// hidden, and the mixture weights of the leaves whose first neuron is in the block's columns; the
// blocks past the tiles' leave partial entropy sums of 16 tokens each
// (kOwn false: an earlier launch has left the weights in a.mix and the sums where they belong)
template <int MT, int NT, bool kOwn>
__global__ __launch_bounds__(512) void soft_small_hidden_kernel(const SoftArgs a, int64_t tile_blocks, float* __restrict__ mix_out,
                                                                float* __restrict__ ent_part) {
    __shared__ f32x4_t part[8][MT * NT][kWave];
    __shared__ float weight[16 * MT * 16 * NT];               // [token][leaf of the tile's columns]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (kOwn && blockIdx.x >= tile_blocks) {
        const int64_t b = blockIdx.x - tile_blocks, t0 = 16 * b;
        for (int64_t n = tid; n < a.NN; n += 512) {
            float c[16], s = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) c[r] = a.choice[(t0 + r < a.T ? t0 + r : a.T - 1) * a.NL + n];
#pragma unroll
            for (int r = 0; r < 16; ++r) s += t0 + r < a.T ? bernoulli_entropy(c[r]) : 0.0f;
            ent_part[b * a.NN + n] = s;
        }
        return;
    }
    const int NH = (int)(a.NL * a.L);
    const SmallTile at = small_tile<MT, NT>(NH);
    const int n0 = (int)at.n0, last = n0 + 16 * NT < NH ? n0 + 16 * NT - 1 : NH - 1;
    const int leaf_lo = n0 / a.L, n_leaf = last / a.L - leaf_lo + 1;      // at most 16 NT leaves
    for (int i = tid; i < 16 * MT * n_leaf; i += 512) {
        const int r = i / n_leaf, leaf = leaf_lo + i % n_leaf;
        const int64_t t = at.t0 + r;
        if (t >= a.T) continue;
        const float m = kOwn ? leaf_weight(a.choice + t * a.NL, a.depth, leaf) : a.mix[t * a.NL + leaf];
        weight[i] = m;
        if (kOwn && leaf * a.L >= n0) {
            if (mix_out) mix_out[t * a.NL + leaf] = m;
            a.hid[t * a.K2 + NH + leaf] = f32_to_bf16(m);
            if (leaf == 0)
                for (int64_t k = NH + a.NL; k < a.K2; ++k) a.hid[t * a.K2 + k] = 0;
        }
    }
    const f32x4_t v = small_contract<MT, NT>(a.x, a.T, a.w1, NH, a.D, at, part);   // (its barrier covers weight[] too)
    const int r = 16 * (wv / NT) + (lane & 15), n = n0 + 16 * (wv % NT) + 4 * (lane >> 4);
    const int64_t t = at.t0 + r;
    if (wv >= MT * NT || t >= a.T || n >= NH) return;
    uint16_t h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t nq = (uint32_t)(n + q < NH ? n + q : NH - 1);
        h[q] = f32_to_bf16(activate_bulk(v[q] + bf16_to_f32(a.b1[nq]), a.act) * weight[r * n_leaf + (int)(nq / (uint32_t)a.L) - leaf_lo]);
    }
    uint16_t* dst = a.hid + t * a.K2 + n;
    if (n + 4 <= NH) {
        *(uint2*)dst = make_uint2(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16);
    } else {
        for (int q = 0; n + q < NH; ++q) dst[q] = h[q];
    }
}

// nodes + mixture weights + partial entropy sums: 16 tokens against all nodes (up to 255).  16 waves:
// 64 nodes a wave, the rest of them splitting K; then a wave per token multiplies the paths.
constexpr size_t kSmallPartBytes = 16 * 4 * kWave * sizeof(f32x4_t);
__host__ __device__ inline int small_node_groups(int64_t NN) { return NN <= 64 ? 1 : NN <= 128 ? 2 : 4; }
inline size_t small_nodes_lds(int64_t NN) { return kSmallPartBytes + 16 * (64 * small_node_groups(NN) + 4) * sizeof(float); }

template <> __global__ __launch_bounds__(1024) void soft_nodes_mix_kernel<16>(const SoftArgs a, float* __restrict__ ent_part) {
    extern __shared__ f32x4_t small_lds[];
    f32x4_t* const part = small_lds;                                   // [wave][4][64]
    float* const S = (float*)(small_lds + 16 * 4 * kWave);             // [16][pitch] scores
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int NN = (int)a.NN, NL = (int)a.NL;
    const int groups = small_node_groups(NN), ks = 16 / groups, pitch = 64 * groups + 4;
    const int64_t t0 = (int64_t)blockIdx.x * 16;
    {
        int k_begin, k_end;
        k_slice(a.D, ks, wv % ks, &k_begin, &k_end);
        f32x4_t acc[1][4];
        mfma_wave_slice<1, 4, 4>(a.x, a.D, a.T, t0, a.node_w, a.D, NN, 64 * (wv / ks), k_begin, k_end, acc);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) part[(wv * 4 + nt) * kWave + lane] = acc[0][nt];
    }
    __syncthreads();
    for (int e = tid; e < groups * 256; e += 1024) {
        const int cg = e >> 8, at = e & 255, l = at & 63;
        f32x4_t v = part[cg * ks * 256 + at];
        for (int s = 1; s < ks; ++s) v += part[(cg * ks + s) * 256 + at];
        const int n = 64 * cg + 16 * (at >> 6) + 4 * (l >> 4);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = 1.0f / (1.0f + __expf(-(v[q] + (n + q < NN ? bf16_to_f32(a.node_b[n + q]) : 0.0f))));
        *(f32x4_t*)(S + (l & 15) * pitch + n) = v;
    }
    __syncthreads();
    const int64_t t = t0 + wv;
    if (t < a.T) {
        const float* c = S + wv * pitch;
        uint16_t* hrow = a.hid + t * a.K2 + a.NL * a.L;
        for (int leaf = lane; leaf < NL; leaf += kWave) {
            float m = 1.0f;
            for (int lvl = 0; lvl < a.depth; ++lvl) {
                const float cs = c[((1 << lvl) - 1) + (leaf >> (a.depth - lvl))];
                m *= (leaf >> (a.depth - 1 - lvl)) & 1 ? cs : 1.0f - cs;
            }
            a.mix[t * a.NL + leaf] = m;
            hrow[leaf] = f32_to_bf16(m);
        }
        for (int k = NL + lane; k < (int)(a.K2 - a.NL * a.L); k += kWave) hrow[k] = 0;
    }
    if (ent_part != nullptr && tid < NN) {
        float ent = 0.0f;
        for (int r = 0; r < 16 && t0 + r < a.T; ++r) ent += bernoulli_entropy(S[r * pitch + tid]);
        ent_part[(int64_t)blockIdx.x * NN + tid] = ent;
    }
}

// Element c of eight rows of bf16 values (`words` 32-bit words of each) as one MFMA operand piece.
template <int kWords>
__device__ __forceinline__ uint4 transpose_piece(const uint32_t (&r)[8][kWords], int c) {
    const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
    const int w = c >> 1;
    return make_uint4(__builtin_amdgcn_perm(r[1][w], r[0][w], sel), __builtin_amdgcn_perm(r[3][w], r[2][w], sel),
                      __builtin_amdgcn_perm(r[5][w], r[4][w], sel), __builtin_amdgcn_perm(r[7][w], r[6][w], sel));
}

// out: 16 MT tokens x 16 C outputs a block, eight slices of K2.  W2 and b2 rows run along the outputs
// while the instruction wants K contiguous: a lane loads outputs C j .. C j + C - 1 of its eight K
// rows and turns them around in registers, so that column j of the c-th instruction stands for output
// o0 + C j + c.  The blocks past the outputs' add up the entropies, a wave per node.
template <int MT, int C>
__global__ __launch_bounds__(512) void soft_small_out_kernel(const SoftArgs a, int64_t out_blocks,
                                                             const float* __restrict__ ent_part, int64_t n_parts,
                                                             float* __restrict__ entropy) {
    extern __shared__ f32x4_t small_lds[];                    // [8][MT C][64]
    constexpr int kWords = C / 2;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = lane & 15, kg = lane >> 4;
    if (blockIdx.x >= out_blocks) {
        const int64_t n = (blockIdx.x - out_blocks) * 8 + wv;
        if (n >= a.NN) return;
        float s = 0.0f;
        for (int64_t b = lane; b < n_parts; b += kWave) s += ent_part[b * a.NN + n];
        s = wave_sum(s);
        if (lane == 0) entropy[n] = s / (float)a.T;
        return;
    }
    const SmallTile at = small_tile<MT, C>(a.O);
    const int64_t t0 = at.t0, o0 = at.n0;
    const bool vec = a.O % C == 0 && ((reinterpret_cast<uintptr_t>(a.w2) | reinterpret_cast<uintptr_t>(a.b2) |
                                       reinterpret_cast<uintptr_t>(a.out)) & (2 * C - 1)) == 0;
    const int NH = (int)(a.NL * a.L), NB = NH + (int)a.NL;       // rows of W2, rows of W2 and b2
    int k_begin, k_end;
    k_slice((int)a.K2, 8, wv, &k_begin, &k_end);
    f32x4_t acc[MT][C];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[mt][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const uint16_t* ph[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int64_t t = t0 + 16 * mt + j;
        ph[mt] = a.hid + (t < a.T ? t : a.T - 1) * a.K2;
    }
    const int64_t o = o0 + C * j;
    const int64_t oc = o + C <= a.O ? o : (vec ? a.O - C : 0);   // results past the last output are dropped
    constexpr int kUnroll = C == 8 ? 2 : 4;
    for (int k0 = k_begin; k0 < k_end; k0 += 32 * kUnroll) {
        uint4 qa[kUnroll][MT];
        uint32_t qw[kUnroll][8][kWords];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + 32 * u + 8 * kg, kc = k < k_end ? k : k_begin;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) qa[u][mt] = *(const uint4*)(ph[mt] + kc);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = kc + i < NB ? kc + i : NB - 1;
                const uint16_t* w = row < NH ? a.w2 + (int64_t)row * a.O : a.b2 + (int64_t)(row - NH) * a.O;
                if (vec && C == 8) {
                    const uint4 v = *(const uint4*)(w + oc);
                    qw[u][i][0] = v.x; qw[u][i][1] = v.y; qw[u][i][2 % kWords] = v.z; qw[u][i][3 % kWords] = v.w;
                } else if (vec) {
                    const uint2 v = *(const uint2*)(w + oc);
                    qw[u][i][0] = v.x; qw[u][i][1] = v.y;
                } else {
#pragma unroll
                    for (int c = 0; c < kWords; ++c)
                        qw[u][i][c] = w[o + 2 * c < a.O ? o + 2 * c : a.O - 1] |
                                      (uint32_t)w[o + 2 * c + 1 < a.O ? o + 2 * c + 1 : a.O - 1] << 16;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + 32 * u + 8 * kg;
            const bool in = k < k_end;
            bf16x8_t fa[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) fa[mt] = __builtin_bit_cast(bf16x8_t, keep_if(in, qa[u][mt]));
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int w = 0; w < kWords; ++w) qw[u][i][w] = in && k + i < NB ? qw[u][i][w] : 0u;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, transpose_piece<kWords>(qw[u], c));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa[mt], acc[mt][c], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MT * C; ++i) small_lds[(wv * MT * C + i) * kWave + lane] = acc[i / C][i % C];
    __syncthreads();
    // thread (mt, lane, q): C consecutive outputs o0 + C (4 kg + q) + c of token 16 mt + j
    if (tid >= MT * 256) return;
    const float* const pf = (const float*)small_lds;
    const int mt = tid >> 8, l = (tid >> 2) & 63, q = tid & 3;
    float y[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        y[c] = 0.0f;
#pragma unroll
        for (int s = 0; s < 8; ++s) y[c] += pf[((s * MT * C + mt * C + c) * kWave + l) * 4 + q];
    }
    const int64_t t = t0 + 16 * mt + (l & 15), oy = o0 + C * (4 * (l >> 4) + q);
    if (t >= a.T || oy >= a.O) return;
    uint16_t* dst = a.out + t * a.O + oy;
    if (vec) {
        uint32_t w[kWords];
#pragma unroll
        for (int c = 0; c < kWords; ++c) w[c] = pack_bf16x2(y[2 * c], y[2 * c + 1]);
        if (C == 8) *(uint4*)dst = make_uint4(w[0], w[1], w[2 % kWords], w[3 % kWords]);
        else *(uint2*)dst = make_uint2(w[0], w[1]);
    } else {
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (oy + c < a.O) dst[c] = f32_to_bf16(y[c]);
    }
}

double small_out_cost(int64_t T, int64_t O, double K) { return 4 + (double)((small_blocks(T, O, 2, 8) + 255) / 256) * (3 + 0.006 * K); }
double big_cost(int64_t T, int64_t N, double K) {
    const int64_t blocks = (T + kBigM - 1) / kBigM * ((N + kBigN - 1) / kBigN);
    return (16 + 0.017 * K) * (blocks <= 256 ? 1.0 : 1.5 * (double)((blocks + 511) / 512));
}
constexpr double kLaunchCost = 3;          // a launch of its own: host time, ramp and drain

}  // namespace

// bf16, D a multiple of 8, 16-byte aligned rows of x, node_w, leaf_w1
bool soft_shape_ok(const Problem& p) {
    return p.bf16 && vec_ok(p.x, p.D, true) && (p.depth == 0 || vec_ok(p.node_w, p.D, true)) &&
           vec_ok(p.leaf_w1, p.D, true) && p.D < (1 << 30) && p.O < (1 << 30) &&
           (((int64_t)p.L + 1) << p.depth) < ((int64_t)1 << 30);        // the hidden matrix's width fits 32 bits
}

static int64_t soft_k2(const Problem& p) {
    const int64_t NL = (int64_t)1 << p.depth;
    return (NL * (p.L + 1) + 7) / 8 * 8;
}

// 32-bit words of scratch: choice scores, mixture weights, hidden matrix, transposed output weights
int64_t soft_scratch_words(const Problem& p) {
    const int64_t NL = (int64_t)1 << p.depth, NN = NL - 1, K2 = soft_k2(p);
    auto up = [](int64_t w) { return (w + 63) / 64 * 64; };
    return up(p.T * NL) + up(p.T * NL) + up((p.T * K2 + 1) / 2) + up((p.O * K2 + 1) / 2) +
           up((p.T + kEntPartTokens - 1) / kEntPartTokens * (NN > 0 ? NN : 1));
}

// mix (optional, [T, 2^d] fp32) and entropy (optional, [2^d - 1] fp32) are caller buffers
hipError_t launch_forward_soft(const Problem& p, int32_t* scratch, float* mix_out, float* entropy_out,
                               hipStream_t s) {
    if (p.T == 0) return hipSuccess;
    auto up = [](int64_t w) { return (w + 63) / 64 * 64; };
    SoftArgs a;
    a.NL = (int64_t)1 << p.depth;
    a.NN = a.NL - 1;
    a.K2 = soft_k2(p);
    a.x = (const uint16_t*)p.x;
    a.node_w = (const uint16_t*)p.node_w;
    a.node_b = (const uint16_t*)p.node_b;
    a.w1 = (const uint16_t*)p.leaf_w1;
    a.b1 = (const uint16_t*)p.leaf_b1;
    a.w2 = (const uint16_t*)p.leaf_w2;
    a.b2 = (const uint16_t*)p.leaf_b2;
    a.out = (uint16_t*)p.out;
    a.T = p.T;
    a.D = (int)p.D;
    a.O = (int)p.O;
    a.depth = p.depth;
    a.L = p.L;
    a.act = p.act;
    int32_t* w = scratch;
    a.choice = (float*)w;
    w += up(p.T * a.NL);
    a.mix = mix_out ? mix_out : (float*)w;
    w += up(p.T * a.NL);
    a.hid = (uint16_t*)w;
    w += up((p.T * a.K2 + 1) / 2);
    a.w2x = (uint16_t*)w;
    w += up((p.O * a.K2 + 1) / 2);
    float* ent_part = (float*)w;
    const DeviceInfo di = device_info();
    hipError_t e;
    const bool want_entropy = entropy_out && a.NN > 0;
    const int64_t NH = a.NL * a.L, K2 = a.K2;
    const auto grid = [](int64_t blocks) { return dim3((unsigned)blocks); };

    // ---- which kernel makes each contraction.  The 128 x 256 tile where batch and width fill it, the
    // 64 x 128 tile in between, slices of K over a block's waves where tiles leave the chip idle.
    enum Kind { kSmall, kTile, kBig };
    // (a small block is 512 threads on 32 rows, and a launch ends at 2^32 threads: narrow contractions would ask for more)
    const bool small_ok = p.T < ((int64_t)1 << 27);
    const auto pick = [&](double small, double tile, double big, bool big_ok) {
        if (g_soft_small_tiles == 1) return kTile;
        if (g_soft_small_tiles == 2 && small_ok) return kSmall;
        if (small_ok && small <= tile && (small <= big || !big_ok)) return kSmall;
        return big_ok && big < tile ? kBig : kTile;
    };
    const bool big_rows = p.T >= 16 * kBigM;
    // up to 2047 tokens the scores go to memory and a small hidden launch multiplies its own mixture
    // weights; from there on, up to 255 nodes, one launch makes scores, weights and entropy sums
    const bool own_ok = a.NN >= 1 && a.depth <= kSmallMaxDepth && !big_rows && g_soft_small_tiles != 1;
    const bool fused_nodes = big_rows && a.NN >= 1 && a.NN < kBigN;
    const Kind hidden = pick(small_cost(p.T, NH, a.D, own_ok),
                             tile_cost(p.T, NH, a.D) + (own_ok ? 2 * kLaunchCost : 0),
                             big_cost(p.T, NH, a.D), big_rows && NH >= kBigN);
    const Kind out = pick(small_out_cost(p.T, p.O, K2), tile_cost(p.T, p.O, K2) + kLaunchCost, big_cost(p.T, p.O, K2) + kLaunchCost,
                          big_rows && p.O >= kBigN);
    const bool own_weights = own_ok && hidden == kSmall;
    const int groups = small_node_groups(a.NN);
    const double fused16_cost = (double)((p.T + 4095) / 4096) * (7 + 0.0019 * a.D + (groups - 1) * (2 + 0.0025 * a.D));
    const bool rows16 = fused_nodes && g_soft_small_tiles != 1 && (g_soft_small_tiles == 2 || fused16_cost < 8 + big_cost(p.T, 1, a.D));

    // ---- nodes, mixture weights, entropy sums
    int64_t ent_parts = 0;                   // rows of partial sums somebody has left in ent_part
    if (fused_nodes && rows16) {
        static bool raised[64];              // the limit on dynamic LDS, once per device
        if (!raised[di.dev]) {
            e = hipFuncSetAttribute((const void*)soft_nodes_mix_kernel<16>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)small_nodes_lds(kBigN - 1));
            if (e != hipSuccess) return e;
            raised[di.dev] = true;
        }
        note_launch("soft_nodes_mix_kernel<16>");
        ent_parts = (p.T + 15) / 16;
        soft_nodes_mix_kernel<16><<<grid(ent_parts), dim3(1024), small_nodes_lds(a.NN), s>>>(a, want_entropy ? ent_part : nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (fused_nodes) {
        note_launch("soft_nodes_mix_kernel<128>");
        ent_parts = (p.T + kBigM - 1) / kBigM;
        soft_nodes_mix_kernel<kBigM><<<dim3(big_grid(p.T, 1)), dim3(256), 0, s>>>(a, want_entropy ? ent_part : nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (a.NN > 0) {
        const Kind nodes = pick(a.depth <= kSmallMaxDepth ? small_cost(p.T, a.NN, a.D, false) : 1e30, tile_cost(p.T, a.NN, a.D),
                                big_cost(p.T, a.NN, a.D), big_rows && a.NN >= kBigN - 1);
        constexpr int64_t enough = kSmallEnoughBlocks;
        if (nodes == kBig) {
            note_launch("soft_nodes_big_kernel");
            soft_nodes_big_kernel<<<dim3(big_grid(p.T, (a.NN + kBigN - 1) / kBigN)), dim3(256), 0, s>>>(a);
        } else if (nodes == kTile) {
            note_launch("soft_nodes_kernel");
            soft_nodes_kernel<<<grid((p.T + kTileM - 1) / kTileM * ((a.NN + kTileN - 1) / kTileN)), dim3(256), 0, s>>>(a);
        } else {
            note_launch("soft_small_nodes_kernel");
            if (small_blocks(p.T, a.NN, 2, 4) >= enough)
                soft_small_nodes_kernel<2, 4><<<grid(small_blocks(p.T, a.NN, 2, 4)), dim3(512), 0, s>>>(a);
            else if (small_blocks(p.T, a.NN, 1, 2) >= enough)
                soft_small_nodes_kernel<1, 2><<<grid(small_blocks(p.T, a.NN, 1, 2)), dim3(512), 0, s>>>(a);
            else
                soft_small_nodes_kernel<1, 1><<<grid(small_blocks(p.T, a.NN, 1, 1)), dim3(512), 0, s>>>(a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (!fused_nodes && !own_weights) {
        if (a.NL <= kMixMaxLeaves) {
            note_launch("soft_mix_rows_kernel");
            const int waves = a.NL > 1024 ? 2 : 4;
            int64_t blocks = (p.T + waves - 1) / waves;
            const int64_t cap = (int64_t)di.cus * 8;
            if (blocks > cap) blocks = cap;
            const size_t lds_bytes = sizeof(float) * 3 * waves * (size_t)a.NL;      // at most 48 KB
            soft_mix_rows_kernel<<<dim3((unsigned)blocks), dim3(64 * waves), lds_bytes, s>>>(a);
        } else {
            note_launch("soft_mix_kernel");
            soft_mix_kernel<<<dim3((unsigned)((p.T * a.NL + 255) / 256)), dim3(256), 0, s>>>(a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (want_entropy) {
            note_launch("soft_entropy_part_kernel");
            ent_parts = (p.T + kEntTokens - 1) / kEntTokens;
            soft_entropy_part_kernel<<<grid(ent_parts), dim3(256), 0, s>>>(a.choice, p.T, a.NN, a.NL, ent_part);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }

    // ---- hidden
    if (hidden == kBig) {
        note_launch("soft_hidden_big_kernel");
        const dim3 g(big_grid(p.T, (NH + kBigN - 1) / kBigN));
        const bool one_leaf = a.L % 4 == 0;
        const auto launch = [&](auto kern) { kern<<<g, dim3(256), 0, s>>>(a); };
        if (a.act != 0) one_leaf ? launch(soft_hidden_big_kernel<true, true>) : launch(soft_hidden_big_kernel<true, false>);
        else one_leaf ? launch(soft_hidden_big_kernel<false, true>) : launch(soft_hidden_big_kernel<false, false>);
    } else if (hidden == kTile) {
        note_launch("soft_hidden_kernel");
        soft_hidden_kernel<<<grid((p.T + kTileM - 1) / kTileM * ((NH + kTileN - 1) / kTileN)), dim3(256), 0, s>>>(a);
    } else {
        note_launch("soft_small_hidden_kernel");
        const int64_t enough = kSmallEnoughBlocks, parts = own_weights && want_entropy ? (p.T + 15) / 16 : 0;
        if (parts) ent_parts = parts;
        const auto launch = [&](auto own_kern, auto given_kern, int mt, int nt) {
            const int64_t blocks = small_blocks(p.T, NH, mt, nt);
            if (own_weights) own_kern<<<grid(blocks + parts), dim3(512), 0, s>>>(a, blocks, mix_out, ent_part);
            else given_kern<<<grid(blocks), dim3(512), 0, s>>>(a, blocks, nullptr, nullptr);
        };
        if (small_blocks(p.T, NH, 2, 4) >= enough) launch(soft_small_hidden_kernel<2, 4, true>, soft_small_hidden_kernel<2, 4, false>, 2, 4);
        else if (small_blocks(p.T, NH, 1, 2) >= enough) launch(soft_small_hidden_kernel<1, 2, true>, soft_small_hidden_kernel<1, 2, false>, 1, 2);
        else launch(soft_small_hidden_kernel<1, 1, true>, soft_small_hidden_kernel<1, 1, false>, 1, 1);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;

    // ---- out
    if (out == kSmall) {
        static bool raised[64];
        if (!raised[di.dev]) {
            e = hipFuncSetAttribute((const void*)soft_small_out_kernel<2, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
            if (e == hipSuccess)
                e = hipFuncSetAttribute((const void*)soft_small_out_kernel<1, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
            if (e != hipSuccess) return e;
            raised[di.dev] = true;
        }
        note_launch("soft_small_out_kernel");
        const int64_t enough = kSmallEnoughBlocks, ent_blocks = want_entropy ? (a.NN + 7) / 8 : 0;
        const auto launch = [&](auto kern, int mt, int c) {
            const int64_t blocks = small_blocks(p.T, p.O, mt, c);
            kern<<<grid(blocks + ent_blocks), dim3(512), (size_t)8 * mt * c * kWave * sizeof(f32x4_t), s>>>(a, blocks, ent_part, ent_parts,
                                                                                                            entropy_out);
        };
        if (small_blocks(p.T, p.O, 2, 8) >= enough) launch(soft_small_out_kernel<2, 8>, 2, 8);
        else if (small_blocks(p.T, p.O, 1, 8) >= enough) launch(soft_small_out_kernel<1, 8>, 1, 8);
        else launch(soft_small_out_kernel<1, 4>, 1, 4);
        return hipGetLastError();
    }
    note_launch(out == kBig ? "soft_w2x_kernel + soft_out_big_kernel" : "soft_w2x_kernel + soft_out_kernel");
    soft_w2x_kernel<<<dim3((unsigned)(((K2 + 31) / 32) * ((p.O + 31) / 32))), dim3(256), 0, s>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (out == kBig) soft_out_big_kernel<<<dim3(big_grid(p.T, (p.O + kBigN - 1) / kBigN)), dim3(256), 0, s>>>(a);
    else soft_out_kernel<<<grid((p.T + kTileM - 1) / kTileM * ((p.O + kTileN - 1) / kTileN)), dim3(256), 0, s>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (want_entropy) {
        note_launch("soft_entropy_sum_kernel");
        soft_entropy_sum_kernel<<<dim3((unsigned)a.NN), dim3(256), 0, s>>>(ent_part, ent_parts, p.T, a.NN, entropy_out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fff
