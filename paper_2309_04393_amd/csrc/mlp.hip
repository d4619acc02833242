// Brick-request predictor: a 24-64-64-9 perceptron (ReLU hidden layers, one
// logit per resolution level) trained with masked binary cross-entropy.
// This network is an addition to the paper's method; it only changes which
// bricks are streamed, never how a frame is rendered from a cache state.
//
// All products run on MFMA (v_mfma_f32_16x16x16_f16: FP16 operands, FP32
// accumulation).  A wave owns 16 rows at a time.  Layer shapes with padding:
// X [rows][32] (24 features), W1 [32][64], W2 [64][64], W3 [64][16] (9
// logits), Z [rows][16].  Operand lane layout of the 16x16x16 instruction
// (wave64, lane l = 16 q + r, i = 0..3):
//   A (16 x 16, row-major M x K):  A[r][4 q + i]
//   B (16 x 16, K x N):            B[4 q + i][r]
//   C/D (16 x 16, M x N):          D[4 q + i][r]
// So a 4-vector per lane, a fragment, that is A of a matrix is B of its
// transpose, a product's D is B of the matrix and A of its transpose, and
// D^T is the product with the operands exchanged.  Every operand is therefore
// made in registers, in the training kernel by taking each layer both ways:
// nothing goes through LDS, where the 2-byte fragment reads and their waits
// were what the kernels spent their time on.  Weights are held as fragments
// over all the rows of a wave; the FP16 copies hold W2 and W3 in both orders,
// so that a fragment is one 8-byte load.
// Training recomputes the forward pass per tile, backpropagates with the loss
// scaled by the number of unmasked entries (so FP16 operands stay in range),
// accumulates weight gradients in FP32 per wave, sums a block's four waves in
// LDS and the blocks' partials in a fixed order (deterministic) and applies
// Adam to FP32 master weights, refreshing the FP16 copies.
#include <math.h>
#include <string.h>

#include "common.h"

namespace ro {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// FP32 parameter block layout (floats), padded shapes.
constexpr int kW1 = 0, kB1 = kW1 + 32 * 64, kW2 = kB1 + 64, kB2 = kW2 + 64 * 64, kW3 = kB2 + 64,
              kB3 = kW3 + 64 * 16, kNP = kB3 + 16;  // 7312
// FP16 copies (halves): W1^T [64][32], W2 [64][64], W2^T [64][64],
// W3 [64][16], W3^T [16][64]
constexpr int kH1T = 0, kH2 = kH1T + 64 * 32, kH2T = kH2 + 64 * 64, kH3 = kH2T + 64 * 64, kH3T = kH3 + 64 * 16,
              kNH = kH3T + 16 * 64;  // 12288
constexpr int kWaves = 4;          // waves per workgroup
constexpr int kPartials = 256;     // most workgroups of the gradient kernel: one partial each, one per CU
constexpr int kStat = 4;           // per-partial scalars: loss sum, mask count

// A partial holds the weight gradients as fragments (D layout, four values of
// a lane together: 8 of W1, 16 of W2, 4 of W3), then the biases and the
// scalars, so that a wave stores and sums 16 bytes a lane.
constexpr int kFrag1 = 0, kFrag2 = 8, kFrag3 = 24, kFrags = 28;
constexpr int kPartB1 = kFrags * 256, kPartB2 = kPartB1 + 64, kPartB3 = kPartB2 + 64, kPartStat = kPartB3 + 16,
              kPartLen = kPartStat + kStat;
static_assert(kPartLen == kNP + kStat && kPartLen % 4 == 0, "partial length");

// Parameter at position k of a partial (k < kPartStat).
__device__ __forceinline__ int param_of(int k) {
    if (k >= kPartB3) return kB3 + k - kPartB3;
    if (k >= kPartB2) return kB2 + k - kPartB2;
    if (k >= kPartB1) return kB1 + k - kPartB1;
    const int f = k >> 8, lane = k >> 2 & 63, r = lane & 15, row = 4 * (lane >> 4) + (k & 3);
    if (f >= kFrag3) return kW3 + (16 * (f - kFrag3) + row) * 16 + r;
    const int g = f >= kFrag2 ? f - kFrag2 : f;
    return (f >= kFrag2 ? kW2 : kW1) + (16 * (g >> 2) + row) * 64 + 16 * (g & 3) + r;
}

__device__ __forceinline__ f4_t mfma16(half4_t a, half4_t b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ half4_t to_half(f4_t v) {
    return half4_t{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

// Forward weights as fragments: B of W1, w1[ks][j] = W1[16 ks + 4 q + i]
// [16 j + r], and so on (A of the transposes).
struct Weights {
    half4_t w1[2][4], w2[4][4], w3[4];
    __device__ __forceinline__ Weights(const _Float16 *__restrict__ wh) {
        const int r = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (ks < 2) w1[ks][j] = *(const half4_t *)(wh + kH1T + (16 * j + r) * 32 + 16 * ks + 4 * q);
                w2[ks][j] = *(const half4_t *)(wh + kH2T + (16 * j + r) * 64 + 16 * ks + 4 * q);
            }
            w3[ks] = *(const half4_t *)(wh + kH3T + r * 64 + 16 * ks + 4 * q);
        }
    }
};

// FP16 copies of parameter k.
__device__ __forceinline__ void put_half(_Float16 *__restrict__ wh, int k, float w) {
    const _Float16 h = (_Float16)w;
    if (k < kB1) {
        wh[kH1T + (k & 63) * 32 + (k >> 6)] = h;
    } else if (k >= kW2 && k < kB2) {
        const int e = k - kW2;
        wh[kH2 + e] = h;
        wh[kH2T + (e & 63) * 64 + (e >> 6)] = h;
    } else if (k >= kW3 && k < kB3) {
        const int e = k - kW3;
        wh[kH3 + e] = h;
        wh[kH3T + (e & 15) * 64 + (e >> 4)] = h;
    }
}

// Columns 16 ks + 4 q + i of row r0 + r of x (A fragments); zero past the
// end.  kWide: x is 8-byte aligned.
template <bool kWide>
__device__ __forceinline__ void load_x(const _Float16 *__restrict__ x, uint32_t rows, uint32_t r0, half4_t xa[2]) {
    const int r = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
    const _Float16 *at = x + (size_t)(r0 + r) * 32 + 4 * q;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        xa[ks] = half4_t{0, 0, 0, 0};
        if (r0 + r >= rows) continue;
        if (kWide) xa[ks] = *(const half4_t *)(at + 16 * ks);
        else
#pragma unroll
            for (int i = 0; i < 4; ++i) xa[ks][i] = at[16 * ks + i];
    }
}

__device__ __forceinline__ f4_t relu(f4_t v) {
    return f4_t{fmaxf(v[0], 0.0f), fmaxf(v[1], 0.0f), fmaxf(v[2], 0.0f), fmaxf(v[3], 0.0f)};
}

// Logits of 16 rows a wave and turn: every product transposed (units x rows),
// so that a layer's D is the next layer's B and a lane ends with four logits
// of one row.  32768 rows: 13 us with the tiles in LDS, 9 us now.
template <bool kWide>
__global__ void __launch_bounds__(256) k_mlp_fwd(const _Float16 *__restrict__ x, uint32_t rows,
                                                 const _Float16 *__restrict__ wh, const float *__restrict__ p,
                                                 float *__restrict__ z, bool z_wide) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const Weights W(wh);
    f4_t b1[4], b2[4], b3;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            b1[j][i] = p[kB1 + 16 * j + 4 * q + i];
            b2[j][i] = p[kB2 + 16 * j + 4 * q + i];
        }
        b3[i] = p[kB3 + 4 * q + i];
    }
    const uint32_t ntiles = (rows + 15) / 16;
    for (uint32_t t = blockIdx.x * kWaves + (threadIdx.x >> 6); t < ntiles; t += gridDim.x * kWaves) {
        half4_t xa[2], h1[4], h2[4];
        load_x<kWide>(x, rows, t * 16, xa);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t acc = {0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) acc = mfma16(W.w1[ks][j], xa[ks], acc);
            h1[j] = to_half(relu(acc + b1[j]));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t acc = {0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = mfma16(W.w2[ks][j], h1[ks], acc);
            h2[j] = to_half(relu(acc + b2[j]));
        }
        f4_t acc = {0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = mfma16(W.w3[ks], h2[ks], acc);
        acc += b3;
        const uint32_t row = t * 16 + r;
        if (row >= rows) continue;
        float *o = z + (size_t)row * 16 + 4 * q;
        if (z_wide) *(f4_t *)o = acc;
        else
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = acc[i];
    }
}

// Inputs of one tile: A of x and of x^T, labels and masks in both orders,
// [row 4 q + i][r] and [row r][4 q + i]; zero past the end.
struct Tile {
    half4_t xa[2], xt[2];
    uint8_t y[4], m[4];
    uint32_t yt, mt;  // four bytes
};

__device__ __forceinline__ float byte_of(uint32_t v, int i) { return (float)(v >> (8 * i) & 255u); }

// kWide: x is 8-byte aligned, y and msk are 4-byte aligned.
template <bool kWide>
__device__ __forceinline__ void load_tile(const _Float16 *__restrict__ x, const uint8_t *__restrict__ y,
                                          const uint8_t *__restrict__ msk, uint32_t rows, uint32_t r0, Tile &T) {
    const int r = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
    load_x<kWide>(x, rows, r0, T.xa);
    T.yt = T.mt = 0;
    if (r0 + r < rows) {
        const size_t at = (size_t)(r0 + r) * 16 + 4 * q;
        if (kWide) {
            T.yt = *(const uint32_t *)(y + at);
            T.mt = *(const uint32_t *)(msk + at);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                T.yt |= (uint32_t)y[at + i] << (8 * i);
                T.mt |= (uint32_t)msk[at + i] << (8 * i);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t row = r0 + 4 * q + i;
        T.y[i] = T.m[i] = 0;
        T.xt[0][i] = T.xt[1][i] = (_Float16)0.0f;
        if (row >= rows) continue;
        T.y[i] = y[(size_t)row * 16 + r];
        T.m[i] = msk[(size_t)row * 16 + r];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) T.xt[mt][i] = x[(size_t)row * 32 + 16 * mt + r];
    }
}

// Gradient partials, one per block: kPartLen floats to part[block].
// 32768 rows: 80 us with 256 waves on 64 CUs and the tiles in LDS, 18.6 us with
// two tiles on each of 1024 waves.  A wave holds the weights, the sums and a
// tile in 446 registers, so a SIMD has one wave and what bounds it is that
// wave's own chain: 2.5 us a tile, the rest loading weights and summing.
template <bool kWide, bool kLoss>
__global__ void __launch_bounds__(256, 1) k_mlp_grad(const _Float16 *__restrict__ x, const uint8_t *__restrict__ y,
                                                     const uint8_t *__restrict__ msk, uint32_t rows,
                                                     const _Float16 *__restrict__ wh, const float *__restrict__ p,
                                                     float *__restrict__ part) {
    __shared__ f4_t S[2][kPartLen / 4];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const uint32_t ntiles = (rows + 15) / 16;
    uint32_t t = blockIdx.x * kWaves + wv;
    Tile cur;  // the next tile's inputs are on their way while one is worked on
    if (t < ntiles) load_tile<kWide>(x, y, msk, rows, t * 16, cur);
    const Weights W(wh);
    // W2^T and W3^T as B fragments: rows of the matrices
    half4_t w2t[4][4], w3t[4];
    float b1[4], b2[4];
    f4_t b1t[4], b2t[4], b3t;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) w2t[ks][j] = *(const half4_t *)(wh + kH2 + (16 * j + r) * 64 + 16 * ks + 4 * q);
        w3t[j] = *(const half4_t *)(wh + kH3 + (16 * j + r) * 16 + 4 * q);
        b1[j] = p[kB1 + 16 * j + r];
        b2[j] = p[kB2 + 16 * j + r];
        b3t[j] = p[kB3 + 4 * q + j];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b1t[j][i] = p[kB1 + 16 * j + 4 * q + i];
            b2t[j][i] = p[kB2 + 16 * j + 4 * q + i];
        }
    }
    const float b3 = p[kB3 + r];
    f4_t g1[2][4], g2[4][4], g3[4];
    float gb1[4] = {0, 0, 0, 0}, gb2[4] = {0, 0, 0, 0}, gb3 = 0.0f, lsum = 0.0f, msum = 0.0f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        g3[a] = f4_t{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            g2[a][b] = f4_t{0, 0, 0, 0};
            if (a < 2) g1[a][b] = f4_t{0, 0, 0, 0};
        }
    }
    const f4_t zero = {0, 0, 0, 0};
    for (; t < ntiles; t += gridDim.x * kWaves) {
        const uint32_t r0 = t * 16;
        const Tile T = cur;
        if (t + gridDim.x * kWaves < ntiles) load_tile<kWide>(x, y, msk, rows, (t + gridDim.x * kWaves) * 16, cur);
        const bool in_r = r0 + r < rows;
        // forward: rows x units (h, for the weight gradients) and units x rows
        // (ht, the next layer's operand); bit 4 j + i of on*: the unit is on
        f4_t z = zero, zt = zero;
        half4_t h1[4], h1t[4], h2[4], h2t[4];
        f4_t s1[4], s2[4], s2t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t a = zero, at = zero;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                a = mfma16(T.xa[ks], W.w1[ks][j], a);
                at = mfma16(W.w1[ks][j], T.xa[ks], at);
            }
            a += b1[j];
            at += b1t[j];
            s1[j] = a;
            h1[j] = to_half(relu(a));
            h1t[j] = to_half(relu(at));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t a = zero, at = zero;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                a = mfma16(h1t[ks], W.w2[ks][j], a);
                at = mfma16(W.w2[ks][j], h1t[ks], at);
            }
            a += b2[j];
            at += b2t[j];
            s2[j] = a;
            s2t[j] = at;
            h2[j] = to_half(relu(a));
            h2t[j] = to_half(relu(at));
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            z = mfma16(h2t[ks], W.w3[ks], z);
            zt = mfma16(W.w3[ks], h2t[ks], zt);
        }
        z += b3;
        zt += b3t;
        // dz = mask * (sigmoid(z) - y)   (loss scaled by the mask count)
        f4_t dzf, dzft;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float d = 0.0f, dt = 0.0f;
            if (r0 + 4 * q + i < rows) {
                const float zz = z[i], mk = (float)T.m[i], yy = (float)T.y[i];
                const float s = 1.0f / (1.0f + expf(-zz));
                d = mk * (s - yy);
                // softplus(z) - y z, stably
                if (kLoss) lsum += mk * (fmaxf(zz, 0.0f) + log1pf(expf(-fabsf(zz))) - yy * zz);
                msum += mk;
            }
            if (in_r) dt = byte_of(T.mt, i) * (1.0f / (1.0f + expf(-zt[i])) - byte_of(T.yt, i));
            dzf[i] = d;
            dzft[i] = dt;
            gb3 += d;
        }
        const half4_t dz = to_half(dzf), dzt = to_half(dzft);
        // gW3 += h2^T dz; da2 = (dz W3^T) * (a2 > 0), both ways
        half4_t d2[4], d2t[4], d1[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            g3[j] = mfma16(h2[j], dz, g3[j]);
            f4_t a = mfma16(dzt, w3t[j], zero), at = mfma16(w3t[j], dzt, zero);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = s2[j][i] > 0.0f ? a[i] : 0.0f;
                at[i] = s2t[j][i] > 0.0f ? at[i] : 0.0f;
                gb2[j] += a[i];
            }
            d2[j] = to_half(a);
            d2t[j] = to_half(at);
        }
        // gW2 += h1^T da2; da1 = (da2 W2^T) * (a1 > 0)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) g2[mt][nt] = mfma16(h1[mt], d2[nt], g2[mt][nt]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f4_t a = zero;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = mfma16(d2t[ks], w2t[ks][j], a);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = s1[j][i] > 0.0f ? a[i] : 0.0f;
                gb1[j] += a[i];
            }
            d1[j] = to_half(a);
        }
        // gW1 += x^T da1
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) g1[mt][nt] = mfma16(T.xt[mt], d1[nt], g1[mt][nt]);
    }
    // bias partials: sum the four lane groups (q) of each column
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        gb1[j] += __shfl_xor(gb1[j], 16, 64);
        gb1[j] += __shfl_xor(gb1[j], 32, 64);
        gb2[j] += __shfl_xor(gb2[j], 16, 64);
        gb2[j] += __shfl_xor(gb2[j], 32, 64);
    }
    gb3 += __shfl_xor(gb3, 16, 64);
    gb3 += __shfl_xor(gb3, 32, 64);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lsum += __shfl_xor(lsum, off, 64);
        msum += __shfl_xor(msum, off, 64);
    }
    // (wave 0 + wave 2) + (wave 1 + wave 3)
    f4_t *o = S[wv & 1];
    float *ob = (float *)o;
#pragma unroll
    for (int turn = 0; turn < 2; ++turn) {
        if (wv >> 1 == turn) {
            auto put = [&](int f, f4_t v) { o[f * 64 + lane] = turn ? o[f * 64 + lane] + v : v; };
            auto put1 = [&](int k, float v) { ob[k] = turn ? ob[k] + v : v; };
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    if (mt < 2) put(kFrag1 + 4 * mt + nt, g1[mt & 1][nt]);
                    put(kFrag2 + 4 * mt + nt, g2[mt][nt]);
                }
                put(kFrag3 + mt, g3[mt]);
            }
            if (q == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    put1(kPartB1 + 16 * j + r, gb1[j]);
                    put1(kPartB2 + 16 * j + r, gb2[j]);
                }
                put1(kPartB3 + r, gb3);
            }
            if (lane < kStat) put1(kPartStat + lane, lane == 0 ? lsum : lane == 1 ? msum : 0.0f);
        }
        __syncthreads();
    }
    f4_t *to = (f4_t *)(part + (size_t)blockIdx.x * kPartLen);
#pragma unroll 4
    for (int k = threadIdx.x; k < kPartLen / 4; k += 256) to[k] = S[0][k] + S[1][k];
}

struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};

// Sum of the partials in a fixed order (deterministic), the mean over the
// unmasked entries, and, with kStep, the Adam step on the FP32 master weights
// with their FP16 copies: one launch, where a sum, a scaling and a step were
// three.  A block takes 64 positions of the partials; each of its 16 waves sums every 16th
// partial of them (coalesced rows, independent loads), then a pairwise tree
// over the 16 wave sums in LDS.  The count of unmasked entries is summed by
// every block for itself, in the same order.
constexpr int kRedGroups = 16;
template <bool kStep>
__global__ void __launch_bounds__(64 * kRedGroups) k_mlp_update(const float *__restrict__ part, int nparts,
                                                               float *__restrict__ grad, float *__restrict__ stat,
                                                               float *__restrict__ p, float *__restrict__ m,
                                                               float *__restrict__ v, _Float16 *__restrict__ wh,
                                                               AdamStep st) {
    __shared__ float sm[kRedGroups][64], cnt[kRedGroups];
    const int lane = threadIdx.x & 63, gi = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane;
    // partial 16 lane + gi is lane's: 256 at most, so one a lane is enough
    static_assert(kPartials <= 64 * kRedGroups, "one count per thread");
    float n = lane * kRedGroups + gi < nparts ? part[(size_t)(lane * kRedGroups + gi) * kPartLen + kPartStat + 1] : 0.0f;
    float acc = 0.0f;
    if (k < kPartLen) {
#pragma unroll 4
        for (int w = gi; w < nparts; w += kRedGroups) acc += part[(size_t)w * kPartLen + k];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
    sm[gi][lane] = acc;
    if (lane == 0) cnt[gi] = n;
    __syncthreads();
    for (int h = kRedGroups / 2; h >= 1; h >>= 1) {
        if (gi < h) {
            sm[gi][lane] += sm[gi + h][lane];
            if (lane == 0) cnt[gi] += cnt[gi + h];
        }
        __syncthreads();
    }
    if (gi != 0 || k >= kPartLen) return;
    if (k >= kPartStat) {
        stat[k - kPartStat] = sm[0][lane];
        return;
    }
    const int e = param_of(k);
    const float gk = sm[0][lane] / fmaxf(cnt[0], 1.0f);
    grad[e] = gk;
    if (!kStep) return;
    const float mk = st.b1 * m[e] + (1.0f - st.b1) * gk;
    const float vk = st.b2 * v[e] + (1.0f - st.b2) * gk * gk;
    m[e] = mk;
    v[e] = vk;
    const float w = p[e] - st.lr * (mk / st.c1) / (sqrtf(vk / st.c2) + st.eps);
    p[e] = w;
    put_half(wh, e, w);
}

__global__ void k_mlp_refresh(const float *__restrict__ p, _Float16 *__restrict__ wh) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kNP) put_half(wh, k, p[k]);
}

}  // namespace ro

using namespace ro;

// Device layout of the parameter buffer (bytes): FP32 master [kNP], Adam m
// [kNP], Adam v [kNP], gradient [kNP], stats [kStat], FP16 copies [kNH];
// workspace: kPartials x (kNP + kStat) floats.
constexpr uint32_t kFwdBlocks = 512;

struct ro_mlp {
    float *p, *m, *v, *g, *stat;
    _Float16 *wh;
    float *part;
    uint32_t step;
};

static size_t mlp_param_bytes() { return (size_t)(4 * kNP + kStat) * 4 + (size_t)kNH * 2 + 256; }
static size_t mlp_work_bytes() { return (size_t)kPartials * (kNP + kStat) * 4; }

extern "C" ro_status ro_mlp_query(size_t *param_bytes, size_t *workspace_bytes) {
    RO_CHECK(param_bytes && workspace_bytes, RO_E_ARG, "null argument");
    *param_bytes = mlp_param_bytes();
    *workspace_bytes = mlp_work_bytes();
    return RO_OK;
}

extern "C" ro_status ro_mlp_create(void *params_dev, void *workspace_dev, ro_mlp **out) {
    RO_CHECK(params_dev && workspace_dev && out, RO_E_ARG, "null argument");
    RO_CHECK(((uintptr_t)params_dev & 255u) == 0 && ((uintptr_t)workspace_dev & 255u) == 0, RO_E_ARG,
             "device buffers must be 256-byte aligned");
    ro_mlp *n = new (std::nothrow) ro_mlp;
    RO_CHECK(n, RO_E_NOMEM, "out of host memory");
    float *f = (float *)params_dev;
    n->p = f;
    n->m = f + kNP;
    n->v = f + 2 * kNP;
    n->g = f + 3 * kNP;
    n->stat = f + 4 * kNP;
    n->wh = (_Float16 *)(f + 4 * kNP + kStat);
    n->part = (float *)workspace_dev;
    n->step = 0;
    *out = n;
    return RO_OK;
}

extern "C" void ro_mlp_destroy(ro_mlp *n) { delete n; }

// Host weight layout (unpadded): W1[24][64], b1[64], W2[64][64], b2[64],
// W3[64][9], b3[9].

extern "C" ro_status ro_mlp_set_weights(ro_mlp *n, const float *host, void *stream) {
    RO_CHECK(n && host, RO_E_ARG, "null argument");
    std::vector<float> buf(3 * (size_t)kNP, 0.0f);  // p, m = 0, v = 0
    const float *h = host;
    for (int i = 0; i < 24; ++i)
        for (int j = 0; j < 64; ++j) buf[kW1 + i * 64 + j] = *h++;
    for (int j = 0; j < 64; ++j) buf[kB1 + j] = *h++;
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 64; ++j) buf[kW2 + i * 64 + j] = *h++;
    for (int j = 0; j < 64; ++j) buf[kB2 + j] = *h++;
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 9; ++j) buf[kW3 + i * 16 + j] = *h++;
    for (int j = 0; j < 9; ++j) buf[kB3 + j] = *h++;
    hipStream_t s = (hipStream_t)stream;
    RO_HIP(hipMemcpyAsync(n->p, buf.data(), sizeof(float) * 3 * kNP, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_mlp_refresh, dim3((kNP + 255) / 256), dim3(256), 0, s, n->p, n->wh);
    RO_HIP(hipGetLastError());
    RO_HIP(hipStreamSynchronize(s));  // the host buffer dies here
    n->step = 0;
    return RO_OK;
}

extern "C" ro_status ro_mlp_get_weights(const ro_mlp *n, float *host, void *stream) {
    RO_CHECK(n && host, RO_E_ARG, "null argument");
    std::vector<float> buf(kNP);
    hipStream_t s = (hipStream_t)stream;
    RO_HIP(hipMemcpyAsync(buf.data(), n->p, sizeof(float) * kNP, hipMemcpyDeviceToHost, s));
    RO_HIP(hipStreamSynchronize(s));
    float *h = host;
    for (int i = 0; i < 24; ++i)
        for (int j = 0; j < 64; ++j) *h++ = buf[kW1 + i * 64 + j];
    for (int j = 0; j < 64; ++j) *h++ = buf[kB1 + j];
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 64; ++j) *h++ = buf[kW2 + i * 64 + j];
    for (int j = 0; j < 64; ++j) *h++ = buf[kB2 + j];
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 9; ++j) *h++ = buf[kW3 + i * 16 + j];
    for (int j = 0; j < 9; ++j) *h++ = buf[kB3 + j];
    return RO_OK;
}

extern "C" ro_status ro_mlp_forward(ro_mlp *n, const uint16_t *x, uint32_t rows, float *z, void *stream) {
    RO_CHECK(n && (rows == 0 || (x && z)), RO_E_ARG, "null argument");
    if (rows == 0) return RO_OK;
    hipStream_t s = (hipStream_t)stream;
    // two tiles or more a wave once the CUs are full: the weights are read once
    const uint32_t tiles = (rows + 15) / 16;
    uint32_t blocks = (tiles + kWaves - 1) / kWaves;
    if (blocks > kFwdBlocks) blocks = kFwdBlocks;
    const bool z_wide = (uintptr_t)z % 16 == 0;
    if ((uintptr_t)x % 8 == 0)
        hipLaunchKernelGGL(k_mlp_fwd<true>, dim3(blocks), dim3(64 * kWaves), 0, s, (const _Float16 *)x, rows, n->wh,
                           n->p, z, z_wide);
    else
        hipLaunchKernelGGL(k_mlp_fwd<false>, dim3(blocks), dim3(64 * kWaves), 0, s, (const _Float16 *)x, rows, n->wh,
                           n->p, z, z_wide);
    RO_HIP(hipGetLastError());
    return RO_OK;
}

// Gradients of the rows and, with a step, the weights' update; the loss where
// it is asked for (its logarithm is a tenth of the kernel's instructions).
static ro_status mlp_grad(ro_mlp *n, const uint16_t *x, const uint8_t *y, const uint8_t *mask, uint32_t rows,
                          const AdamStep *step, bool loss, hipStream_t s) {
    const uint32_t tiles = (rows + 15) / 16;
    uint32_t blocks = (tiles + kWaves - 1) / kWaves;
    if (blocks > (uint32_t)kPartials) blocks = kPartials;
    if (blocks < 1) blocks = 1;  // no rows: zero gradients
    const bool wide = (uintptr_t)x % 8 == 0 && (uintptr_t)y % 4 == 0 && (uintptr_t)mask % 4 == 0;
    auto grad = wide ? (loss ? k_mlp_grad<true, true> : k_mlp_grad<true, false>)
                     : (loss ? k_mlp_grad<false, true> : k_mlp_grad<false, false>);
    hipLaunchKernelGGL(grad, dim3(blocks), dim3(64 * kWaves), 0, s, (const _Float16 *)x, y, mask, rows, n->wh, n->p,
                       n->part);
    RO_HIP(hipGetLastError());
    const dim3 grid((kPartLen + 63) / 64), block(64 * kRedGroups);
    if (step)
        hipLaunchKernelGGL(k_mlp_update<true>, grid, block, 0, s, n->part, (int)blocks, n->g, n->stat, n->p, n->m, n->v,
                           n->wh, *step);
    else
        hipLaunchKernelGGL(k_mlp_update<false>, grid, block, 0, s, n->part, (int)blocks, n->g, n->stat, n->p, n->m,
                           n->v, n->wh, AdamStep{});
    RO_HIP(hipGetLastError());
    return RO_OK;
}

extern "C" ro_status ro_mlp_gradients(ro_mlp *n, const uint16_t *x, const uint8_t *y, const uint8_t *mask,
                                      uint32_t rows, float *grads_host, float *loss_host, void *stream) {
    RO_CHECK(n && x && y && mask && grads_host, RO_E_ARG, "null argument");
    hipStream_t s = (hipStream_t)stream;
    ro_status st = mlp_grad(n, x, y, mask, rows, nullptr, loss_host != nullptr, s);
    if (st) return st;
    std::vector<float> g(kNP + kStat);
    RO_HIP(hipMemcpyAsync(g.data(), n->g, sizeof(float) * (kNP + kStat), hipMemcpyDeviceToHost, s));
    RO_HIP(hipStreamSynchronize(s));
    float *h = grads_host;
    for (int i = 0; i < 24; ++i)
        for (int j = 0; j < 64; ++j) *h++ = g[kW1 + i * 64 + j];
    for (int j = 0; j < 64; ++j) *h++ = g[kB1 + j];
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 64; ++j) *h++ = g[kW2 + i * 64 + j];
    for (int j = 0; j < 64; ++j) *h++ = g[kB2 + j];
    for (int i = 0; i < 64; ++i)
        for (int j = 0; j < 9; ++j) *h++ = g[kW3 + i * 16 + j];
    for (int j = 0; j < 9; ++j) *h++ = g[kB3 + j];
    if (loss_host) *loss_host = g[kNP + 0] / (g[kNP + 1] > 0 ? g[kNP + 1] : 1.0f);
    return RO_OK;
}

extern "C" ro_status ro_mlp_train_step(ro_mlp *n, const uint16_t *x, const uint8_t *y, const uint8_t *mask,
                                       uint32_t rows, float lr, float *loss_host, void *stream) {
    RO_CHECK(n && x && y && mask, RO_E_ARG, "null argument");
    RO_CHECK(lr > 0.0f, RO_E_ARG, "lr must be > 0");
    hipStream_t s = (hipStream_t)stream;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float t = (float)(n->step + 1);
    const AdamStep step = {lr, b1, b2, eps, 1.0f - powf(b1, t), 1.0f - powf(b2, t)};
    ro_status st = mlp_grad(n, x, y, mask, rows, &step, loss_host != nullptr, s);
    if (st) return st;
    n->step += 1;
    if (loss_host) {
        float stat[kStat];
        RO_HIP(hipMemcpyAsync(stat, n->stat, sizeof(stat), hipMemcpyDeviceToHost, s));
        RO_HIP(hipStreamSynchronize(s));
        *loss_host = stat[0] / (stat[1] > 0 ? stat[1] : 1.0f);
    }
    return RO_OK;
}
