// Learned material model: a small MLP that maps (material label, incidence
// cosine, log10 frequency) to (Gamma_TE, Gamma_TM, S) for every interaction
// slot of a tape, in place of the per-label Fresnel model.
//
//   x (32) = [emb[label] (16), cos, log10(f/1 GHz), 0...]
//   h1 = GELU(W1 x + b1), h2 = GELU(W2 h1 + b2), h3 = GELU(W3 h2 + b3)   (64 each)
//   z = W4 h3 + b4 (5 used of 16); Gamma_TE = (z0 + j z1) tanh|.|/|.|,
//   Gamma_TM = (z2 + j z3) tanh|.|/|.|, S = sigmoid(z4)
//
// BF16 operands, FP32 accumulation, on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16). Lane layout of that instruction (one wavefront):
//   A[i][k]: lane l holds i = l % 16, k = 8 (l / 16) + j, j = 0..7
//   B[k][n]: lane l holds n = l % 16, k = 8 (l / 16) + j
//   C[i][n]: lane l holds n = l % 16, i = 4 (l / 16) + r, r = 0..3
//
// Forward: every layer is computed transposed, Y^T = W X^T, with the weights
// as the A operand (held in registers for the wavefront's whole life) and
// 16 rows as the B operand. The result leaves lane (n, g = l / 16) holding
// row n's outputs 16 t + 4 g + r (t = 0..3 output tiles, r = 0..3). A
// contraction does not care in which order its K index runs, so the next
// layer takes its K index in exactly that order: K step ks, element j is
// input 16 (2 ks + j / 4) + 4 g + j % 4, which lane (n, g) already holds. The
// weights are loaded in the same permuted order, and the activations never
// leave the registers between layers.
// Backward: the forward recompute and the gradient chain dH = W^T dZ run the
// same way; the weight gradients dW = dZ^T H contract over rows: a block's
// wavefronts hand their rows to each other through LDS and share the tiles of
// every weight gradient, each accumulating its own in registers, written
// once per block as a partial that a fixed-order reduction adds up.
//
// GELU: erf by Abramowitz & Stegun 7.1.26 (absolute error below 1.5e-7 in
// erf; GELU within 3.3e-7) in the backward pass; the forward pass
// interpolates linearly in a table of that GELU at 8193 nodes over [-8, 8]
// (spacing 2^-9, built in LDS by every block; beyond the ends the end
// intervals extend linearly), within 1e-6. Both are far below the BF16
// rounding of the activations (2^-8 relative).
#include <cstring>

#include "common.h"
#include "internal.h"
#include "pcrt.h"

namespace pcrt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = 32, kHid = 64, kOut = 16, kEmb = 16;
constexpr int kW1 = kHid * kIn, kW2 = kHid * kHid, kW3 = kHid * kHid, kW4 = kOut * kHid;
constexpr int kWAll = kW1 + kW2 + kW3 + kW4;       // 11264 bf16
constexpr int kBAll = kHid * 3 + kOut;             // 208 floats
constexpr int kTileRows = 16;

__device__ __forceinline__ float bf(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ __forceinline__ uint16_t to_bf(float f) {  // round to nearest even
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ __bf16 as_b(uint16_t u) { return __builtin_bit_cast(__bf16, u); }

// Lanes of one wavefront hand tiles to each other through LDS: order the
// writes before the following reads (wave-scope fence + scheduling barrier).
// GELU(z) = z Phi(z), Phi(z) = (1 + erf(z / sqrt 2)) / 2. With x = |z| / sqrt 2,
// erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x)
// (Abramowitz & Stegun 7.1.26), so h = (1 - erf(x)) / 2 = Phi(-|z|) and
// GELU(z) = max(z, 0) - |z| h. Returns h; e receives exp(-z^2 / 2).
__device__ __forceinline__ float norm_tail(float z, float &e) {
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, fabsf(z), 1.0f));
    const float poly =  // the coefficients halved
        fmaf(fmaf(fmaf(fmaf(0.5307027145f, t, -0.7265760135f), t, 0.7107068705f), t, -0.142248368f), t, 0.127414796f) *
        t;
    e = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);  // 2^(-z^2 log2(e) / 2)
    return poly * e;
}
// max(z, 0) on the bit pattern: a non-negative float is a non-negative int32,
// a negative one a negative int32 (one integer max, no NaN canonicalisation)
__device__ __forceinline__ float relu(float z) { return __int_as_float(max(__float_as_int(z), 0)); }
__device__ __forceinline__ float gelu(float z) {
    float e;
    const float h = norm_tail(z, e);
    return fmaf(-fabsf(z), h, relu(z));
}
// GELU'(z) = Phi(z) + z phi(z), phi(z) = exp(-z^2 / 2) / sqrt(2 pi).
__device__ __forceinline__ float gelu_grad(float z) {
    float e;
    const float h = norm_tail(z, e);
    return fmaf(z * 0.39894228040143268f, e, z >= 0.f ? 1.0f - h : h);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Two floats to two bf16 (round to nearest even), low half first.
__device__ __forceinline__ uint32_t pack_bf2(float a, float b) {
    const bf16x2 v = __builtin_convertvector((f32x2){a, b}, bf16x2);
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ bf16x8 bf8_of(u32x4 p) { return __builtin_bit_cast(bf16x8, p); }

// (u + j v) tanh(r)/r and its Jacobian (a = d re/du, b = d re/dv = d im/du, d = d im/dv).
__device__ __forceinline__ void radial(float u, float v, float &re, float &im, float &a, float &b, float &d) {
    float r = sqrtf(u * u + v * v);
    float g, gp;  // g(r) = tanh r / r, gp = g'(r) / r
    if (r < 1e-4f) {
        g = 1.f - r * r / 3.f;
        gp = -2.f / 3.f;
    } else {
        float t = tanhf(r);
        g = t / r;
        gp = (r * (1.f - t * t) - t) / (r * r * r);
    }
    re = u * g;
    im = v * g;
    a = g + u * u * gp;
    b = u * v * gp;
    d = g + v * v * gp;
}

struct MlpArgs {
    const uint16_t *w;   // bf16 bits: W1 [64][32], W2 [64][64], W3 [64][64], W4 [16][64] (row = output)
    const float *b;      // b1 [64], b2 [64], b3 [64], b4 [16]
    const float *emb;    // [n_labels][16] float32
    uint32_t n_labels;
    uint32_t n;          // rows
    const uint16_t *label;
    const float *cosv;
    float logf;
    float *out;          // [n][8]
    const float *gout;   // [n][8]
    float *part;         // per-block gradient partials [blocks][part_stride]
    uint32_t part_stride;
};

// Per-lane MFMA A fragments of the weights in the transposed formulation
// (lane (i, g): output 16 t + i, K elements j = 0..7 of K step ks), and the
// biases of the outputs the lane holds (16 t + 4 g + r at index 4 t + r).
struct RegNet {
    bf16x8 w1[4], w2[4][2], w3[4][2], w4[2];
    f32x4 b1[4], b2[4], b3[4], b4;  // the MFMA accumulators start from these
};

// Input index of K step ks, element j, lane group g, for the hidden layers
// (the order in which the previous layer's outputs sit in the registers).
__device__ __forceinline__ int perm_k(int ks, int g, int j) { return 16 * (2 * ks + (j >> 2)) + 4 * g + (j & 3); }

__device__ __forceinline__ bf16x8 wfrag(const uint16_t *W, int ld, int row, int ks, int g, bool natural) {
    u32x4 p;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = 2 * q;
        const int k0 = natural ? 8 * g + j : perm_k(ks, g, j), k1 = natural ? 8 * g + j + 1 : perm_k(ks, g, j + 1);
        p[q] = (uint32_t)W[row * ld + k0] | ((uint32_t)W[row * ld + k1] << 16);
    }
    return bf8_of(p);
}

__device__ __forceinline__ void load_regnet(const MlpArgs &M, int lane, RegNet &R) {
    const int i = lane & 15, g = lane >> 4;
    const uint16_t *w1 = M.w, *w2 = w1 + kW1, *w3 = w2 + kW2, *w4 = w3 + kW3;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        R.w1[t] = wfrag(w1, kIn, 16 * t + i, 0, g, true);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            R.w2[t][ks] = wfrag(w2, kHid, 16 * t + i, ks, g, false);
            R.w3[t][ks] = wfrag(w3, kHid, 16 * t + i, ks, g, false);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            R.b1[t][r] = M.b[16 * t + 4 * g + r];
            R.b2[t][r] = M.b[kHid + 16 * t + 4 * g + r];
            R.b3[t][r] = M.b[2 * kHid + 16 * t + 4 * g + r];
        }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) R.w4[ks] = wfrag(w4, kHid, i, ks, g, false);
#pragma unroll
    for (int r = 0; r < 4; ++r) R.b4[r] = M.b[3 * kHid + 4 * g + r];
}

// Input B fragment of one row for lane group g (natural K order): g = 0, 1
// the embedding's halves, g = 2 (cos, log f, 0, ...), g = 3 zeros; an empty
// slot or a row past the end gives zeros.
__device__ __forceinline__ bf16x8 input_frag(const MlpArgs &M, uint32_t row, uint16_t lab, int g) {
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (lab < M.n_labels) {
        if (g < 2) {
            const float4 *e = (const float4 *)(M.emb + (size_t)lab * kEmb + 8 * g);
            const float4 a = e[0], b = e[1];
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else if (g == 2) {
            v[0] = M.cosv[row];
            v[1] = M.logf;
        }
    }
    return bf8_of(u32x4{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])});
}

// GELU of one layer's outputs (C layout, bias included) into the next layer's two B
// fragments (K order perm_k).
constexpr int kGeluN = 8192;  // table intervals over [-8, 8): node i at -8 + i / 512
// GELU from the table (value, slope to the next node) of the node below z;
// z outside [-8, 8) uses the end interval's line (GELU(z) = z and 0 there to
// FP32 precision).
__device__ __forceinline__ float gelu_tab(const float2 *tab, float z) {
    const float x = fmaf(z, 512.f, 4096.f);
    const float c = __builtin_amdgcn_fmed3f(floorf(x), 0.f, (float)(kGeluN - 1));
    const float2 e = tab[(int)c];
    return fmaf(x - c, e.y, e.x);
}
__device__ void build_gelu_table(float2 *tab) {  // tab[kGeluN + 1], every thread of the block
    for (int i = threadIdx.x; i <= kGeluN; i += blockDim.x) tab[i].x = gelu(-8.f + (float)i * (1.f / 512.f));
    __syncthreads();
    constexpr int kPer = kGeluN / 256;
    float slope[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = threadIdx.x + 256 * k;
        slope[k] = tab[i + 1].x - tab[i].x;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) tab[threadIdx.x + 256 * k].y = slope[k];
    __syncthreads();
}
__device__ __forceinline__ void act_frags(const f32x4 (&acc)[4], bf16x8 (&h)[2], const float2 *tab) {
    float v[16];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[4 * t + r] = gelu_tab(tab, acc[t][r]);  // the accumulation started from the bias
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        h[ks] = bf8_of(u32x4{pack_bf2(v[8 * ks + 0], v[8 * ks + 1]), pack_bf2(v[8 * ks + 2], v[8 * ks + 3]),
                             pack_bf2(v[8 * ks + 4], v[8 * ks + 5]), pack_bf2(v[8 * ks + 6], v[8 * ks + 7])});
}

#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)

// The three hidden layers and the output layer of one 16-row tile; x: the
// input fragment. Returns z4 (C layout: lane (n, g) holds outputs 4 g + r).
__device__ __forceinline__ f32x4 net_forward(const RegNet &R, bf16x8 x, const float2 *tab) {
    f32x4 acc[4];
    bf16x8 h[2];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = MFMA16(R.w1[t], x, R.b1[t]);
    act_frags(acc, h, tab);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = MFMA16(R.w2[t][1], h[1], MFMA16(R.w2[t][0], h[0], R.b2[t]));
    act_frags(acc, h, tab);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = MFMA16(R.w3[t][1], h[1], MFMA16(R.w3[t][0], h[0], R.b3[t]));
    act_frags(acc, h, tab);
    return MFMA16(R.w4[1], h[1], MFMA16(R.w4[0], h[0], R.b4));
}

constexpr int kFwdTiles = 8;  // 16-row tiles a wavefront carries at once (independent MFMA chains); 1 where there are few

// Persistent wavefronts, each holding the whole network in registers; tiles
// are dealt by wavefront index (grid stride), kFwdTiles at a time.
// Output map of the forward pass: (u + j v) tanh(r) / r with tanh r =
// 1 - 2 / (e^{2r} + 1) (relative error near 1e-6 down to r = 0.1), and the
// series 1 - r^2 / 3 + 2 r^4 / 15 below (truncation 6e-8 relative).
__device__ __forceinline__ void radial_fwd(float u, float v, float &re, float &im) {
    const float r2 = u * u + v * v;
    float g;
    if (r2 < 0.01f) {
        g = fmaf(fmaf(0.133333333f, r2, -0.333333333f), r2, 1.0f);
    } else {
        const float rinv = __builtin_amdgcn_rsqf(r2), r = r2 * rinv;
        const float ex = __builtin_amdgcn_exp2f(2.8853900817779268f * r);  // e^{2r}
        g = (1.0f - 2.0f * __builtin_amdgcn_rcpf(ex + 1.0f)) * rinv;
    }
    re = u * g;
    im = v * g;
}

template <int kT>
__global__ __launch_bounds__(256) void k_mlp_forward(MlpArgs M) {
    __shared__ float2 tab[kGeluN + 1];
    build_gelu_table(tab);
    const int lane = threadIdx.x & 63, g = lane >> 4, nl = lane & 15;
    RegNet R;
    load_regnet(M, lane, R);
    const uint32_t wave = blockIdx.x * 4 + (threadIdx.x >> 6), n_waves = gridDim.x * 4;
    const uint32_t n_tiles = (M.n + kTileRows - 1) / kTileRows;
    for (uint32_t t0 = wave * kT; t0 < n_tiles; t0 += n_waves * kT) {
        uint32_t row[kT];
        uint16_t lab[kT];
        f32x4 z4[kT];
#pragma unroll
        for (int tt = 0; tt < kT; ++tt) {
            row[tt] = (t0 + tt) * kTileRows + nl;
            lab[tt] = row[tt] < M.n ? M.label[row[tt]] : (uint16_t)0xffff;
        }
#pragma unroll
        for (int tt = 0; tt < kT; ++tt) z4[tt] = net_forward(R, input_frag(M, row[tt], lab[tt], g), tab);
#pragma unroll
        for (int tt = 0; tt < kT; ++tt) {
            if (row[tt] >= M.n || g > 1) continue;
            float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
            if (lab[tt] < M.n_labels) {
                if (g == 0) {
                    radial_fwd(z4[tt][0], z4[tt][1], o.x, o.y);
                    radial_fwd(z4[tt][2], z4[tt][3], o.z, o.w);
                } else {
                    o.x = 1.f / (1.f + expf(-z4[tt][0]));  // S from output 4
                }
            }
            ((float4 *)(M.out + 8 * (size_t)row[tt]))[g] = o;
        }
    }
}

// ------------------------------------------------------------------ backward
// One kernel. A block of kBwdW wavefronts takes kBwdW tiles of 16 rows at a
// time. Each wavefront carries its own tile through the forward recompute
// (keeping GELU'(z) of every hidden unit and the bf16 activations), the output
// Jacobian and the gradient chain dH = W^T dZ, dZ = dH GELU'(z) on the matrix
// cores (transposed formulation, K order as in the forward). The weight
// gradients dW = dZ^T H contract over rows, so the block does them together:
// every wavefront leaves its rows' dZ and H of a layer in LDS as they stand
// ([row][unit], 16 bytes at a time), and each takes its share of the 16 x 16
// tiles of dW over all rows of the block, reading both operands through the
// transposing LDS load (ds_read_b64_tr_b16) 32 rows to an instruction. Bias
// gradients are one more such product, with ones. Embedding gradients are
// FP32 products of a one-hot label matrix and dX (v_mfma_f32_16x16x4_f32),
// straight from the registers. Every block writes its partials once; a
// fixed-order reduction over the blocks gives the gradients. The grid depends on
// the row count alone (at most kBwdBlocks), so the result does not depend on the device.
// Bound: the vector unit (GELU and GELU' of 192 units a row: about 25
// instructions and two transcendentals each). With the accumulators of all of
// dW in every wavefront (176 registers, one wavefront per SIMD) nothing hid
// the LDS and matrix-core latencies; shared over the block they take 40 registers
// and two wavefronts fit. Before, a wavefront's 2-byte transposes, bias sums
// and row-by-row embedding updates came on top, and 1 024 partials of 50 KB.
// 2^20 rows: 467 -> 276 us, the sums over partials 38 -> 10; 8 960 rows: 37 -> 22 us, 33 -> 9.
constexpr int kBwdW = 8;               // wavefronts per block
constexpr uint32_t kBwdBlocks = 256;   // one per CU
constexpr int kBwdRows = kBwdW * kTileRows;
constexpr int kLdH = 72;               // bf16 per LDS row (64 units + 16 B: spreads a transposing load's rows over the banks)
constexpr int kMaxLabels = 64;
// Weight fragments in LDS, fragment-major (fragment f, lane l at f * 64 + l,
// 16 B each): forward W1 (4), W2 (4 x 2), W3 (4 x 2), W4 (2); then for the
// chain W4^T (4; K = the 16 outputs, lane group g holds outputs 4 g .. 4 g + 3
// and zeros), W3^T (4 x 2), W2^T (4 x 2), W1^T rows 0..15 (2).
constexpr int kFF1 = 0, kFF2 = 4, kFF3 = 12, kFF4 = 20, kFB4 = 22, kFB3 = 26, kFB2 = 34, kFB1 = 42, kFrags = 44;
constexpr int kPartW = kWAll + kBAll;  // per-block partial: weights then biases, then the embedding table

typedef short s16x4 __attribute__((ext_vector_type(4)));

struct BwdShared {
    bf16x8 frag[kFrags * 64];
    float bias[kBAll];
    // dZ and H of the current layer, [row][unit] with the hidden units in the order the fragments hold them
    // (unit_of); two of each in turn, so that one barrier per layer is enough
    alignas(16) uint16_t dz[2][kBwdRows * kLdH], h[2][kBwdRows * kLdH];
};
static_assert(sizeof(float) * kBwdW * kMaxLabels * kEmb <= sizeof(BwdShared::dz), "the embedding tables reuse dz");

// Unit at LDS position s: fragment s / 32 of lane group (s / 8) % 4, element s % 8.
__device__ __forceinline__ int unit_of(int s) { return perm_k(s >> 5, (s >> 3) & 3, s & 7); }

__device__ __forceinline__ bf16x8 gather_frag(const uint16_t *W, int f, int lane) {
    // element j of lane's fragment f is W[base + row * ld + col]
    const int i = lane & 15, g = lane >> 4;
    u32x4 p;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * q + h;
            int row, col, base;
            bool zero = false;
            if (f < kFF2) { base = 0; row = 16 * (f - kFF1) + i; col = 8 * g + j; }
            else if (f < kFF3) { base = kW1; const int t = (f - kFF2) >> 1, ks = (f - kFF2) & 1; row = 16 * t + i; col = perm_k(ks, g, j); }
            else if (f < kFF4) { base = kW1 + kW2; const int t = (f - kFF3) >> 1, ks = (f - kFF3) & 1; row = 16 * t + i; col = perm_k(ks, g, j); }
            else if (f < kFB4) { base = kW1 + kW2 + kW3; row = i; col = perm_k(f - kFF4, g, j); }
            else if (f < kFB3) { base = kW1 + kW2 + kW3; row = 4 * g + (j & 3); col = 16 * (f - kFB4) + i; zero = j >= 4; }
            else if (f < kFB2) { base = kW1 + kW2; const int t = (f - kFB3) >> 1, ks = (f - kFB3) & 1; row = perm_k(ks, g, j); col = 16 * t + i; }
            else if (f < kFB1) { base = kW1; const int t = (f - kFB2) >> 1, ks = (f - kFB2) & 1; row = perm_k(ks, g, j); col = 16 * t + i; }
            else { base = 0; row = perm_k(f - kFB1, g, j); col = i; }
            const int ldw = base == 0 ? kIn : kHid;
            v[h] = zero ? 0u : (uint32_t)W[base + row * ldw + col];
        }
        p[q] = v[0] | (v[1] << 16);
    }
    return bf8_of(p);
}

// Operand of 32 rows x 16 units from LDS, transposed: lane (i, g) gets unit column 16 t + i of rows
// 32 kb + 16 h + 4 g + (0..3), h = 0, 1. Each group of 16 lanes reads 4 rows of 16 units, 8 bytes a lane.
// (Which row is which K does not matter, as both operands are read alike.)
typedef s16x4 __attribute__((address_space(3))) lds_s16x4;
__device__ __forceinline__ uint32_t get_t_lane(int lane) {  // the lane's part of the address
    const int i = lane & 15, g = lane >> 4;
    return (4 * g + (i >> 2)) * kLdH + 4 * (i & 3);
}
__device__ __forceinline__ bf16x8 get_t(const uint16_t *T, int t, int kb, uint32_t at) {
    const uint16_t *p = T + 32 * kb * kLdH + 16 * t + at;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 16 * kLdH));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ __launch_bounds__(64 * kBwdW) void k_mlp_backward(MlpArgs M) {
    __shared__ BwdShared S;
    for (int e = threadIdx.x; e < kFrags * 64; e += 64 * kBwdW) S.frag[e] = gather_frag(M.w, e / 64, e % 64);
    for (int e = threadIdx.x; e < kBAll; e += 64 * kBwdW) S.bias[e] = M.b[e];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 15,
              g = lane >> 4;
    __syncthreads();
    const bf16x8 *F = S.frag + lane;
    const float *B = S.bias + 4 * g;
    uint32_t at = 0;
    auto bias4 = [&](int off, int t) { return *(const f32x4 *)(B + off + 16 * t); };
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const bf16x8 ones = bf8_of(u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
    // This wavefront's share of dW: out tile oa; in tiles 2 ob, 2 ob + 1 of the hidden layers, ob of the first;
    // the last layer's in tile `wave` (wavefronts 0..3). The last layer's biases: wavefront 4.
    const int oa = wave >> 1, ob = wave & 1;
    f32x4 gw1 = zero, gw2[2] = {zero, zero}, gw3[2] = {zero, zero}, gw4 = zero;
    f32x4 gb1 = zero, gb2 = zero, gb3 = zero, gb4 = zero;
    f32x4 ge[kMaxLabels / 16];  // labels 16 t + 4 g + r, dimension n: this wavefront's rows
#pragma unroll
    for (int t = 0; t < kMaxLabels / 16; ++t) ge[t] = zero;
    // GELU and GELU' of a layer's outputs (C layout, bias included)
    auto layer = [&](const f32x4 (&acc)[4], bf16x8 (&h)[2], float (&gp)[16]) {
        float v[16];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float z = acc[t][r];
                float e;
                const float tail = norm_tail(z, e);
                v[4 * t + r] = fmaf(-fabsf(z), tail, relu(z));
                gp[4 * t + r] = fmaf(z * 0.39894228040143268f, e, z >= 0.f ? 1.0f - tail : tail);
            }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            h[ks] = bf8_of(u32x4{pack_bf2(v[8 * ks + 0], v[8 * ks + 1]), pack_bf2(v[8 * ks + 2], v[8 * ks + 3]),
                                 pack_bf2(v[8 * ks + 4], v[8 * ks + 5]), pack_bf2(v[8 * ks + 6], v[8 * ks + 7])});
    };
    // dZ = (W^T dZ_next) GELU'(z), rounded to bf16 (K order perm_k)
    auto chain = [&](int fb, const bf16x8 *src, int nks, const float (&gp)[16], bf16x8 (&out)[2]) {
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[t] = zero;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                if (ks < nks) acc[t] = MFMA16(F[64 * (fb + nks * t + ks)], src[ks], acc[t]);
        }
        float v[16];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[4 * t + r] = acc[t][r] * gp[4 * t + r];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            out[ks] = bf8_of(u32x4{pack_bf2(v[8 * ks + 0], v[8 * ks + 1]), pack_bf2(v[8 * ks + 2], v[8 * ks + 3]),
                                   pack_bf2(v[8 * ks + 4], v[8 * ks + 5]), pack_bf2(v[8 * ks + 6], v[8 * ks + 7])});
    };
    // this lane's row of a layer: 8 units of each fragment
    const int my_row = (wave * kTileRows + n) * kLdH;
    auto put = [&](uint16_t *T, const bf16x8 (&v)[2]) {
        *(bf16x8 *)(T + my_row + 8 * g) = v[0];
        *(bf16x8 *)(T + my_row + 32 + 8 * g) = v[1];
    };
    // dW and bias gradient of a hidden layer over the block's rows
    auto wgrad = [&](int p, f32x4 (&gw)[2], f32x4 &gb) {
#pragma unroll
        for (int kb = 0; kb < kBwdRows / 32; ++kb) {
            const bf16x8 av = get_t(S.dz[p], oa, kb, at);
#pragma unroll
            for (int b = 0; b < 2; ++b) gw[b] = MFMA16(av, get_t(S.h[p], 2 * ob + b, kb, at), gw[b]);
            gb = MFMA16(av, ones, gb);  // (by both wavefronts of an out tile: cheaper than a branch)
        }
    };
    const uint32_t n_tiles = (M.n + kTileRows - 1) / kTileRows;
    // every wavefront of the block goes through the barriers: one without a tile carries rows past the end
    for (uint32_t t0 = blockIdx.x * kBwdW; t0 < n_tiles; t0 += gridDim.x * kBwdW) {
        // weights and biases are read from LDS in every iteration: their addresses are made opaque, or the
        // compiler keeps all 57 of them in registers and spills the rest
        uint32_t fo = lane, bo = 4 * g;
        at = get_t_lane(lane);
        asm volatile("" : "+v"(fo), "+v"(bo), "+v"(at));
        F = S.frag + fo;
        B = S.bias + bo;
        const uint32_t row = (t0 + wave) * kTileRows + n;
        const bool has = t0 + wave < n_tiles && row < M.n;
        const uint16_t lab = has ? M.label[row] : (uint16_t)0xffff;
        const bool live = has && lab < M.n_labels;
        const bf16x8 x = input_frag(M, row, lab, g);
        bf16x8 h1[2], h2[2], h3[2];
        float gp1[16], gp2[16], gp3[16];
        f32x4 acc[4];
        // forward recompute
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = MFMA16(F[64 * (kFF1 + t)], x, bias4(0, t));
        layer(acc, h1, gp1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[t] = MFMA16(F[64 * (kFF2 + 2 * t + 1)], h1[1], MFMA16(F[64 * (kFF2 + 2 * t)], h1[0], bias4(kHid, t)));
        layer(acc, h2, gp2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[t] = MFMA16(F[64 * (kFF3 + 2 * t + 1)], h2[1], MFMA16(F[64 * (kFF3 + 2 * t)], h2[0], bias4(2 * kHid, t)));
        layer(acc, h3, gp3);
        __builtin_amdgcn_sched_barrier(0);
        const f32x4 z4 = MFMA16(F[64 * (kFF4 + 1)], h3[1],
                                MFMA16(F[64 * kFF4], h3[0], bias4(3 * kHid, 0)));
        // output Jacobian of live rows: outputs 0, 1 in lane group 0, 2, 3 in group 2 (one pass through the
        // same code), 4 in group 1
        const float z2 = __shfl(z4[2], n, kWave), z3 = __shfl(z4[3], n, kWave);
        float da = 0.f, db = 0.f;
        if (live && g < 3) {
            const float *go = M.gout + 8 * (size_t)row;
            if (g != 1) {
                float re, im, a, b, d;
                radial(g ? z2 : z4[0], g ? z3 : z4[1], re, im, a, b, d);
                da = go[g] * a + go[g + 1] * b;
                db = go[g] * b + go[g + 1] * d;
            } else {
                const float s4 = 1.f / (1.f + expf(-z4[0]));
                da = go[4] * s4 * (1.f - s4);
            }
        }
        const uint32_t dab = pack_bf2(da, db), dcd = __shfl(dab, 32 + n, kWave);
        const uint32_t d4lo = g < 2 ? dab : 0u, d4hi = g == 0 ? dcd : 0u;
        const bf16x8 d4 = bf8_of(u32x4{d4lo, d4hi, 0u, 0u});
        __builtin_amdgcn_sched_barrier(0);
        // layer 4: dZ4 (outputs 4 g + r) and H3
        *(uint2 *)(S.dz[0] + my_row + 4 * g) = make_uint2(d4lo, d4hi);
        put(S.h[0], h3);
        __syncthreads();
        if (wave < 4) {
#pragma unroll
            for (int kb = 0; kb < kBwdRows / 32; ++kb)
                gw4 = MFMA16(get_t(S.dz[0], 0, kb, at), get_t(S.h[0], wave, kb, at), gw4);
        } else if (wave == 4) {
#pragma unroll
            for (int kb = 0; kb < kBwdRows / 32; ++kb) gb4 = MFMA16(get_t(S.dz[0], 0, kb, at), ones, gb4);
        }
        // layer 3
        bf16x8 dz3[2], dz2[2], dz1[2];
        chain(kFB4, &d4, 1, gp3, dz3);
        put(S.dz[1], dz3);
        put(S.h[1], h2);
        __syncthreads();
        wgrad(1, gw3, gb3);
        __builtin_amdgcn_sched_barrier(0);
        // layer 2 (the barrier above: every wavefront is done with the first pair)
        chain(kFB3, dz3, 2, gp2, dz2);
        put(S.dz[0], dz2);
        put(S.h[0], h1);
        __syncthreads();
        wgrad(0, gw2, gb2);
        __builtin_amdgcn_sched_barrier(0);
        // layer 1 (H = the input: 32 features in natural order, element j of lane group g is feature 8 g + j)
        chain(kFB2, dz2, 2, gp1, dz1);
        put(S.dz[1], dz1);
        *(bf16x8 *)(S.h[1] + my_row + 8 * g) = x;
        // dX = dZ1 W1, embedding dimensions, untransposed: lane (n, g) holds dimension n of rows 4 g + r
        const f32x4 dx = MFMA16(dz1[1], F[64 * (kFB1 + 1)], MFMA16(dz1[0], F[64 * kFB1], zero));
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < kBwdRows / 32; ++kb) {
            const bf16x8 av = get_t(S.dz[1], oa, kb, at);
            gw1 = MFMA16(av, get_t(S.h[1], ob, kb, at), gw1);
            gb1 = MFMA16(av, ones, gb1);
        }
        // embedding gradient: dE[label][dim] += onehot[label][row] dX[row][dim], K = rows 4 g + r of step r
        uint32_t lr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lr[r] = __shfl(live ? (uint32_t)lab : 0xffffu, 4 * g + r, kWave);
        bool fin = true;
#pragma unroll
        for (int r = 0; r < 4; ++r) fin = fin && fabsf(dx[r]) < __builtin_inff();
        if (__all(fin)) {
#pragma unroll
            for (int t = 0; t < kMaxLabels / 16; ++t)
                if (16u * t < M.n_labels)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        ge[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(lr[r] == 16u * t + n ? 1.f : 0.f, dx[r], ge[t], 0, 0, 0);
        } else {  // 0 x infinity: a row's gradient must reach its own label only
            for (uint32_t L = 0; L < M.n_labels; ++L) {
                f32x4 d = zero;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    d = __builtin_amdgcn_mfma_f32_16x16x4f32(1.f, lr[r] == L ? dx[r] : 0.f, d, 0, 0, 0);
#pragma unroll
                for (int t = 0; t < kMaxLabels / 16; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (16u * t + 4 * g + r == L) ge[t][r] += d[r];
            }
        }
    }
    // partials: the weight gradients from the accumulators (C layout: lane
    // holds in position 16 b + n, out positions 16 a + 4 g + r), the biases'
    // (alike in every column), the embedding tables added in wavefront order
    float *P = M.part + (size_t)blockIdx.x * M.part_stride;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = unit_of(16 * oa + 4 * g + r);
        P[o * kIn + 16 * ob + n] = gw1[r];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int i = unit_of(16 * (2 * ob + b) + n);
            P[kW1 + o * kHid + i] = gw2[b][r];
            P[kW1 + kW2 + o * kHid + i] = gw3[b][r];
        }
        if (wave < 4) P[kW1 + kW2 + kW3 + (4 * g + r) * kHid + unit_of(16 * wave + n)] = gw4[r];
        if (ob == 0 && n == 0) {
            P[kWAll + o] = gb1[r];
            P[kWAll + kHid + o] = gb2[r];
            P[kWAll + 2 * kHid + o] = gb3[r];
        }
        if (wave == 4 && n == 0) P[kWAll + 3 * kHid + 4 * g + r] = gb4[r];
    }
    __syncthreads();  // done with dz and h
    float *E = (float *)S.dz;
#pragma unroll
    for (int t = 0; t < kMaxLabels / 16; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) E[wave * kMaxLabels * kEmb + (16 * t + 4 * g + r) * kEmb + n] = ge[t][r];
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < M.n_labels * kEmb; e += 64 * kBwdW) {
        float v = 0.f;
        for (int q = 0; q < kBwdW; ++q) v += E[q * kMaxLabels * kEmb + e];
        P[kPartW + e] = v;
    }
}

// Fixed-order sum of per-block partials, first stage: block (x, y) adds, for
// columns 64 x .. 64 x + 63, the partials of split y (kSumSplits contiguous
// ranges) -- each of its four wavefronts a quarter of the range in order,
// then the four in wavefront order -- into part2[y][column].
constexpr uint32_t kSumSplits = 16;
__global__ __launch_bounds__(256) void k_sum_parts_split(const float *part, uint32_t n_parts, uint32_t width,
                                                         uint32_t stride, float *part2) {
    __shared__ float red[4][64];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t i = blockIdx.x * 64 + lane;
    const uint32_t p0 = (uint32_t)((uint64_t)blockIdx.y * n_parts / kSumSplits);
    const uint32_t p1 = (uint32_t)((uint64_t)(blockIdx.y + 1) * n_parts / kSumSplits);
    const uint32_t b0 = p0 + (uint32_t)((uint64_t)wave * (p1 - p0) / 4);
    const uint32_t b1 = p0 + (uint32_t)((uint64_t)(wave + 1) * (p1 - p0) / 4);
    float s = 0.f;
    if (i < width)
        for (uint32_t b = b0; b < b1; ++b) s += part[(size_t)b * stride + i];
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && i < width)
        part2[(size_t)blockIdx.y * width + i] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// Second stage: the sum over the splits in order; column i goes to the weights',
// biases' or embedding table's gradient.
__global__ void k_sum_parts(const float *part2, uint32_t width, float *gw, float *gb, float *ge) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= width) return;
    float s = 0.f;
    for (uint32_t y = 0; y < kSumSplits; ++y) s += part2[(size_t)y * width + i];
    *(i < (uint32_t)kWAll ? gw + i : i < (uint32_t)kPartW ? gb + (i - kWAll) : ge + (i - kPartW)) = s;
}

}  // namespace pcrt

using namespace pcrt;

namespace {
struct MlpLayout {
    size_t part, part2, total;
    uint32_t stride;
};
// Per-block partials of the backward kernel (weights, biases, embedding
// table), then the first-stage sums of the fixed-order reduction.
MlpLayout mlp_layout(uint32_t n_labels) {
    Bump b;
    MlpLayout L;
    L.stride = kPartW + n_labels * kEmb;
    L.part = b.take(4ull * kBwdBlocks * L.stride);
    L.part2 = b.take(4ull * kSumSplits * L.stride);
    L.total = b.off;
    return L;
}
}  // namespace

extern "C" {

pcrt_status pcrt_mlp_workspace_size(uint32_t n, uint32_t n_labels, size_t *bytes) {
    if (!bytes) return PCRT_EINVAL;
    (void)n;  // the partials are per block of a bounded grid, not per row
    *bytes = mlp_layout(std::max<uint32_t>(n_labels, 1)).total;
    return PCRT_OK;
}

pcrt_status pcrt_mlp_forward(const pcrt_mlp *net, uint32_t n, const uint16_t *label, const float *cosv, float log_f,
                             float *out, void *stream) {
    if (!net || !net->w || !net->b || !net->emb || !label || !cosv || !out) return PCRT_EINVAL;
    if (n == 0) return PCRT_OK;
    MlpArgs M;
    memset(&M, 0, sizeof M);
    M.w = net->w;
    M.b = net->b;
    M.emb = net->emb;
    M.n_labels = net->n_labels;
    M.n = n;
    M.label = label;
    M.cosv = cosv;
    M.logf = log_f;
    M.out = out;
    const uint32_t tiles = (n + kTileRows - 1) / kTileRows;
    // One tile per wavefront while those fit the chip together: a wavefront's tiles run one after another. 8 960
    // rows: 24 us with 8 tiles (18 blocks), 12 us with 1 (140 blocks); at 2^20 rows
    // one tile at a time takes 153 us instead of 87.
    static const uint32_t cap1 = resident_blocks((const void *)k_mlp_forward<1>, 256);
    static const uint32_t cap = resident_blocks((const void *)k_mlp_forward<kFwdTiles>, 256);
    const bool few = tiles <= 4 * cap1;
    const uint32_t per = few ? 4 : 4 * kFwdTiles;
    const uint32_t grid = std::min<uint32_t>((tiles + per - 1) / per, few ? cap1 : cap);
    hipLaunchKernelGGL(few ? k_mlp_forward<1> : k_mlp_forward<kFwdTiles>, dim3(grid), dim3(256), 0, (hipStream_t)stream, M);
    return hipGetLastError() == hipSuccess ? PCRT_OK : PCRT_EDEVICE;
}

pcrt_status pcrt_mlp_backward(const pcrt_mlp *net, uint32_t n, const uint16_t *label, const float *cosv, float log_f,
                              const float *g_out, void *ws, size_t ws_bytes, float *grad_w, float *grad_b,
                              float *grad_emb, void *stream) {
    if (!net || !net->w || !net->b || !net->emb || !label || !cosv || !g_out || !ws || !grad_w || !grad_b || !grad_emb)
        return PCRT_EINVAL;
    if (n == 0) return PCRT_EINVAL;
    if (net->n_labels == 0 || net->n_labels > 64) return PCRT_EUNSUPPORTED;
    MlpLayout L = mlp_layout(net->n_labels);
    if (ws_bytes < L.total) return PCRT_ENOMEM;
    char *w = (char *)ws;
    hipStream_t s = (hipStream_t)stream;
    MlpArgs M;
    memset(&M, 0, sizeof M);
    M.w = net->w;
    M.b = net->b;
    M.emb = net->emb;
    M.n_labels = net->n_labels;
    M.n = n;
    M.label = label;
    M.cosv = cosv;
    M.logf = log_f;
    M.gout = g_out;
    M.part = (float *)(w + L.part);
    M.part_stride = L.stride;
    float *part2 = (float *)(w + L.part2);
    const uint32_t tiles = (n + kTileRows - 1) / kTileRows, n_parts = std::min(kBwdBlocks, (tiles + kBwdW - 1) / kBwdW);
    hipLaunchKernelGGL(k_mlp_backward, dim3(n_parts), dim3(64 * kBwdW), 0, s, M);
    // all columns at once (a pair of launches each for weights, biases and table took twice the time)
    hipLaunchKernelGGL(k_sum_parts_split, dim3((L.stride + 63) / 64, kSumSplits), dim3(256), 0, s, M.part, n_parts,
                       L.stride, L.stride, part2);
    hipLaunchKernelGGL(k_sum_parts, dim3((L.stride + 255) / 256), dim3(256), 0, s, part2, L.stride, grad_w, grad_b,
                       grad_emb);
    return hipGetLastError() == hipSuccess ? PCRT_OK : PCRT_EDEVICE;
}

}  // extern "C"
