// Learned particle initialisation: a small MLP maps a summary of the
// previous step's particle set and the new observation to a K-component
// diagonal Gaussian mixture, from which the N initial particles of the step
// are drawn (the predictive initialisation stays the fallback).  The
// proposal is trained on converged particle sets the method produces, by the
// mixture negative log-likelihood.  GEMMs take BF16 operands and accumulate
// in FP32 on the matrix cores (v_mfma_f32_16x16x16bf16_1k).
//
// Features (64, zero padded), with a = f_t(x_{t-1}^{best}), best the lowest
// argmax of the previous forward-recursion scores, M_j = f_t(x_{t-1}^j) and
// s = sqrt(q):
//   [0..3]   family one-hot
//   [4]      ln(n) / 7
//   [5..11]  (mean_j M_j - a) / s
//   [12..18] ln(var_j M_j / s^2 + 1e-6) / 8
//   [19..25] asinh(s * grad_x log p(z_t | a)) / 4
//   [26]     asinh(log p(z_t | a)) / 8
//   [27..63] zero
// (entries k >= d of each per-dimension block are zero).  No feature holds
// the absolute position: the mixture is placed relative to a.
// Outputs (120 = 8 x 15): component c has logit o[15c], mean offsets
// o[15c + 1 + k] and log-scales o[15c + 8 + k]: mean a + s mu, standard
// deviation s exp(clamp(rho, -7, 3)) per dimension k < d.
#pragma once

#include "smsq_batch.hpp"

namespace smsq {

constexpr int kInitFeat = 64;
constexpr int kInitHidden = 256;
constexpr int kInitK = 8;
constexpr int kInitComp = 15;                    // logit + 7 means + 7 log-scales
constexpr int kInitOut = kInitK * kInitComp;     // 120
constexpr int kInitOutPad = 128;
constexpr float kRhoMin = -7.f, kRhoMax = 3.f;
// flattened FP32 parameters: W1 [256][64], b1, W2 [256][256], b2, W3 [120][256], b3
constexpr long kOffW1 = 0;
constexpr long kOffB1 = kOffW1 + (long)kInitHidden * kInitFeat;
constexpr long kOffW2 = kOffB1 + kInitHidden;
constexpr long kOffB2 = kOffW2 + (long)kInitHidden * kInitHidden;
constexpr long kOffW3 = kOffB2 + kInitHidden;
constexpr long kOffB3 = kOffW3 + (long)kInitOut * kInitHidden;
constexpr long kInitParams = kOffB3 + kInitOut;  // 113,272

typedef short bf16x4 __attribute__((ext_vector_type(4)));

// round to nearest even; NaN stays NaN
__host__ __device__ inline uint16_t to_bf16(float f)
{
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__host__ __device__ inline float from_bf16(uint16_t h)
{
    const uint32_t u = (uint32_t)h << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

// One example of the proposal: a sequence step (training: `target` holds the
// converged particles; sampling: the initial particles are written there).
struct InitExample {
    DevModel<float> m;
    const float *xprev;     // [np][d]
    const float *phiprev;   // [np] or null (all equal)
    const float *z;         // [obs_dim]
    const uint8_t *mask;    // [n_obs] or null
    float *target;          // [n][d]
    int np, n, t, code, seq;
    uint64_t seed;
};

// Features of examples [0, count): one wave each.  Also the anchor a and
// scale s per example ([8] each).
template <int KIND, int D>
__device__ void init_features_one(const InitExample &e, float *F, uint16_t *Fb, float *anc, float *scl)
{
    using Fm = Family<float, KIND, D>;
    const int lane = threadIdx.x & 63;
    // best previous particle: lowest index among the maxima
    ArgBest<float> ab{-__builtin_huge_valf(), -__builtin_huge_valf(), 0x7fffffff};
    for (int j = lane; j < e.np; j += kWave) {
        const float v = e.phiprev ? e.phiprev[j] : 0.f;
        if (j == lane) { ab.best = v; ab.arg = j; }
        else argbest_push(ab, v, j);
    }
    ab = wave_argbest(ab);
    const int best = ab.arg < e.np ? ab.arg : 0;
    float a[D], xb[D];
#pragma unroll
    for (int k = 0; k < D; ++k) xb[k] = e.xprev[(long)best * D + k];
    Fm::mean(e.m, e.t, xb, a);
    // moments of the propagated set (two passes for the variance)
    float mu[D], var[D];
#pragma unroll
    for (int k = 0; k < D; ++k) mu[k] = 0.f;
    for (int j = lane; j < e.np; j += kWave) {
        float x[D], mj[D];
#pragma unroll
        for (int k = 0; k < D; ++k) x[k] = e.xprev[(long)j * D + k];
        Fm::mean(e.m, e.t, x, mj);
#pragma unroll
        for (int k = 0; k < D; ++k) mu[k] += mj[k];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) mu[k] = wave_sum(mu[k]) / (float)e.np;
#pragma unroll
    for (int k = 0; k < D; ++k) var[k] = 0.f;
    for (int j = lane; j < e.np; j += kWave) {
        float x[D], mj[D];
#pragma unroll
        for (int k = 0; k < D; ++k) x[k] = e.xprev[(long)j * D + k];
        Fm::mean(e.m, e.t, x, mj);
#pragma unroll
        for (int k = 0; k < D; ++k) var[k] += (mj[k] - mu[k]) * (mj[k] - mu[k]);
    }
#pragma unroll
    for (int k = 0; k < D; ++k) var[k] = wave_sum(var[k]) / (float)e.np;
    float g[D];
    Fm::grad(e.m, e.z, e.mask, a, g);
    const float ll = Fm::loglik(e.m, e.z, e.mask, a);
    // lane f writes feature f; none holds the absolute position (offsets
    // from the anchor, spreads and the likelihood around it only)
    float v = 0.f;
    const int f = lane;
    if (f < 4) v = f == KIND ? 1.f : 0.f;
    else if (f == 4) v = logf((float)e.n) / 7.f;
    else if (f == 26) v = asinhf(ll) / 8.f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const float s = e.m.sqrt_q[k];
        if (f == 5 + k) v = (mu[k] - a[k]) / s;
        if (f == 12 + k) v = logf(var[k] / (s * s) + 1e-6f) / 8.f;
        if (f == 19 + k) v = asinhf(s * g[k]) / 4.f;
    }
    F[f] = v;
    Fb[f] = to_bf16(v);
    if (lane < 8) {
        float av = 0.f, sv = 1.f;
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (lane == k) { av = a[k]; sv = e.m.sqrt_q[k]; }
        anc[lane] = av;
        scl[lane] = sv;
    }
}

__global__ __launch_bounds__(64) void k_init_features(const InitExample *__restrict__ ex, int count,
                                                      float *F, uint16_t *Fb, float *anc, float *scl)
{
    const int e = blockIdx.x;
    if (e >= count) return;
    const InitExample &x = ex[e];
    float *f = F + (long)e * kInitFeat;
    uint16_t *fb = Fb + (long)e * kInitFeat;
    switch (x.code) {
    case GROWTH1D: init_features_one<GROWTH1D, 1>(x, f, fb, anc + e * 8, scl + e * 8); break;
    case RANGE2D: init_features_one<RANGE2D, 2>(x, f, fb, anc + e * 8, scl + e * 8); break;
    case CV4D: init_features_one<CV4D, 4>(x, f, fb, anc + e * 8, scl + e * 8); break;
    default: init_features_one<ARM7, 7>(x, f, fb, anc + e * 8, scl + e * 8); break;
    }
}

// ---- the network's products ----
// A wave forms 16x16 tiles of a product, 16 of the inner index per MFMA, in
// order.  Operand layout of v_mfma_f32_16x16x16bf16_1k: lane l gives A[l %
// 16][4 (l / 16) + j] and B[4 (l / 16) + j][l % 16], j = 0..3; result register
// r of lane l is C[4 (l / 16) + r][l % 16].  Every operand lies with its inner
// index contiguous, so that a lane reads its four values as one 8-byte word:
// activations and gradients are kept transposed ([feature][row], a result
// tile's lane holds four rows of one feature), W2 and W3 in both orders.
// Read through strides, 2 bytes at a time with each load waited for, the
// products of 512 examples took 7 to 18 us each, and the bias sums, one serial
// thread per feature, 84 to 106 us; a training step of 512 examples of 256
// particles 547 us in 15 launches, now 90 us in 5 (8.5 us of it features, 22
// forward, 14 likelihood, 17 data and 10 weight gradients with Adam).
constexpr int kMlpRows = 16;                    // rows (examples) of a workgroup
constexpr int kMlpStride = kInitHidden + 8;     // of a row's bf16 in LDS
constexpr int kInitBias = kInitOut + 2 * kInitHidden;

__device__ __forceinline__ bf16x4 load_bf16x4(const uint16_t *p) { return *(const bf16x4 *)p; }
__device__ __forceinline__ bf16x4 pack_bf16x4(const float (&v)[4])
{
    return bf16x4{(short)to_bf16(v[0]), (short)to_bf16(v[1]), (short)to_bf16(v[2]), (short)to_bf16(v[3])};
}

// Forward of 16 rows per workgroup, one tile column per wave: the three layers
// need no other row, so nothing but the saved pre-activations and the
// transposed activations leaves the workgroup, and the weights of all layers
// are in flight before the first product.
__global__ __launch_bounds__(1024) void k_mlp_forward(int B, const uint16_t *__restrict__ Fb,
                                                      const uint16_t *__restrict__ w1b,
                                                      const uint16_t *__restrict__ w2b,
                                                      const uint16_t *__restrict__ w3b, const float *__restrict__ P,
                                                      float *pre1, float *pre2, float *out, uint16_t *FbT,
                                                      uint16_t *h1T, uint16_t *h2T, long ldT)
{
    constexpr int H = kInitHidden;
    __shared__ __align__(16) uint16_t h1[kMlpRows * kMlpStride], h2[kMlpRows * kMlpStride];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    const int b0 = blockIdx.x * kMlpRows, n = wave * 16 + col;
    const bool last = n < kInitOutPad;          // (W3's rows 120..127 are zero)
    bf16x4 w1[kInitFeat / 16], w2[H / 16], w3[H / 16];
    bf16x4 x[kInitFeat / 16];
    const int row = min(b0 + col, B - 1);       // (a row past the batch: its results go nowhere)
#pragma unroll
    for (int k = 0; k < kInitFeat / 16; ++k) {
        x[k] = load_bf16x4(Fb + (long)row * kInitFeat + 16 * k + 4 * g);
        w1[k] = load_bf16x4(w1b + n * kInitFeat + 16 * k + 4 * g);
    }
#pragma unroll
    for (int k = 0; k < H / 16; ++k) w2[k] = load_bf16x4(w2b + n * H + 16 * k + 4 * g);
#pragma unroll
    for (int k = 0; k < H / 16; ++k) w3[k] = load_bf16x4(w3b + (last ? n : 0) * H + 16 * k + 4 * g);
    // hidden layer: pre = acc + bias, relu(pre) as bf16 to LDS and transposed
    // (rows past the batch as zeros)
    auto hidden = [&](const f32x4 &acc, float bias, float *pre, uint16_t *h, uint16_t *hT) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = b0 + 4 * g + r;
            const float p = acc[r] + bias;
            if (m < B) pre[(long)m * H + n] = p;
            v[r] = m < B && p > 0.f ? p : 0.f;
        }
        const bf16x4 q = pack_bf16x4(v);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[(4 * g + r) * kMlpStride + n] = (uint16_t)q[r];
        *(bf16x4 *)(hT + n * ldT + b0 + 4 * g) = q;
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kInitFeat / 16; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x[k], w1[k], acc, 0, 0, 0);
    hidden(acc, P[kOffB1 + n], pre1, h1, h1T);
    if (threadIdx.x < 4 * kInitFeat) {          // the features transposed
        const int f = threadIdx.x >> 2, r0 = 4 * (threadIdx.x & 3);
        bf16x4 q;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = b0 + r0 + r;
            q[r] = m < B ? (short)Fb[(long)m * kInitFeat + f] : (short)0;
        }
        *(bf16x4 *)(FbT + f * ldT + b0 + r0) = q;
    }
    __syncthreads();
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(load_bf16x4(h1 + col * kMlpStride + 16 * k + 4 * g), w2[k],
                                                        acc, 0, 0, 0);
    hidden(acc, P[kOffB2 + n], pre2, h2, h2T);
    __syncthreads();
    if (!last) return;
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(load_bf16x4(h2 + col * kMlpStride + 16 * k + 4 * g), w3[k],
                                                        acc, 0, 0, 0);
    if (n >= kInitOut) return;
    const float bias = P[kOffB3 + n];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = b0 + 4 * g + r;
        if (m < B) out[(long)m * kInitOut + n] = acc[r] + bias;
    }
}

// Data gradients of 16 rows per workgroup, likewise, through both ReLUs: the
// transposed bf16 gradients of the three layers' outputs, and the workgroup's
// share of the bias gradients (FP32 sums over its rows of the unrounded
// values), part[workgroup][b3 | b2 | b1].
__global__ __launch_bounds__(1024) void k_mlp_backward(int B, const float *__restrict__ dout,
                                                       const uint16_t *__restrict__ w2t,
                                                       const uint16_t *__restrict__ w3t,
                                                       const float *__restrict__ pre1, const float *__restrict__ pre2,
                                                       uint16_t *doutT, uint16_t *d2T, uint16_t *d1T, float *part,
                                                       long ldT)
{
    constexpr int H = kInitHidden, O = kInitOut;
    __shared__ __align__(16) uint16_t d2[kMlpRows * kMlpStride];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    const int b0 = blockIdx.x * kMlpRows, n = wave * 16 + col;
    float *share = part + (long)blockIdx.x * kInitBias;
    bf16x4 x[kInitOutPad / 16], w3[kInitOutPad / 16], w2[H / 16];
    const int row = min(b0 + col, B - 1);
#pragma unroll
    for (int k = 0; k < kInitOutPad / 16; ++k) {
        const int o = 16 * k + 4 * g;
        x[k] = bf16x4{0, 0, 0, 0};
        if (o < O) {
            const f32x4 v = *(const f32x4 *)(dout + (long)row * O + o);
            x[k] = pack_bf16x4({v[0], v[1], v[2], v[3]});
        }
        w3[k] = load_bf16x4(w3t + n * kInitOutPad + o);
    }
#pragma unroll
    for (int k = 0; k < H / 16; ++k) w2[k] = load_bf16x4(w2t + n * H + 16 * k + 4 * g);
    float m1[4], m2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = b0 + 4 * g + r;
        m1[r] = m < B ? pre1[(long)m * H + n] : 0.f;
        m2[r] = m < B ? pre2[(long)m * H + n] : 0.f;
    }
    // through a ReLU
    auto gradient = [&](const f32x4 &acc, const float (&pre)[4], uint16_t *dT, float *db) {
        float v[4], s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = pre[r] > 0.f ? acc[r] : 0.f;
            s += v[r];
        }
        const bf16x4 q = pack_bf16x4(v);
        *(bf16x4 *)(dT + n * ldT + b0 + 4 * g) = q;
        s += __shfl_xor(s, 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (g == 0) db[n] = s;
        return q;
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kInitOutPad / 16; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x[k], w3[k], acc, 0, 0, 0);
    const bf16x4 q = gradient(acc, m2, d2T, share + O);
#pragma unroll
    for (int r = 0; r < 4; ++r) d2[(4 * g + r) * kMlpStride + n] = (uint16_t)q[r];
    if (threadIdx.x < 4 * O) {
        const int o = threadIdx.x >> 2, r0 = 4 * (threadIdx.x & 3);
        float v[4], s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = b0 + r0 + r;
            v[r] = m < B ? dout[(long)m * O + o] : 0.f;
            s += v[r];
        }
        *(bf16x4 *)(doutT + o * ldT + b0 + r0) = pack_bf16x4(v);
        s += __shfl_xor(s, 1, kWave);
        s += __shfl_xor(s, 2, kWave);
        if (r0 == 0) share[o] = s;
    }
    __syncthreads();
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < H / 16; ++k)
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(load_bf16x4(d2 + col * kMlpStride + 16 * k + 4 * g), w2[k],
                                                        acc, 0, 0, 0);
    gradient(acc, m1, d1T, share + O + H);
}

// The parameters, their gradients and the bf16 copies of the weights: W1, W2,
// W3 as [out][in] (W3 padded to 128 rows; rows 120..127 stay zero), and W2, W3
// as [in][out].
struct MlpParams {
    float *P, *G, *mo, *ve;
    uint16_t *w1b, *w2b, *w3b, *w2t, *w3t;
};
// Adam's constants; c1 = 1 / (1 - b1^t) and c2 = 1 / (1 - b2^t) are the bias
// corrections of step t, computed by the host in FP64 (in FP32, 1 - b2^t
// cancels: relative error ~3e-5 at t = 2).
struct AdamStep { float lr, b1, b2, eps, c1, c2; };

// Parameter i after a step with gradient g
__device__ __forceinline__ float adam_update(const MlpParams &q, const AdamStep &a, long i, float g)
{
    const float m = a.b1 * q.mo[i] + (1.f - a.b1) * g;
    const float v = a.b2 * q.ve[i] + (1.f - a.b2) * g * g;
    q.mo[i] = m;
    q.ve[i] = v;
    const float mh = m * a.c1, vh = v * a.c2;
    const float p = q.P[i] - a.lr * mh / (sqrtf(vh) + a.eps);
    q.P[i] = p;
    return p;
}

// Weight gradients, one tile per one-wave workgroup (448), each over all rows
// of the batch: enough waves for the chip without splitting the sum.  Then a
// workgroup per 64 bias gradients, summed over the rows' workgroups, and the
// mean of the losses.  A training step applies Adam to what a lane holds
// (`train`), so that the gradients are not read again.
constexpr int kGradTiles1 = kInitHidden / 16 * (kInitFeat / 16);
constexpr int kGradTiles2 = kInitHidden / 16 * (kInitHidden / 16);
constexpr int kGradTiles3 = kInitOutPad / 16 * (kInitHidden / 16);
constexpr int kGradTiles = kGradTiles1 + kGradTiles2 + kGradTiles3;
constexpr int kGradBias = (kInitBias + 63) / 64;
__global__ __launch_bounds__(64) void k_mlp_grad(int B, const uint16_t *__restrict__ FbT,
                                                 const uint16_t *__restrict__ h1T, const uint16_t *__restrict__ h2T,
                                                 const uint16_t *__restrict__ d1T, const uint16_t *__restrict__ d2T,
                                                 const uint16_t *__restrict__ doutT, const float *__restrict__ part,
                                                 const float *__restrict__ loss, float *mean_loss, long ldT,
                                                 MlpParams q, AdamStep adam, int train)
{
    constexpr int H = kInitHidden;
    const int lane = threadIdx.x, g = lane >> 4, col = lane & 15;
    int tile = blockIdx.x;
    if (tile == kGradTiles + kGradBias) {
        float s = 0.f;
        for (int i = lane; i < B; i += kWave) s += loss[i];
        s = wave_sum(s);
        if (lane == 0) mean_loss[0] = s / (float)B;
        return;
    }
    if (tile >= kGradTiles) {
        const int c = (tile - kGradTiles) * kWave + lane;
        if (c >= kInitBias) return;
        const int nb = (B + kMlpRows - 1) / kMlpRows;
        float s = 0.f;
#pragma unroll 8
        for (int k = 0; k < nb; ++k) s += part[(long)k * kInitBias + c];
        const long i = c < kInitOut ? kOffB3 + c : c < kInitOut + H ? kOffB2 + (c - kInitOut) : kOffB1 + (c - kInitOut - H);
        q.G[i] = s;
        if (train) adam_update(q, adam, i, s);
        return;
    }
    const uint16_t *A, *Bm;
    int rows = H, cols = H;
    long off = kOffW2;
    if (tile < kGradTiles1) {
        A = d1T; Bm = FbT; cols = kInitFeat; off = kOffW1;
    } else if (tile < kGradTiles1 + kGradTiles2) {
        tile -= kGradTiles1;
        A = d2T; Bm = h1T;
    } else {
        tile -= kGradTiles1 + kGradTiles2;
        A = doutT; Bm = h2T; rows = kInitOut; off = kOffW3;
    }
    const int tn = cols / 16, m0 = tile / tn * 16, n = tile % tn * 16 + col;
    // (past the outputs' rows: the last one, and nothing is stored)
    const uint16_t *pa = A + min(m0 + col, rows - 1) * ldT + 4 * g, *pb = Bm + n * ldT + 4 * g;
    constexpr int kDepth = 8;   // steps in flight behind the ones being multiplied
    const int steps = (B + 15) / 16;
    bf16x4 a[kDepth], b[kDepth];
    auto fetch = [&](int k, bf16x4 &av, bf16x4 &bv) {
        const int at = 16 * min(k, steps - 1);
        av = load_bf16x4(pa + at);
        bv = load_bf16x4(pb + at);
    };
#pragma unroll
    for (int u = 0; u < kDepth; ++u) fetch(u, a[u], b[u]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + kDepth < steps; k += kDepth) {
        bf16x4 an[kDepth], bn[kDepth];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) fetch(k + kDepth + u, an[u], bn[u]);
#pragma unroll
        for (int u = 0; u < kDepth; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[u], b[u], acc, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            a[u] = an[u];
            b[u] = bn[u];
        }
    }
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
        if (k + u >= steps) break;
        // rows past the batch count nothing, whatever an earlier pass left there
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (16 * (k + u) + 4 * g + j >= B) a[u][j] = b[u][j] = 0;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[u], b[u], acc, 0, 0, 0);
    }
    const int m = m0 + 4 * g;
    if (m >= rows) return;   // (a multiple of four)
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const long i = off + (long)(m + r) * cols + n;
        q.G[i] = acc[r];
        p[r] = train ? adam_update(q, adam, i, acc[r]) : 0.f;
    }
    if (!train) return;
    const bf16x4 w = pack_bf16x4(p);
    uint16_t *wb = off == kOffW1 ? q.w1b : off == kOffW2 ? q.w2b : q.w3b;
#pragma unroll
    for (int r = 0; r < 4; ++r) wb[(m + r) * cols + n] = (uint16_t)w[r];
    if (off == kOffW2) *(bf16x4 *)(q.w2t + n * H + m) = w;
    if (off == kOffW3) *(bf16x4 *)(q.w3t + n * kInitOutPad + m) = w;
}

__global__ void k_to_bf16(const float *__restrict__ src, uint16_t *dst, long count)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = to_bf16(src[i]);
}

// Mixture NLL of each example's target particles and its gradient with
// respect to the 120 outputs (scaled by gscale).  A workgroup per example, one
// wave per component: the waves exchange the components' log densities of 256
// particles at a time, and each reduces its own 15 sums (one wave for all 120
// of them, 56 of each kind in registers, took 36 us for 512 examples of 256
// particles).
constexpr int kNllChunk = 256;
__global__ __launch_bounds__(64 * kInitK) void k_mix_nll(const InitExample *__restrict__ ex, int count,
                                                         const float *__restrict__ out, const float *__restrict__ anc,
                                                         const float *__restrict__ scl, float *dout, float *loss,
                                                         float gscale)
{
    __shared__ float slc[kInitK][kNllChunk];
    const int e = blockIdx.x;
    if (e >= count) return;
    const int lane = threadIdx.x & 63, c = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const InitExample &x = ex[e];
    const int d = x.m.d, n = x.n;
    const float *o = out + (long)e * kInitOut;
    float s[7], mean[7], isd[7], lsd[7];  // of this component: mean, 1 / sd, log sd
    bool rin[7];
    float lmax = -__builtin_huge_valf();
#pragma unroll
    for (int q = 0; q < kInitK; ++q) lmax = fmaxf(lmax, o[q * kInitComp]);
    float lse = 0.f;
#pragma unroll
    for (int q = 0; q < kInitK; ++q) lse += expf(o[q * kInitComp] - lmax);
    lse = lmax + logf(lse);
    const float pl = o[c * kInitComp] - lse;  // log pi_c
    const float pc = expf(pl);
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const float a = anc[e * 8 + k];
        s[k] = scl[e * 8 + k];
        const float r = o[c * kInitComp + 8 + k];
        rin[k] = r >= kRhoMin && r <= kRhoMax;
        const float rc = fminf(fmaxf(r, kRhoMin), kRhoMax);
        mean[k] = a + s[k] * o[c * kInitComp + 1 + k];
        isd[k] = 1.f / (s[k] * expf(rc));
        lsd[k] = logf(s[k]) + rc;
    }
    float gl = 0.f, gm[7], gr[7], lsum = 0.f;
#pragma unroll
    for (int k = 0; k < 7; ++k) gm[k] = gr[k] = 0.f;
    const float hl2pi = 0.91893853320467274178f;
    constexpr int kPer = kNllChunk / kWave;
    for (int i0 = 0; i0 < n; i0 += kNllChunk) {
        float u[kPer][7], lc[kPer];
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const int i = i0 + t * kWave + lane;
            float v = pl;
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                u[t][k] = 0.f;
                if (k < d && i < n) {
                    u[t][k] = (x.target[(long)i * d + k] - mean[k]) * isd[k];
                    v += -0.5f * u[t][k] * u[t][k] - lsd[k] - hl2pi;
                }
            }
            lc[t] = v;
            slc[c][t * kWave + lane] = v;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            if (i0 + t * kWave + lane >= n) continue;
            float mx = -__builtin_huge_valf(), l[kInitK];
#pragma unroll
            for (int q = 0; q < kInitK; ++q) {
                l[q] = slc[q][t * kWave + lane];
                mx = fmaxf(mx, l[q]);
            }
            float se = 0.f;
#pragma unroll
            for (int q = 0; q < kInitK; ++q) se += expf(l[q] - mx);
            const float lse_i = mx + logf(se);
            lsum += -lse_i;
            const float r = expf(lc[t] - lse_i);  // responsibility
            gl += -(r - pc);
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                if (k < d) {
                    gm[k] += -r * u[t][k] * isd[k] * s[k];
                    gr[k] += -r * (u[t][k] * u[t][k] - 1.f);
                }
            }
        }
        __syncthreads();
    }
    const float w = gscale / (float)n;
    float *go = dout + (long)e * kInitOut + c * kInitComp;
    const float v = wave_sum(gl);
    if (lane == 0) go[0] = v * w;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const float vm = wave_sum(gm[k]);
        const float vr = wave_sum(gr[k]);
        if (lane == 0) {
            go[1 + k] = vm * w;
            go[8 + k] = rin[k] ? vr * w : 0.f;
        }
    }
    if (c == 0) {
        lsum = wave_sum(lsum);
        if (lane == 0) loss[e] = lsum / (float)n;
    }
}

// Draws each example's n particles from its mixture into `target`:
// component from one uniform by the cumulative weights, standard normals by
// Box-Muller, uniforms from Philox4x32-10 keyed by the example seed with
// counter (i, t, seq, 2 + b), b = 0, 1, 2.  Non-finite outputs: used[e] = 0
// and nothing is written (the predictive initialisation applies).
template <int D>
__device__ void mix_sample_one(const InitExample &x, int i, const float *o, const float *anc, const float *scl)
{
    float lmax = -__builtin_huge_valf();
    for (int c = 0; c < kInitK; ++c) lmax = fmaxf(lmax, o[c * kInitComp]);
    float w[kInitK], tot = 0.f;
    for (int c = 0; c < kInitK; ++c) {
        w[c] = expf(o[c * kInitComp] - lmax);
        tot += w[c];
    }
    const uint32_t k0 = (uint32_t)x.seed, k1 = (uint32_t)(x.seed >> 32);
    double u[12];
    for (int b = 0; b < 3; ++b) {
        const U4 r = philox4x32_10(U4{(uint32_t)i, (uint32_t)x.t, (uint32_t)x.seq, 2u + (uint32_t)b}, k0, k1);
        u[4 * b + 0] = ((double)r.x + 0.5) * (1.0 / 4294967296.0);
        u[4 * b + 1] = ((double)r.y + 0.5) * (1.0 / 4294967296.0);
        u[4 * b + 2] = ((double)r.z + 0.5) * (1.0 / 4294967296.0);
        u[4 * b + 3] = ((double)r.w + 0.5) * (1.0 / 4294967296.0);
    }
    const float uc = (float)u[0] * tot;
    int c = kInitK - 1;
    float acc = 0.f;
    for (int q = 0; q < kInitK; ++q) {
        acc += w[q];
        if (uc < acc) { c = q; break; }
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const int p = k / 2;
        const double rad = sqrt(-2.0 * log(u[2 + 2 * p]));
        const double th = 2.0 * kPi * u[3 + 2 * p];
        const float xi = (float)((k & 1) ? rad * sin(th) : rad * cos(th));
        const float rho = fminf(fmaxf(o[c * kInitComp + 8 + k], kRhoMin), kRhoMax);
        x.target[(long)i * D + k] = anc[k] + scl[k] * (o[c * kInitComp + 1 + k] + expf(rho) * xi);
    }
}

__global__ __launch_bounds__(256) void k_mix_sample(const InitExample *__restrict__ ex, int count,
                                                    const float *__restrict__ out, const float *__restrict__ anc,
                                                    const float *__restrict__ scl, int32_t *used)
{
    const int e = blockIdx.y;
    if (e >= count) return;
    const InitExample &x = ex[e];
    const float *o = out + (long)e * kInitOut;
    bool ok = true;
    for (int q = 0; q < kInitOut; ++q) ok &= __builtin_isfinite(o[q]);
    if (blockIdx.x == 0 && threadIdx.x == 0 && used) used[e] = ok ? 1 : 0;
    if (!ok) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= x.n) return;
    const float *a = anc + e * 8, *sc = scl + e * 8;
    switch (x.code) {
    case GROWTH1D: mix_sample_one<1>(x, i, o, a, sc); break;
    case RANGE2D: mix_sample_one<2>(x, i, o, a, sc); break;
    case CV4D: mix_sample_one<4>(x, i, o, a, sc); break;
    default: mix_sample_one<7>(x, i, o, a, sc); break;
    }
}

// Example table of a batch plan's step t: sequence list[k] proposes its
// step-t particles from step t - 1.
__global__ void k_init_prep(const SeqDesc *__restrict__ seqs, const int *__restrict__ list, int count, int t,
                            InitExample *__restrict__ ex)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const SeqDesc &s = seqs[list[k]];
    InitExample x;
    x.m = s.m;
    const long nd = (long)s.n * s.d;
    x.xprev = s.parts + (long)(t - 2) * nd;
    x.phiprev = s.phis + (long)(t - 2) * s.n;
    x.z = s.z + (long)(t - 1) * s.m.obs_dim;
    x.mask = s.mask ? s.mask + (long)(t - 1) * s.m.n_obs : nullptr;
    x.target = s.parts + (long)(t - 1) * nd;
    x.np = s.n;
    x.n = s.use_proposal ? s.n : 0;  // nothing to draw for the others
    x.t = t;
    x.code = s.code;
    x.seq = 0;
    x.seed = s.seed;
    ex[k] = x;
}

// After sampling: the step's items take the sampled particles (init_given)
// where a sequence uses the proposal and its outputs were finite.
__global__ void k_init_apply(StepArgs<float> *items, const InitExample *__restrict__ ex,
                             const int32_t *__restrict__ used, int count)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) items[k].init_given = ex[k].n > 0 ? used[k] : 0;
}

// He initialisation: W ~ N(0, 2 / fan_in) from Philox4x32-10 (key seed,
// counter (i, 0, 0x696e6974, 0)) and Box-Muller; biases zero.
__global__ void k_init_he(float *P, uint64_t seed)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kInitParams) return;
    float fan = 0.f;
    if (i < kOffB1) fan = (float)kInitFeat;
    else if (i >= kOffW2 && i < kOffB2) fan = (float)kInitHidden;
    else if (i >= kOffW3 && i < kOffB3) fan = (float)kInitHidden;
    if (fan == 0.f) {
        P[i] = 0.f;
        return;
    }
    const U4 r = philox4x32_10(U4{(uint32_t)i, 0u, 0x696e6974u, 0u}, (uint32_t)seed, (uint32_t)(seed >> 32));
    const double u1 = ((double)r.x + 0.5) * (1.0 / 4294967296.0), u2 = ((double)r.y + 0.5) * (1.0 / 4294967296.0);
    P[i] = (float)(sqrt(-2.0 * log(u1)) * cos(2.0 * kPi * u2) * sqrt(2.0 / fan));
}

// BF16 copies of the weight matrices from the FP32 parameters
__global__ void k_init_weights_bf16(MlpParams q)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kOffB1) {
        q.w1b[i - kOffW1] = to_bf16(q.P[i]);
    } else if (i >= kOffW2 && i < kOffB2) {
        const long at = i - kOffW2;
        q.w2b[at] = q.w2t[at % kInitHidden * kInitHidden + at / kInitHidden] = to_bf16(q.P[i]);
    } else if (i >= kOffW3 && i < kOffB3) {
        const long at = i - kOffW3;
        q.w3b[at] = q.w3t[at % kInitHidden * kInitOutPad + at / kInitHidden] = to_bf16(q.P[i]);
    }
}

__global__ void k_fill_f32(float *p, float v, long count)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

} // namespace smsq
