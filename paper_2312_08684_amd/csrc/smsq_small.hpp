// Step kernel for small particle sets (n <= 64, n_prev <= 128) in batches
// that leave most of the chip idle: the paper's own experiments (N_s =
// 10..40, one run or some tens).  The same time step as k_step (initial
// particles, L SVGD iterations with the median bandwidth, the score under the
// transition mixture and the Stein update, then the forward-recursion row of
// every particle) in one workgroup.
//
// Such a step is bound by latency, not by arithmetic or memory: 20 particles
// are 400 pairs.  So sixteen lanes share a particle, lane s taking the sources
// s, s + 16, ...: a wave holds four particles, a sum over the sources is at
// most four terms per lane and four rotations within a row of sixteen lanes
// (data-parallel primitives, no LDS), and all sixteen lanes keep their
// particle in registers and move it alike.  While these waves form the scores'
// transition terms, one more selects the median and one more takes the
// observation's gradients, a lane per particle (from 57 particles on the last
// two waves do so besides their own rows).  Three barriers an iteration:
// particles moved, distances written, bandwidth and scores written.
// Measured (us an iteration; one wave per sequence with a lane per particle,
// sources by readlane and a bisection over the median's bits -> here): 20
// particles of the range model in FP32 7.2 -> 2.1, 32 of the growth model in
// FP64 17.0 -> 3.1, and against the workgroup vector-ALU kernel 40 of its
// Matern-kernel ablation in FP64 22.8 -> 5.3.
#pragma once

#include "smsq_kernels.hpp"

namespace smsq {

constexpr int kSmallMaxParticles = 64;
constexpr int kSmallMaxPrev = 128;
constexpr int kPairBlock = 512;                  // distances, see select_near
constexpr int kRowLanes = 16;                    // lanes of a particle
constexpr int kRowsPerWave = kWave / kRowLanes;  // particles of a wave

// v moved round a row of sixteen lanes by N
template <int N> __device__ __forceinline__ int row_rotate(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);
}
template <int N> __device__ __forceinline__ float row_rotate(float v)
{
    return __int_as_float(row_rotate<N>(__float_as_int(v)));
}
template <int N> __device__ __forceinline__ double row_rotate(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = row_rotate<N>((int)b), hi = row_rotate<N>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// over the sixteen lanes of a row, the same bits in each (every step adds two
// halves of the row, in either order)
template <typename T, typename Op> __device__ __forceinline__ T row_reduce(T v, Op op)
{
    v = op(v, row_rotate<8>(v));
    v = op(v, row_rotate<4>(v));
    v = op(v, row_rotate<2>(v));
    return op(v, row_rotate<1>(v));
}
template <typename T> __device__ __forceinline__ T row_sum(T v)
{
    return row_reduce(v, [](T x, T y) { return x + y; });
}

// LDS of the kernel: particles of this and the last iteration, transition and
// observation terms of the scores [D][nst], scaled transition means [D][pst], their log2-weights and previous scores, pair
// distances of i < k at k (k - 1) / 2 + i, observation, bandwidth.
template <typename T> struct SmallLds {
    long off_x, off_s, off_g, off_m, off_c, off_pairs, off_z, off_h, total;
    int nst, pst, nrows, nwaves;  // waves of rows; with the selector and the gradients'
    // the distances, up to whole blocks of the selection that reads them from LDS
    static __host__ __device__ long padded_pairs(int n)
    {
        return ((long)n * (n - 1) / 2 + kPairBlock - 1) / kPairBlock * kPairBlock;
    }
    __host__ __device__ SmallLds(int n, int n_prev, int d)
    {
        nst = (n + kRowLanes - 1) / kRowLanes * kRowLanes;
        pst = (n_prev + kRowLanes - 1) / kRowLanes * kRowLanes;
        nrows = (n + kRowsPerWave - 1) / kRowsPerWave;
        nwaves = nrows <= 14 ? nrows + 2 : 16;
        long o = 0;
        off_x = o; o += align16(2L * d * nst * (long)sizeof(T));
        off_s = o; o += align16((long)d * nst * (long)sizeof(T));
        off_g = o; o += align16((long)d * nst * (long)sizeof(T));
        off_m = o; o += align16((long)d * pst * (long)sizeof(T));
        off_c = o; o += align16(2L * pst * (long)sizeof(T));
        off_pairs = o; o += align16(padded_pairs(n) * (long)sizeof(T));
        off_z = o; o += align16((long)kMaxObs * (long)sizeof(T));
        off_h = o; o += 16;
        total = o;
    }
};

// The r-th smallest (0-based) of the cnt values of buf (not negative, or NaN,
// which counts as largest), by one wave with S values per lane, kept in
// registers (REGS) or read from LDS at every probe (in blocks of kPairBlock,
// padded with infinities).  Probes t are
// counted by ballots until r or r + 1 values lie below one, when the answer
// is the least value from t on or the largest below it.  The first probe is
// `guess`, the others follow the local density of the values (kept from one
// call to the next) within the bracket found so far: three probes on average
// on the workloads, against 32 (FP64: 64) of a bisection over the bits, which
// is left for values tied across the rank.
template <typename T, int S, bool REGS>
__device__ T select_near(const T *buf, uint32_t cnt, uint32_t r, int lane, T guess, float &density)
{
    using KO = KeyOf<T>;
    using K = typename KO::K;
    constexpr int kBits = 8 * (int)sizeof(K);
    const T inf = RealOps<T>::inf();
    T v[REGS ? S : 1];
    if constexpr (REGS) {
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const uint32_t at = (uint32_t)(lane + q * kWave);
            v[q] = at < cnt ? buf[at] : inf;
        }
    }
    // f(value) for every value of the lane
    auto each = [&](auto &&f) {
        if constexpr (REGS) {
#pragma unroll
            for (int q = 0; q < S; ++q) f(v[q]);
        } else {
            for (uint32_t q = 0; q < cnt; q += kPairBlock) {
#pragma unroll
                for (int u = 0; u < kPairBlock; u += kWave) f(buf[q + u + lane]);
            }
        }
    };
    auto below = [&](T t) {
        uint32_t c = 0;
        each([&](T x) { c += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(x < t)); });
        return c;
    };
    T lo = 0, hi = inf;
    uint32_t clo = 0, chi = cnt;
    T t = guess;
    if (!(t > (T)0) || !(t < inf)) {
        T mx = 0;
        each([&](T x) { mx = x < inf && x > mx ? x : mx; });
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const T o = __shfl_xor(mx, off, kWave);
            mx = o > mx ? o : mx;
        }
        hi = mx;
        t = mx * (T)(((float)r + 0.5f) / (float)cnt);
        density = mx > (T)0 ? (float)((T)cnt / mx) : 0.f;
    }
    T tp = t;
    uint32_t cp = 0;
    for (int k = 0; k < 12; ++k) {
        const uint32_t c = below(t);
        if (c == r || c == r + 1) {
            K best = c == r ? ~(K)0 : 0;
            each([&](T x) {
                const K u = KO::key(x);
                if (c == r) best = x < t || u > best ? best : u;
                else best = x < t && u > best ? u : best;
            });
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const K o = __shfl_xor(best, off, kWave);
                best = (c == r) == (o < best) ? o : best;
            }
            return KO::val(best);
        }
        if (c < r) { lo = t; clo = c; }
        else { hi = t; chi = c; }
        if (k > 0 && c != cp) density = (float)((T)((float)c - (float)cp) / (t - tp));
        tp = t;
        cp = c;
        T next = t + (T)(((float)r + 0.5f - (float)c) / density);
        if (!(next > lo) || !(next < hi) || k >= 6) {
            const float frac = k >= 6 ? 0.5f : ((float)(r - clo) + 0.5f) / (float)(chi - clo);
            next = hi < inf ? lo + (hi - lo) * (T)frac : (T)2 * t;
        }
        t = next;
    }
    K prefix = 0;
    for (int b = kBits - 1; b >= 0; --b) {
        const K at = prefix | ((K)1 << b);
        uint32_t c = 0;
        each([&](T x) { c += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(KO::key(x) < at)); });
        if (c <= r) prefix = at;
    }
    return KO::val(prefix);
}
template <typename T>
__device__ T select_near(const T *buf, uint32_t cnt, uint32_t r, int lane, T guess, float &density)
{
    if (cnt <= 4 * kWave) return select_near<T, 4, true>(buf, cnt, r, lane, guess, density);
    if (cnt <= 8 * kWave) return select_near<T, 8, true>(buf, cnt, r, lane, guess, density);
    if (cnt <= 16 * kWave) return select_near<T, 16, true>(buf, cnt, r, lane, guess, density);
    return select_near<T, 32, sizeof(T) == 4>(buf, cnt, r, lane, guess, density);  // (FP64: registers are short)
}

template <typename T, int KIND, int D>
__global__ __launch_bounds__(1024) void k_step_small(StepArgs<T> a)
{
    using F = Family<T, KIND, D>;
    using R = RealOps<T>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int n = a.n, np = a.n_prev;
    const SmallLds<T> L(n, np, D);
    const int nst = L.nst, pst = L.pst;
    T *SX = (T *)(smem + L.off_x), *SS = (T *)(smem + L.off_s), *SG = (T *)(smem + L.off_g);
    T *SM = (T *)(smem + L.off_m), *SC = (T *)(smem + L.off_c);
    T *pairs = (T *)(smem + L.off_pairs), *sz = (T *)(smem + L.off_z), *sh = (T *)(smem + L.off_h);
    const int b = blockIdx.x;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & (kWave - 1), wave = wave_id();
    const int s = lane & (kRowLanes - 1);
    // this row's particle (rows past the set repeat its last one and write nothing)
    const int slot = wave * kRowsPerWave + (lane >> 4), i = min(slot, n - 1);
    const bool own = slot < n, first = own && s == 0;
    const bool selector = wave == L.nwaves - 1, gradients = wave == L.nwaves - 2, idle = wave >= L.nrows;
    const DevModel<T> &m = a.m;
    const T *xprev = a.x_prev + (long)b * a.x_prev_stride;
    T *xg = a.x + (long)b * a.x_stride;
    for (int q = n * (n - 1) / 2 + tid; q < (int)L.padded_pairs(n); q += nt) pairs[q] = R::inf();
    for (int o = tid; o < m.obs_dim; o += nt) sz[o] = a.z[(long)b * a.z_stride + o];
    static_assert(kMaxObs <= kWave, "one lane per element of an observation");
    const bool on = lane < m.n_obs && (!a.mask || a.mask[(long)b * a.mask_stride + lane]);
    const ObsBits mk{__builtin_amdgcn_ballot_w64(on)};

    // particles and means relative to the first previous particle's
    // transition mean, as in k_step; in FP32 iterations to the mean of all of
    // them (every wave forms it), as in the matrix-core step: a particle is
    // rounded at every move, by its distance from the centre (rms error after 50
    // iterations of 64 particles of the clutter model, over the displacement:
    // 8.3e-6 about the first one, 6.2e-6 in the matrix-core step)
    T cen[D], rs[D], irs[D];
    {
        T xp[D];
#pragma unroll
        for (int c = 0; c < D; ++c) xp[c] = xprev[c];
        F::mean(m, a.t, xp, cen);
    }
    if (sizeof(T) == 4 && a.n_iter > 0) {
        T off[D];
#pragma unroll
        for (int c = 0; c < D; ++c) off[c] = (T)0;
        for (int j = lane; j < np; j += kWave) {
            T xp[D], mu[D];
#pragma unroll
            for (int c = 0; c < D; ++c) xp[c] = xprev[(long)j * D + c];
            F::mean(m, a.t, xp, mu);
#pragma unroll
            for (int c = 0; c < D; ++c) off[c] += mu[c] - cen[c];
        }
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const T at = cen[c] + wave_sum(off[c]) / (T)np;
            cen[c] = R::finite(at) ? at : cen[c];
        }
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        rs[c] = m.rs[c];
        irs[c] = (T)1 / rs[c];
    }
    // means, centred and scaled to log2 units, the log2-weights (no source past
    // the last) and the previous scores: all of those are read here, before any
    // new one is written, so that phi may take phi_prev's place (at the end, with
    // a barrier of their own, they took 4% of 100 iterations of 32 particles of
    // the growth model in FP64)
    for (int j = tid; j < pst; j += nt) {
        T mj[D], cj = -R::inf();
#pragma unroll
        for (int c = 0; c < D; ++c) mj[c] = (T)0;
        if (j < np) {
            T xp[D], mu[D];
#pragma unroll
            for (int c = 0; c < D; ++c) xp[c] = xprev[(long)j * D + c];
            F::mean(m, a.t, xp, mu);
#pragma unroll
            for (int c = 0; c < D; ++c) mj[c] = (mu[c] - cen[c]) * rs[c];
            const T lw = a.log_w ? a.log_w[(long)b * a.log_w_stride + j] : -R::log_((T)np);
            cj = lw * (T)kLog2e;
        }
#pragma unroll
        for (int c = 0; c < D; ++c) SM[c * pst + j] = mj[c];
        SC[j] = cj;
        SC[pst + j] = a.do_viterbi && a.phi_prev && j < np ? a.phi_prev[(long)b * a.phi_prev_stride + j] : (T)0;
    }
    // particles, centred
    if (tid < n) {
        T xn[D];
        if (a.init_given) {
#pragma unroll
            for (int c = 0; c < D; ++c) xn[c] = xg[(long)tid * D + c] - cen[c];
        } else {
            T xp[D], mu[D];
            const int j = tid % np;
#pragma unroll
            for (int c = 0; c < D; ++c) xp[c] = xprev[(long)j * D + c];
            F::mean(m, a.t, xp, mu);
            double nz[D];
            normals<D>(a.seed, a.seq_offset + (uint32_t)b, (uint32_t)a.t, (uint32_t)tid, nz);
#pragma unroll
            for (int c = 0; c < D; ++c) xn[c] = (mu[c] - cen[c]) + m.sqrt_q[c] * (T)nz[c];
        }
#pragma unroll
        for (int c = 0; c < D; ++c) SX[c * nst + tid] = xn[c];
    }
    __syncthreads();
    T xi[D];
#pragma unroll
    for (int c = 0; c < D; ++c) xi[c] = SX[c * nst + i];
    // mean of the transition means (paper-literal score reading)
    T mbar_all[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        T v = 0;
        for (int j = s; j < np; j += kRowLanes) v += SM[c * pst + j] / rs[c];
        mbar_all[c] = row_sum(v) / (T)np;
    }

    const uint32_t M = (uint32_t)(n * (n - 1) / 2);
    const T inv_n = (T)1 / (T)n;
    T h = (T)1, med1 = 0, med2 = 0;   // the selector's last two medians
    float density = 0.f;
    for (int it = 0; a.do_svgd && it < a.n_iter; ++it) {
        const T *X = SX + (it & 1) * D * nst;        // this iteration's particles
        T *Xn = SX + (~it & 1) * D * nst;            // the next one's
        const bool bandwidth = a.bw_mode == 0 || it == 0;
        // (1) pair distances
        if (bandwidth && !idle) {
#pragma unroll
            for (int u = 0; u < kSmallMaxParticles / kRowLanes; ++u) {
                const int k = s + u * kRowLanes;
                if (u * kRowLanes >= n) break;
                T dd = 0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const T r = xi[c] - X[c * nst + k];   // (k < nst)
                    dd += r * r;
                }
                if (own && i < k && k < n) pairs[k * (k - 1) / 2 + i] = dd;
            }
        }
        __syncthreads();
        // (2) the bandwidth from their exact lower median, by one wave ...
        if (bandwidth && selector) {
            T med = 0;
            if (M > 0) {
                const T guess = it == 0 ? (T)0 : it == 1 ? med1 : med1 + (med1 - med2);
                med = select_near<T>(pairs, M, (M - 1) / 2, lane, guess, density);
            }
            med2 = med1;
            med1 = med;
            if (lane == 0) sh[0] = bandwidth_from_median(med, n, a.bw_scale);
        }
        // ... the gradients of the observation by another, a particle a lane
        if (gradients) {
            const int k = min(lane, n - 1);
            T xa[D], g[D];
#pragma unroll
            for (int c = 0; c < D; ++c) xa[c] = X[c * nst + k] + cen[c];
            F::grad(m, sz, mk, xa, g);
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (lane < n) SG[c * nst + lane] = g[c];
        }
        // ... and the transition term of this row's particle
        if (!idle) {
            T mb[D];
            if (a.trans_mode == 0) {
                T xs[D];
#pragma unroll
                for (int c = 0; c < D; ++c) xs[c] = xi[c] * rs[c];
                T mx = -R::inf(), sum = 0, acc[D];
#pragma unroll
                for (int c = 0; c < D; ++c) acc[c] = (T)0;
                constexpr int CH = 4;
                for (int j0 = 0; j0 < pst; j0 += CH * kRowLanes) {
                    T av[CH], cm = -R::inf();
#pragma unroll
                    for (int u = 0; u < CH; ++u) {
                        av[u] = -R::inf();
                        const int j = j0 + u * kRowLanes + s;
                        if (j0 + u * kRowLanes < pst) {
                            T q2 = 0;
#pragma unroll
                            for (int c = 0; c < D; ++c) {
                                const T r = xs[c] - SM[c * pst + j];
                                q2 += r * r;
                            }
                            av[u] = SC[j] - q2;
                        }
                        cm = av[u] > cm ? av[u] : cm;
                    }
                    cm = row_reduce(cm, [](T x, T y) { return x > y ? x : y; });
                    const T nm = cm > mx ? cm : mx;
                    const T at = nm > -R::inf() ? nm : (T)0;  // (sources of weight 0 only)
                    const T sf = R::exp2_(mx - at);
                    mx = nm;
                    sum *= sf;
#pragma unroll
                    for (int c = 0; c < D; ++c) acc[c] *= sf;
#pragma unroll
                    for (int u = 0; u < CH; ++u) {
                        if (j0 + u * kRowLanes >= pst) break;
                        const T e = R::exp2_(av[u] - at);
                        sum += e;
#pragma unroll
                        for (int c = 0; c < D; ++c) acc[c] += e * SM[c * pst + j0 + u * kRowLanes + s];
                    }
                }
                const T isum = (T)1 / row_sum(sum);
#pragma unroll
                for (int c = 0; c < D; ++c) mb[c] = row_sum(acc[c]) * isum * irs[c];
            } else {
#pragma unroll
                for (int c = 0; c < D; ++c) mb[c] = mbar_all[c];
            }
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (first) SS[c * nst + i] = (xi[c] - mb[c]) * m.inv_q[c];
        }
        __syncthreads();
        if (bandwidth) h = sh[0];
        if (a.h_out && tid == 0) a.h_out[(long)b * a.h_stride + it] = h;

        // (3) Stein direction and synchronous update
        if (!idle) {
            const T beta = (T)kLog2e / h;
            const T inv_h = (T)1 / h;
            const T cw = a.kernel == 0 ? (T)2 / h : (T)1;
            T as[D], ar[D];
#pragma unroll
            for (int c = 0; c < D; ++c) { as[c] = 0; ar[c] = 0; }
#pragma unroll
            for (int u = 0; u < kSmallMaxParticles / kRowLanes; ++u) {
                const int k = s + u * kRowLanes;
                if (u * kRowLanes >= n) break;
                T dd = 0, df[D];
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    df[c] = xi[c] - X[c * nst + k];
                    dd += df[c] * df[c];
                }
                T kap, w;
                if (a.kernel == 0) {
                    kap = R::exp2_(-beta * dd);
                    w = kap;  // times 2/h below
                } else {
                    stein_kernel<T>(a.kernel, dd, inv_h, kap, w);
                }
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    as[c] += k < n ? kap * (SG[c * nst + k] - SS[c * nst + k]) : (T)0;
                    ar[c] += k < n ? w * df[c] : (T)0;
                }
            }
#pragma unroll
            for (int c = 0; c < D; ++c) {
                xi[c] += a.step * (row_sum(as[c] + cw * ar[c]) * inv_n);
                if (first) Xn[c * nst + i] = xi[c];
            }
        }
        __syncthreads();
    }

    // write particles back; flag non-finite values
    bool bad = false;
    if (a.do_svgd && first) {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const T v = xi[c] + cen[c];
            bad |= !R::finite(v);
            xg[(long)i * D + c] = v;
        }
    }

    if (a.do_viterbi && !idle) {
        // forward recursion: c_ij = log_z - ln2 |xs_i - ms_j|^2 + phi_prev(j),
        // the lanes' candidates merged in the row (the first lane's operand
        // first: a NaN at j = 0 stays)
        T xs[D];
#pragma unroll
        for (int c = 0; c < D; ++c) xs[c] = xi[c] * rs[c];
        ArgBest<T> ab{-R::inf(), -R::inf(), s};
        int nan_seen = 0;
        for (int j = s; j < np; j += kRowLanes) {
            T q2 = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const T r = xs[c] - SM[c * pst + j];
                q2 += r * r;
            }
            const T A = m.log_z - (T)kLn2 * q2;
            const T cij = A + SC[pst + j];
            nan_seen |= cij != cij ? 1 : 0;
            if (j == 0) { ab.best = cij; ab.arg = 0; }
            else argbest_push(ab, cij, j);
        }
        auto merge = [&](ArgBest<T> o, int nan) {
            ab = argbest_merge(ab, o);
            nan_seen |= nan;
        };
        merge({row_rotate<8>(ab.best), row_rotate<8>(ab.second), row_rotate<8>(ab.arg)}, row_rotate<8>(nan_seen));
        merge({row_rotate<4>(ab.best), row_rotate<4>(ab.second), row_rotate<4>(ab.arg)}, row_rotate<4>(nan_seen));
        merge({row_rotate<2>(ab.best), row_rotate<2>(ab.second), row_rotate<2>(ab.arg)}, row_rotate<2>(nan_seen));
        merge({row_rotate<1>(ab.best), row_rotate<1>(ab.second), row_rotate<1>(ab.arg)}, row_rotate<1>(nan_seen));
        if (first) {
            T xa[D];
#pragma unroll
            for (int c = 0; c < D; ++c) xa[c] = xi[c] + cen[c];
            const T ell = F::loglik(m, sz, mk, xa);
            const T ph = ab.best + ell;
            bad |= nan_seen != 0 || ph != ph;
            a.phi[(long)b * a.phi_stride + i] = ph;
            a.psi[(long)b * a.psi_stride + i] = ab.arg;
            if (a.flags) {
                const T sc_ = ab.best > (T)1 || ab.best < (T)-1 ? (ab.best < 0 ? -ab.best : ab.best) : (T)1;
                a.flags[(long)b * a.flags_stride + i] =
                    (np > 1 && ab.second >= ab.best - a.tie_tol * sc_) ? 1 : 0;
            }
        }
    }
    if (__any(bad) && lane == 0) atomicOr(a.status, STATUS_NONFINITE);
}

} // namespace smsq
