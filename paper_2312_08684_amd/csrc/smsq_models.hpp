// Model families as device functions: transition mean f_t, observation
// log-likelihood log p(z | x) and its analytic gradient in x (paper Sec. II,
// eq. SSM; scenario shapes of Sec. V).  The transition density of every family
// is Gaussian, N(f_t(x_{t-1}), diag(q)); the kernels evaluate it themselves.
#pragma once

#include "smsq_common.hpp"

namespace smsq {

enum Kind { GROWTH1D = 0, RANGE2D = 1, CV4D = 2, ARM7 = 3, LINGAUSS = 4, SE2 = 5, ARM14 = 6 };

// Per-launch model constants, precomputed on the host in the kernel's type.
template <typename T> struct DevModel {
    int kind, d, obs_dim, n_obs;
    T q[16];       // transition variances
    T inv_q[16];   // 1 / q
    T sqrt_q[16];  // sqrt(q)
    T rs[16];      // sqrt(log2(e) / (2 q)): x * rs puts -(x-m)^2/(2q) in log2 units
    T log_z;       // -1/2 sum_d log(2 pi q_d)
    T p[64];       // family parameters
    T aux[16];     // family constants (RANGE2D: 1/r_var; CV4D: 1/r_var, log((1-P_D)/V),
                   // log(P_D / (2 pi r_var)); ARM7: cos alpha_i, sin alpha_i;
                   // SE2: 1/r_var, 1/b_var, log-density constant of one landmark)
    double grow[3]; // GROWTH1D cosine term c, omega, phase; ARM14 input amplitude,
                    // frequency, phase step (kept in double)
};

template <typename T, int KIND, int D> struct Family;

// The observed elements: as bits (a wave's uniform value, where a loop over
// them needs no load or branch), or as a caller's byte array, which may be
// null (all observed).
struct ObsBits { uint64_t bits; };
__device__ __forceinline__ bool observed(ObsBits mask, int k) { return (mask.bits >> k) & 1; }
__device__ __forceinline__ bool observed(const uint8_t *mask, int k) { return mask == nullptr || mask[k]; }
__device__ __forceinline__ int observed_count(ObsBits mask, int) { return __builtin_popcountll(mask.bits); }
__device__ __forceinline__ int observed_count(const uint8_t *mask, int n)
{
    int M = 0;
    for (int k = 0; k < n; ++k) M += observed(mask, k) ? 1 : 0;
    return M;
}

// ---------------------------------------------------------------------------
template <typename T> struct Family<T, GROWTH1D, 1> {
    static __device__ __forceinline__ void mean(const DevModel<T> &m, int t, const T *x, T *out)
    {
        const T v = x[0];
        const T c = (T)(m.grow[0] * cos(m.grow[1] * (double)t + m.grow[2]));
        out[0] = m.p[0] * v + m.p[1] * v / ((T)1 + v * v) + c;
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        if (!observed(mask, 0)) return (T)0;
        const T r = z[0] - m.p[5] * x[0] * x[0];
        return (T)-0.5 * r * r / m.p[6] - (T)0.5 * RealOps<T>::log_((T)(2.0 * kPi) * m.p[6]);
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
        g[0] = (T)0;
        if (!observed(mask, 0)) return;
        const T r = z[0] - m.p[5] * x[0] * x[0];
        g[0] = r / m.p[6] * ((T)2 * m.p[5] * x[0]);
    }
};

// ---------------------------------------------------------------------------
template <typename T> struct Family<T, RANGE2D, 2> {
    static __device__ __forceinline__ void mean(const DevModel<T> &, int, const T *x, T *out)
    {
        out[0] = x[0];
        out[1] = x[1];
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        const int nb = m.n_obs;
        const T lc = (T)0.5 * RealOps<T>::log_((T)(2.0 * kPi) * m.p[0]);
        T s = 0;
        for (int b = 0; b < nb; ++b) {
            if (!observed(mask, b)) continue;
            const T dx = x[0] - m.p[2 + 2 * b], dy = x[1] - m.p[3 + 2 * b];
            const T e = z[b] - RealOps<T>::sqrt_(dx * dx + dy * dy);
            s += (T)-0.5 * e * e / m.p[0] - lc;
        }
        return s;
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
        g[0] = g[1] = (T)0;
#pragma unroll 4
        for (int b = 0; b < m.n_obs; ++b) {
            const T dx = x[0] - m.p[2 + 2 * b], dy = x[1] - m.p[3 + 2 * b];
            const T r = RealOps<T>::sqrt_(dx * dx + dy * dy);
            const T w = (z[b] - r) * m.aux[0] / r;  // aux[0] = 1 / r_var
            const bool skip = !observed(mask, b) || r < (T)1e-12;
            g[0] += skip ? (T)0 : w * dx;
            g[1] += skip ? (T)0 : w * dy;
        }
    }
};

// ---------------------------------------------------------------------------
// Detection / clutter mixture: p(Z|x) = V^-(M-1) [(1-P_D)/V + (P_D/M) sum_m
// N(z_m; (px,py), r I)].  Evaluated as a log-sum-exp over the clutter term and
// the M detection terms: the largest term first, then the sums, so that the
// detections do not wait for one another (a running maximum with a rescaling
// branch per detection took the gradients of 512 particles 13,800 cycles of
// an iteration's 120,000).
template <typename T> struct Family<T, CV4D, 4> {
    static __device__ __forceinline__ void mean(const DevModel<T> &m, int, const T *x, T *out)
    {
        out[0] = x[0] + m.p[0] * x[2];
        out[1] = x[1] + m.p[0] * x[3];
        out[2] = x[2];
        out[3] = x[3];
    }
    // log sum = mx + log s, and the responsibility-weighted residual sums gx,
    // gy (scaled like s).  aux: 1 / r, log((1-P_D)/V), log(P_D / (2 pi r)).
    template <class Mask>
    static __device__ __forceinline__ void accumulate(const DevModel<T> &m, const T *z, Mask mask, const T *x,
                                                      int M, T &mx, T &s, T &gx, T &gy)
    {
        const T w = (T)0.5 * m.aux[0], ldet = m.aux[2] - RealOps<T>::log_((T)M);
        mx = m.aux[1];
#pragma unroll 4
        for (int k = 0; k < m.n_obs; ++k) {
            const T ex = z[2 * k] - x[0], ey = z[2 * k + 1] - x[1];
            const T v = observed(mask, k) ? ldet - w * (ex * ex + ey * ey) : -RealOps<T>::inf();
            mx = v > mx ? v : mx;
        }
        s = RealOps<T>::exp_(m.aux[1] - mx);
        gx = gy = (T)0;
#pragma unroll 4
        for (int k = 0; k < m.n_obs; ++k) {
            const bool on = observed(mask, k);  // (a dropped detection may hold anything)
            const T ex = on ? z[2 * k] - x[0] : (T)0, ey = on ? z[2 * k + 1] - x[1] : (T)0;
            const T e = on ? RealOps<T>::exp_(ldet - w * (ex * ex + ey * ey) - mx) : (T)0;
            s += e;
            gx += e * ex;
            gy += e * ey;
        }
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        const int M = observed_count(mask, m.n_obs);
        if (M == 0) return RealOps<T>::log_((T)1 - m.p[2]);
        T mx, s, gx, gy;
        accumulate(m, z, mask, x, M, mx, s, gx, gy);
        return -(T)(M - 1) * RealOps<T>::log_(m.p[3]) + mx + RealOps<T>::log_(s);
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
        g[0] = g[1] = g[2] = g[3] = (T)0;
        const int M = observed_count(mask, m.n_obs);
        if (M == 0) return;
        T mx, s, gx, gy;
        accumulate(m, z, mask, x, M, mx, s, gx, gy);
        const T sc = m.aux[0] / s;
        g[0] = gx * sc;
        g[1] = gy * sc;
    }
};

// ---------------------------------------------------------------------------
// Standard-DH 7-joint chain; the gradient is J^T (z - p) / r with the
// geometric Jacobian column z_{i-1} x (p - o_{i-1}) of each revolute joint.
// No frame is built: going back from the end effector, v_{i-1} = A_i v_i is
// the vector p - o_{i-1} in the coordinates of frame i-1 (v_7 = 0, p = v_0);
// going forward, the residual e turns into each frame by the transpose of its
// rotation, and the joint's gradient there is (z x v) . e = v_x e_y - v_y e_x.
// 10 + 8 operations a joint; two sweeps over the frames themselves (rotation
// matrices and origins) took 75 a joint, and the gradients of 1024 particles
// 12% of an iteration of the matrix-core step.
template <typename T> struct Family<T, ARM7, 7> {
    static __device__ __forceinline__ void mean(const DevModel<T> &, int, const T *x, T *out)
    {
#pragma unroll
        for (int a = 0; a < 7; ++a) out[a] = x[a];
    }
    // v_{i-1} (x, y parts in vx, vy if wanted) of every joint, with
    // A_i = Rz(q_i) Tz(d_i) Tx(a_i) Rx(alpha_i); p = v_0
    static __device__ __forceinline__ void end_effector(const DevModel<T> &m, const T *q, T *st, T *ct, T *vx, T *vy, T *p)
    {
        T x = 0, y = 0, w = 0;
#pragma unroll
        for (int i = 6; i >= 0; --i) {
            const T ca = m.aux[i], sa = m.aux[7 + i];
            RealOps<T>::sincos_(q[i], &st[i], &ct[i]);
            const T ux = x + m.p[1 + i], uy = ca * y - sa * w, uz = sa * y + ca * w;
            x = ct[i] * ux - st[i] * uy;
            y = st[i] * ux + ct[i] * uy;
            w = uz + m.p[15 + i];
            vx[i] = x;
            vy[i] = y;
        }
        p[0] = x; p[1] = y; p[2] = w;
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        if (!observed(mask, 0)) return (T)0;
        T st[7], ct[7], vx[7], vy[7], p[3];
        end_effector(m, x, st, ct, vx, vy, p);
        const T e0 = z[0] - p[0], e1 = z[1] - p[1], e2 = z[2] - p[2];
        return (T)-0.5 * (e0 * e0 + e1 * e1 + e2 * e2) / m.p[0]
               - (T)1.5 * RealOps<T>::log_((T)(2.0 * kPi) * m.p[0]);
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
#pragma unroll
        for (int a = 0; a < 7; ++a) g[a] = (T)0;
        if (!observed(mask, 0)) return;
        T st[7], ct[7], vx[7], vy[7], p[3];
        end_effector(m, x, st, ct, vx, vy, p);
        const T ir = (T)1 / m.p[0];
        T e0 = (z[0] - p[0]) * ir, e1 = (z[1] - p[1]) * ir, e2 = (z[2] - p[2]) * ir;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            g[i] = vx[i] * e1 - vy[i] * e0;
            const T ca = m.aux[i], sa = m.aux[7 + i];
            const T f0 = ct[i] * e0 + st[i] * e1, f1 = ct[i] * e1 - st[i] * e0;
            e0 = f0;
            e1 = ca * f1 + sa * e2;
            e2 = ca * e2 - sa * f1;
        }
    }
};

// ---------------------------------------------------------------------------
// 14-D manipulator of Sec. V-D, x = [q; qdot]: q_t = q + qdot dt and
// qdot_t = qdot + u_{t-1} dt with u_{t-1,i} = amp sin(freq (t - 1) + phase_step i).
// The observation is the end effector of the same DH chain as ARM7, whose
// constants sit at the same parameter slots: the likelihood and its
// joint-angle gradient are ARM7's, the velocity gradient is zero.
template <typename T> struct Family<T, ARM14, 14> {
    using Arm = Family<T, ARM7, 7>;
    static __device__ __forceinline__ void mean(const DevModel<T> &m, int t, const T *x, T *out)
    {
        const T dt = m.p[22];
#pragma unroll
        for (int a = 0; a < 7; ++a) {
            const T u = (T)(m.grow[0] * sin(m.grow[1] * (double)(t - 1) + m.grow[2] * (double)a));
            out[a] = x[a] + x[7 + a] * dt;
            out[7 + a] = x[7 + a] + u * dt;
        }
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        return Arm::loglik(m, z, mask, x);
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
        Arm::grad(m, z, mask, x, g);
#pragma unroll
        for (int a = 7; a < 14; ++a) g[a] = (T)0;
    }
};

// ---------------------------------------------------------------------------
// SE(2) pose (px, py, heading) of Sec. V-B: the heading turns by omega dt and
// the position moves v dt along the new heading.  One range-bearing
// measurement per step from one of n_l landmarks whose identity is unknown:
// the likelihood is the equal-weight mixture over the landmarks, evaluated as
// a running-max log-sum-exp in one pass (the gradient is the
// responsibility-weighted sum of the per-landmark gradients, accumulated in
// the same pass).  The bearing residual is mapped into [-pi, pi).
template <typename T> struct Family<T, SE2, 3> {
    static __device__ __forceinline__ void mean(const DevModel<T> &m, int, const T *x, T *out)
    {
        const T th = x[2] + m.p[2] * m.p[0];
        T s, c;
        RealOps<T>::sincos_(th, &s, &c);
        const T vdt = m.p[1] * m.p[0];
        out[0] = x[0] + vdt * c;
        out[1] = x[1] + vdt * s;
        out[2] = th;
    }
    static __device__ __forceinline__ T wrap(T a)
    {
        const T tau = (T)(2.0 * kPi);
        return a - tau * RealOps<T>::floor_((a + (T)kPi) / tau);
    }
    // log-mixture and, with g != nullptr, its gradient in (px, py)
    static __device__ __forceinline__ T mixture(const DevModel<T> &m, const T *z, const T *x, T *g)
    {
        const int nl = (int)m.p[5];
        T mx = -RealOps<T>::inf(), s = 0, g0 = 0, g1 = 0;
        for (int l = 0; l < nl; ++l) {
            const T dx = x[0] - m.p[6 + 2 * l], dy = x[1] - m.p[7 + 2 * l];
            const T r2 = dx * dx + dy * dy;
            const T rho = RealOps<T>::sqrt_(r2);
            const T er = z[0] - rho;
            const T eb = wrap(z[1] - RealOps<T>::atan2_(dy, dx));
            const T tl = (T)-0.5 * (er * er * m.aux[0] + eb * eb * m.aux[1]);
            T l0 = 0, l1 = 0;
            if (g && rho >= (T)1e-12) {
                const T gr = er * m.aux[0] / rho, gb = eb * m.aux[1] / r2;
                l0 = gr * dx - gb * dy;
                l1 = gr * dy + gb * dx;
            }
            if (tl > mx) {
                const T sc = RealOps<T>::exp_(mx - tl);
                s = s * sc + (T)1;
                g0 = g0 * sc + l0;
                g1 = g1 * sc + l1;
                mx = tl;
            } else {
                const T w = RealOps<T>::exp_(tl - mx);
                s += w;
                g0 += w * l0;
                g1 += w * l1;
            }
        }
        if (g) {
            g[0] = g0 / s;
            g[1] = g1 / s;
        }
        return mx + RealOps<T>::log_(s) + m.aux[2];
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        if (!observed(mask, 0)) return (T)0;
        return mixture(m, z, x, nullptr);
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
        g[0] = g[1] = g[2] = (T)0;
        if (!observed(mask, 0)) return;
        mixture(m, z, x, g);
    }
};

// ---------------------------------------------------------------------------
template <typename T, int D> struct Family<T, LINGAUSS, D> {
    static __device__ __forceinline__ void mean(const DevModel<T> &m, int, const T *x, T *out)
    {
#pragma unroll
        for (int a = 0; a < D; ++a) {
            T s = 0;
#pragma unroll
            for (int b = 0; b < D; ++b) s += m.p[a * D + b] * x[b];
            out[a] = s;
        }
    }
    template <class Mask>
    static __device__ __forceinline__ T loglik(const DevModel<T> &m, const T *z, Mask mask, const T *x)
    {
        if (!observed(mask, 0)) return (T)0;
        T s = 0;
        for (int r = 0; r < m.obs_dim; ++r) {
            T hx = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) hx += m.p[16 + r * D + c] * x[c];
            const T e = z[r] - hx;
            s += (T)-0.5 * e * e / m.p[32 + r] - (T)0.5 * RealOps<T>::log_((T)(2.0 * kPi) * m.p[32 + r]);
        }
        return s;
    }
    template <class Mask>
    static __device__ __forceinline__ void grad(const DevModel<T> &m, const T *z, Mask mask, const T *x, T *g)
    {
#pragma unroll
        for (int c = 0; c < D; ++c) g[c] = (T)0;
        if (!observed(mask, 0)) return;
        for (int r = 0; r < m.obs_dim; ++r) {
            T hx = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) hx += m.p[16 + r * D + c] * x[c];
            const T w = (z[r] - hx) / m.p[32 + r];
#pragma unroll
            for (int c = 0; c < D; ++c) g[c] += m.p[16 + r * D + c] * w;
        }
    }
};

} // namespace smsq
