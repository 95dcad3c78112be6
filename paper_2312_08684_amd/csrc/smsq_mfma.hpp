// FP32 step kernel on the matrix cores (v_mfma_f32_16x16x32_bf16 and
// v_mfma_f32_16x16x32_f16, wave64).
//
// Same computation as k_step (one workgroup per sequence, state in LDS), with
// the pairwise work of every SVGD iteration (eq. SVGD_newupdate) on MFMA:
//   * bandwidth: half the squared distances, n_i / 2 + n_k / 2 - x_i . x_k,
//     come from 16x16 Gram tiles; the exact lower median is found by one pass
//     that counts the distances below a window predicted from the previous
//     iterations' medians and keeps those inside it, then a rank among the
//     kept values (histogram and radix passes as fallbacks);
//   * scores: the transition-mixture softmax over the previous particles,
//     logit_kj = 2 mh_j . xh_k + c_j - |mh_j|^2 (log2 units; the common
//     -|xh_k|^2 drops out), as 16x16 tiles relative to a per-particle
//     reference, exp2 on the VALU, and the weighted sums
//     sum_j e_kj [2 mh_j, 1] accumulated by MFMA;
//   * Stein direction: tiles of the exponent of kappa,
//     2 beta x_k . x_i - beta n_k - beta n_i with beta = log2(e) / h, exp2,
//     and sum_k kappa_ik [s_k - (2/h) x_k, 1] accumulated by MFMA.
// Particles are stored centred on the mean of the previous step's transition
// means, which keeps |x|^2 small next to the squared distances in FP32.
//
// FP32 operands on the 16-bit units.  The FP32 MFMA of gfx950 occupies the
// vector ALU (34 cycles per 16x16x4 product, nothing else issues on the SIMD
// meanwhile), the 16-bit one runs beside it (a 16x16x32 product takes 6 to 8
// cycles of the ALU's time), so every contraction runs on the latter with its
// FP32 operands split:
//   * logits, Gram tiles and distances: each operand is cut (round to nearest)
//     into three bf16 pieces h + m + l, which hold all 24 bits exactly, |m| and
//     |l| at most 2^-8 and 2^-17 of the value's power of two and of either
//     sign, and the products hh, hm, mh, mm, hl, lh and ml fill the K-slots;
//     lm and ll are left out, 2^-25 of the operands' powers of two at most and
//     without bias (pieces cut by truncation left out up to 2^-22, all of the
//     product's sign);
//   * weighted sums: the vectors are cut (round to nearest) into three f16
//     pieces, which hold 24 bits of values above 2, with a power of two of its
//     own as scale for each component (kScaledMax, kTinyShare).  The
//     exponentials are cut into two f16 pieces, held near 2^3 (softmax) or at
//     most 2^3 (kappa): the pair is the FP32 value or, for a quarter of them, its
//     even neighbour, as far off as v_exp_f32 itself, and the same in the sums
//     and in their divisor (a third piece changes no error below in its third
//     digit and takes 25% longer).
// Products of pieces are exact in FP32.  The products of a block of 32 sources
// are summed by the matrix cores, the blocks by the vector ALU: an MFMA adds
// with 0.6 units in the last place (rms) of its largest addend, and 16 blocks
// chained through its accumulator put the direction of 512 particles 1.6 times
// as far off as FP32 MFMAs do.
// Error of an iteration's direction against 64 bits (rms over sets; FP32 MFMA
// -> here): 64 and 256 particles of the arm 4.4e-7 -> 3.6e-7 and 4.1e-7 -> 3.4e-7,
// of the range model 3.3e-7 -> 3.1e-7 and 3.2e-7 -> 2.8e-7, 512 of the clutter
// model 2.2e-7 -> 1.9e-7.
// Measured (us an SVGD iteration of 256 sequences; FP32 MFMA -> here): 1024
// particles of the arm 240 -> 145, 512 of the clutter model 70 -> 45, 256 of the
// range model 21 -> 17.  What bounds it now is vector issue at 1024 (active in 74%
// of the cycles: exponentials, operand splits and block sums, 11.8 vector
// instructions per 64 pairs of both passes, beside matrix units busy 37%) and,
// below 512, the serial stages between barriers.
//
// Operand layouts of the 16x16x32 MFMA (checked on gfx950): lane l gives
// A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16], j = 0..7; result
// register r of lane l is D[4 (l / 16) + r][l % 16].
#pragma once

#include "smsq_kernels.hpp"

namespace smsq {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

__device__ __forceinline__ f32x4 mfma_f16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

// low / high bf16 of a packed word as a float
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// two floats as bf16, packed (first float in the low half)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
// the three bf16 pieces of two floats, packed
struct Pieces3 {
    uint32_t h, m, l;
};
__device__ __forceinline__ Pieces3 split3(float a, float b)
{
    Pieces3 p;
    p.h = pack_bf16(a, b);
    a -= bf_lo(p.h);
    b -= bf_hi(p.h);
    p.m = pack_bf16(a, b);
    p.l = pack_bf16(a - bf_lo(p.m), b - bf_hi(p.m));
    return p;
}

// The same with the second float's pieces cut by truncation, all of its sign: a
// component that meets a pad's norm, whose products of pieces overflow, and may
// do so to one infinity only.
__device__ __forceinline__ Pieces3 split3_last(float a, float b)
{
    auto put = [](float lo, float hi) { return (pack_bf16(lo, 0.f) & 0xffffu) | (__float_as_uint(hi) & 0xffff0000u); };
    Pieces3 p;
    p.h = put(a, b);
    a -= bf_lo(p.h);
    b -= bf_hi(p.h);
    p.m = put(a, b);
    p.l = put(a - bf_lo(p.m), b - bf_hi(p.m));
    return p;
}

// the two f16 pieces of two floats, packed.  `neg1` is -1 held in a register
// the compiler cannot see through, so that the residuals stay mixed-precision
// fused multiply-adds into FP32 (v_fma_mix_f32, 4 cycles each, and one packed
// conversion; writing f16 halves with v_fma_mixlo / mixhi takes 8 cycles each).
__device__ __forceinline__ void split_f16(float a, float b, float neg1, uint32_t &hi, uint32_t &lo)
{
    const f16x2 h = __builtin_convertvector(f32x2{a, b}, f16x2);
    const float ra = __builtin_fmaf((float)h[0], neg1, a), rb = __builtin_fmaf((float)h[1], neg1, b);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{ra, rb}, f16x2));
}

__device__ __forceinline__ float fmax_(float a, float b) { return a > b ? a : b; }

// a block-uniform value kept in a scalar register
__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Reductions over a wave's lanes without LDS: rotations within the 16-lane
// rows (DPP), then across the rows; every lane gets the result.
template <int N> __device__ __forceinline__ uint32_t row_rotate(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + N, 0xf, 0xf, false);
}
template <typename Op> __device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op)
{
    v = op(v, row_rotate<8>(v));
    v = op(v, row_rotate<4>(v));
    v = op(v, row_rotate<2>(v));
    v = op(v, row_rotate<1>(v));
    auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op(a[0], a[1]);
    a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return op(a[0], a[1]);
}
// largest of non-negative values (as bit patterns; a NaN counts as larger)
__device__ __forceinline__ float wave_max_abs(float v)
{
    return __uint_as_float(wave_reduce(__float_as_uint(v), [](uint32_t a, uint32_t b) { return a > b ? a : b; }));
}
__device__ __forceinline__ uint32_t wave_count(uint32_t v)
{
    return wave_reduce(v, [](uint32_t a, uint32_t b) { return a + b; });
}

// max over the four 16-lane groups that hold the same column (lanes l, l^16,
// l^32, l^48)
__device__ __forceinline__ float group_max4(float v)
{
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float m1 = fmax_(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(m1), __float_as_uint(m1), false, false);
    return fmax_(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Up to sixteen waves per workgroup (four per SIMD), one 64-particle task
// each at the largest size.
constexpr int kMaxWaves = 16;
constexpr int kMaxParticles = 1024;  // largest sequence the kernel takes
// A workgroup of W waves takes up to W * TS tasks (TS task slots per wave).
// Exponentials of the softmax are taken relative to a reference 3 below (in
// log2 units) the particle's log-sum-exp at the previous iteration, so they
// sum to about 2^3.  A pass whose sums leave [1, inf) repeats with the
// reference at the largest logit: above 2^16 an f16 piece overflows (and
// turns the sum into a NaN), and below 1 the smallest pieces, of absolute
// error 2^-25, would show beside FP32 rounding.  The shift also adds to the
// rounding of the exponents, which are largest where the weights are: at 10
// the direction of 256 particles of the clutter model is off by 3.6e-7, at 3
// by 2.1e-7.
constexpr float kRefShift = 3.f;
constexpr float kRefMinSum = 1.f;
constexpr float kNoSource = -1e30f;  // logit of a source that takes no part (its exponential is 0)
// Half the squared norm of a pad particle: its distances are never the median
// and its kernel values are 0 (one bf16 piece, so no infinity minus infinity)
constexpr float kPadHalfNorm = 8.507059173023462e37f;  // 2^126
constexpr float kKapShift = 3.f;   // kappa is held times 2^3 (same reasons)
constexpr float kKapScale = 8.f;
// Largest beta |x|^2 whose kappa is formed from norms and products.  The
// rounding of their difference reaches 0.5 in the exponent there (2^-21 of
// beta |x|^2, the same for serial, truncating and single-rounding sums) and 13
// at 2^25, where an f16 piece of 2^3 kappa overflows and its sums are NaN.  Sets
// beyond (tight clouds far from their transition means, a particle far from all
// others, a small bw_scale) take their differences directly, on the vector ALU (us
// an iteration of 256 sequences, products and differences: 256 of the range model
// 17 and 36, 512 of the clutter model 45 and 166, 1024 of the arm 146 and 478).
constexpr float kMaxProductExponent = 1048576.f;  // 2^20
// Scales of the sums' vectors, a power of two for each component, bring the
// largest value to 2^13 .. 2^14 when they are set, and stay until a value
// reaches 2^15 or more than one in kTinyShare of a wave's values lie below 2,
// where three f16 pieces hold fewer than 24 bits.  (Fewer than that are values
// near a zero crossing, which count for nothing beside the others.)  Where fresh
// scales leave as many below 2 (one particle far beyond all others), the sums
// are formed on the vector ALU.
constexpr float kScaledMax = 32768.f;
constexpr int kTinyShare = 4;

// LDS byte layout of the MFMA step workgroup, and how its waves share the
// pairwise work.  Large sequences (more 32-particle tasks than waves): each
// wave takes whole tasks of 64 targets over all sources.  The others (split):
// tasks of 32 targets, whose 32-source blocks are split among several waves
// where there are waves left: a wave handles task w % ntasks over the split
// w / ntasks of the source range and leaves partial sums in LDS, merged in
// split order (the same result whatever the timing).  32-target tasks halve
// the longest wave's share at up to 192 particles and the splits to merge
// above (64-target tasks: 0.81 to 0.91 of today's rate at 48 and 64
// particles, where they left two waves; equal work at 384 and 512).  ns_sc /
// ns_st are the splits of the score and Stein passes (at most the blocks each
// pass has); nwaves the waves a launch of this shape uses.
// A workgroup of the multi-workgroup mode owns targets_local particles as its
// targets and holds every particle.
//
// k4 (d <= 3): rows of four components (three coordinates and the last) in
// place of eight.  Tables, with R = 4 or 8 components:
//   off_x   three planes [npad][R] bf16, the pieces of [x, |x|^2 / 2]
//   off_vt  three planes [chunk][R] bf16, the pieces of [2 mh, c']
//   off_v   [npad / 32][sum_rows][32] f16: pieces of the scaled [v, 1] (Stein sums)
//   off_ms  [chunk / 32][sum_rows][32] f16: pieces of the scaled [2 mh, 1]
//   off_b   operands of the workgroup's targets, in turn of the score and the
//           Stein pass, where several waves share a task (each would form them
//           again: 250 to 550 instructions a pass, as much as the pass itself
//           at 256 particles)
// The two sums' tables share one region where LDS is short (1024 particles of
// d >= 4): the transition one is then rebuilt each iteration.  Previous sets of
// d >= 4 that are too large even so (beyond 1088 particles of the arm and 1280 of
// the clutter model after 1024, 1376 and 1632 after 64; FP32 rows held 1376 and
// 2000) are taken in `chunks` of `chunk` sources, whose tables every iteration
// forms again from the previous particles (CHUNKED).
__host__ __device__ constexpr int sum_rows(int d) { return d <= 3 ? 12 : d == 4 ? 13 : 24; }
struct MfmaLds {
    int off_x, off_vt, off_v, off_ms, off_b, off_win, off_z, off_red, off_ones, off_part, total;
    int npad, nwaves, task, ntasks, ns_sc, ns_st, ns_max, win_cap, chunk, chunks;
    bool split, ms_shared, b_table;
    __host__ __device__ MfmaLds(int d, int n, int n_prev, int waves = kMaxWaves, int targets_local = 0,
                                int max_chunks = kMaxChunks)
    {
        const bool k4 = d <= 3;
        npad = (n + 63) / 64 * 64;
        const int targets = targets_local > 0 ? targets_local : npad;
        split = targets / 32 <= waves;
        task = split ? 32 : 64;
        ntasks = targets / task;
        const int row = k4 ? 8 : 16;  // bytes of a table row
        // the multi-workgroup mode keeps the partial sums over the sums' tables
        const bool alias = targets_local > 0;
        const int sources = (n_prev + 31) / 32;  // blocks of them
        int sums = 0, part = 0, bb = 0;
        bool fits = false;
        for (chunks = 1; !fits; ++chunks) {
            chunk = (sources + chunks - 1) / chunks * 32;
            ns_sc = ns_st = ns_max = 1;
            nwaves = waves;
            if (split) {
                const int cap = waves / ntasks;
                ns_sc = cap < chunk / 32 ? cap : chunk / 32;
                ns_st = cap < npad / 32 ? cap : npad / 32;
                ns_max = ns_sc > ns_st ? ns_sc : ns_st;
                // (from 256 particles on the idle waves take part in the median's pass)
                if (npad < 256) nwaves = ntasks * ns_max;
            }
            // partial sums of the splits: [ns_max][targets][R + 1] floats
            part = split ? (int)align16(ns_max * targets * (k4 ? 5 : 9) * 4) : 0;
            const int vb = npad * 2 * sum_rows(d), mb = chunk * 2 * sum_rows(d);
            // (also the rows [mh, phi] of the forward recursion, in FP32; in
            // chunks from off_vt on)
            const int rows = sources * 32 * (k4 ? 16 : 32) - (chunks > 1 ? 3 * row * chunk : 0);
            // target operands: four planes (k4: three) of 16 bytes per target
            bb = targets * (k4 ? 48 : 64);
            const int fixed = 3 * row * (npad + chunk) + 128 + 512 + 16 + (alias ? 0 : part) + 1024;
            // what fits, in the order of what it saves: target operands in a table
            // (several waves share each task), the sums' tables apart (else the
            // transition one is rebuilt each iteration), a window buffer of 4096
            // values (else 2048; also the histogram of a range or radix pass)
            for (int choice = 0; choice < 8 && !fits; ++choice) {
                b_table = !(choice & 4);
                ms_shared = alias || (choice & 2);
                win_cap = alias || (choice & 1) ? 2048 : 4096;
                if (b_table && !split) continue;
                sums = ms_shared ? (vb > mb ? vb : mb) : vb + mb;
                if (alias && sums < part) sums = part;
                if (sums < rows) sums = rows;
                off_ms = ms_shared ? 0 : vb;
                fits = fixed + sums + (b_table ? bb : 0) + 4 * win_cap <= kMfmaLdsBytes;
            }
            if (fits || k4 || alias || chunks >= max_chunks) break;
        }
        int o = 0;
        off_x = o; o += 3 * row * npad;
        off_vt = o; o += 3 * row * chunk;
        off_v = o;
        off_ms += o;
        off_part = alias ? o : o + sums;
        o += sums + (alias ? 0 : part);
        off_b = o; o += b_table ? bb : 0;
        off_win = o; o += 4 * win_cap + 1024;  // window buffer, bins of its selection
        off_z = o; o += 128;
        off_red = o; o += 512;  // uint slots 0..63, float slots from byte 256
        off_ones = o; o += 16;
        total = o;
    }
    static constexpr int kMaxChunks = 8;
    static constexpr int kMfmaLdsBytes = 160 * 1024 - 256;  // less the persistent kernels' static words
};

// LDS addresses held as such, opaque to the compiler (which would keep an offset
// and add the array's address at every read)
__device__ __forceinline__ uint32_t lds_address(const unsigned char *p, uint32_t offset)
{
    uint32_t a = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)p + offset;
    asm("" : "+v"(a));
    return a;
}
template <typename V> __device__ __forceinline__ V lds_read(uint32_t address)
{
    return *(const __attribute__((address_space(3))) V *)(uintptr_t)address;
}

// A lane's 16-bit A operands of one table: rows are sources, K-slots the
// piece products.  With eight components lane group g holds in the first MFMA
// piece (h, h, m, m)[g] against the B pieces (h, m, h, m)[g], in the second
// (h, l, 1, m)[g] against (l, h, constant, l)[g]; with four components the
// one MFMA holds two products per group, (hh, hm | mh, mm | hl, lh |
// constant, ml).  The constant's slots carry the pieces of a per-target
// constant against ones.
template <bool K4> struct SourceRows {
    uint32_t o0, o1, s1;
    __device__ void init(const unsigned char *smem, int base, int rows, int ones, int g, int col)
    {
        if (K4) {
            o0 = lds_address(smem, (uint32_t)(g == 3 ? ones : base + (g == 1 ? rows * 8 : 0) + col * 8));
            o1 = lds_address(smem, (uint32_t)(base + (g == 3 ? 1 : g) * rows * 8 + col * 8));
            s1 = g == 3 ? 0u : 128u;
        } else {
            o0 = lds_address(smem, (uint32_t)(base + (g >> 1) * rows * 16 + col * 16));
            o1 = lds_address(smem, (uint32_t)(g == 2 ? ones : base + (g == 0 ? 0 : g == 1 ? 2 : 1) * rows * 16 + col * 16));
            s1 = g == 2 ? 0u : 256u;
        }
    }
    __device__ __forceinline__ void load(int tile, u32x4 &a0, u32x4 &a1) const
    {
        if (K4) {
            const u32x2 p = lds_read<u32x2>(o0 + (uint32_t)tile * s1);
            const u32x2 q = lds_read<u32x2>(o1 + (uint32_t)tile * 128u);
            a0 = u32x4{p[0], p[1], q[0], q[1]};
        } else {
            a0 = lds_read<u32x4>(o0 + (uint32_t)tile * 256u);
            a1 = lds_read<u32x4>(o1 + (uint32_t)tile * s1);
        }
    }
    // moves the rows on by some tiles
    __device__ __forceinline__ void skip(int tiles)
    {
        o0 += (uint32_t)tiles * (K4 ? s1 : 256u);
        o1 += (uint32_t)tiles * (K4 ? 128u : s1);
    }
    static __device__ __forceinline__ f32x4 dot(u32x4 a0, u32x4 a1, u32x4 b0, u32x4 b1,
                                                f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f})
    {
        return K4 ? mfma_bf16(a0, b0, c) : mfma_bf16(a0, b0, mfma_bf16(a1, b1, c));
    }
};

// bits of a where mask is set, of b elsewhere (lane masks are 0 or ~0; written
// as bit operations so that no branch comes of it)
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// B operands of a target: the packed pieces of its R components and its
// constant, in the slots matching SourceRows.
template <bool K4>
__device__ __forceinline__ void target_operand(const uint32_t *h, const uint32_t *m, const uint32_t *l, float cst, int g,
                                               u32x4 &b0, u32x4 &b1)
{
    const Pieces3 c = split3(cst, 0.f);
    const uint32_t cc[2] = {c.h | (c.m << 16), c.l};
    const uint32_t odd = 0u - (uint32_t)(g & 1), high = 0u - (uint32_t)(g >> 1);
    if (K4) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            b0[q] = pick(high, pick(odd, cc[q], l[q]), h[q]);
            b0[2 + q] = pick(high, pick(odd, l[q], h[q]), m[q]);
        }
    } else {
        const uint32_t g1 = odd & ~high, g2 = high & ~odd;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            b0[q] = pick(odd, m[q], h[q]);
            b1[q] = pick(g2, q < 2 ? cc[q < 2 ? q : 0] : 0u, pick(g1, h[q], l[q]));
        }
    }
}
// its constant alone
template <bool K4> __device__ __forceinline__ void target_constant(float cst, int g, u32x4 &b0, u32x4 &b1)
{
    const Pieces3 c = split3(cst, 0.f);
    u32x4 &b = K4 ? b0 : b1;
    const uint32_t at = 0u - (uint32_t)(g == (K4 ? 3 : 2));
    b[0] = pick(at, c.h | (c.m << 16), b[0]);
    b[1] = pick(at, c.l, b[1]);
}

// The table of target operands: planes h, m, l and the constant ([h m], [l h]
// and [constant l] with four components) of 16 bytes per target.
template <bool K4>
__device__ __forceinline__ void put_target(unsigned char *smem, int base, int rows, int r, const float (&v)[K4 ? 4 : 8],
                                           float cst)
{
    constexpr int W = K4 ? 2 : 4;
    u32x4 *t = (u32x4 *)(smem + base) + r;
    uint32_t h[W], m[W], l[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const Pieces3 p = q == W - 1 ? split3_last(v[2 * q], v[2 * q + 1]) : split3(v[2 * q], v[2 * q + 1]);
        h[q] = p.h;
        m[q] = p.m;
        l[q] = p.l;
    }
    const Pieces3 c = split3(cst, 0.f);
    const u32x4 cc = {c.h | (c.m << 16), c.l, 0u, 0u};
    if constexpr (K4) {
        t[0] = u32x4{h[0], h[1], m[0], m[1]};
        t[rows] = u32x4{l[0], l[1], h[0], h[1]};
        t[2 * rows] = u32x4{cc[0], cc[1], l[0], l[1]};
    } else {
        t[0] = u32x4{h[0], h[1], h[2], h[3]};
        t[rows] = u32x4{m[0], m[1], m[2], m[3]};
        t[2 * rows] = u32x4{l[0], l[1], l[2], l[3]};
        t[3 * rows] = cc;
    }
}
template <bool K4>
__device__ __forceinline__ void load_target(const unsigned char *smem, int base, int rows, int r, int g, u32x4 &b0,
                                            u32x4 &b1)
{
    const u32x4 *t = (const u32x4 *)(smem + base) + r;
    if (K4) {
        b0 = t[(g > 1 ? g - 1 : 0) * rows];
    } else {
        b0 = t[(g & 1) * rows];
        b1 = t[(g == 1 ? 0 : g == 2 ? 3 : 2) * rows];
    }
}

// Rows of a three-plane table: the FP32 values are the exact sums of their
// pieces.
template <bool K4>
__device__ __forceinline__ void put_row(unsigned char *smem, int base, int rows, int r, const float (&v)[K4 ? 4 : 8])
{
    constexpr int W = K4 ? 2 : 4;
    uint32_t h[W], m[W], l[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const Pieces3 p = split3(v[2 * q], v[2 * q + 1]);
        h[q] = p.h;
        m[q] = p.m;
        l[q] = p.l;
    }
    if constexpr (K4) {
        *(u32x2 *)(smem + base + r * 8) = u32x2{h[0], h[1]};
        *(u32x2 *)(smem + base + (rows + r) * 8) = u32x2{m[0], m[1]};
        *(u32x2 *)(smem + base + (2 * rows + r) * 8) = u32x2{l[0], l[1]};
    } else {
        *(u32x4 *)(smem + base + r * 16) = u32x4{h[0], h[1], h[2], h[3]};
        *(u32x4 *)(smem + base + (rows + r) * 16) = u32x4{m[0], m[1], m[2], m[3]};
        *(u32x4 *)(smem + base + (2 * rows + r) * 16) = u32x4{l[0], l[1], l[2], l[3]};
    }
}
template <bool K4> struct PieceRow {
    static constexpr int W = K4 ? 2 : 4;
    uint32_t h[W], m[W], l[W];
    __device__ __forceinline__ void load(const unsigned char *smem, int base, int rows, int r)
    {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            uint32_t *d = p == 0 ? h : p == 1 ? m : l;
            if constexpr (K4) {
                const u32x2 v = *(const u32x2 *)(smem + base + (p * rows + r) * 8);
                d[0] = v[0]; d[1] = v[1];
            } else {
                const u32x4 v = *(const u32x4 *)(smem + base + (p * rows + r) * 16);
                d[0] = v[0]; d[1] = v[1]; d[2] = v[2]; d[3] = v[3];
            }
        }
    }
    __device__ __forceinline__ float at(int c) const
    {
        return (c & 1) ? (bf_hi(h[c / 2]) + bf_hi(m[c / 2])) + bf_hi(l[c / 2])
                       : (bf_lo(h[c / 2]) + bf_lo(m[c / 2])) + bf_lo(l[c / 2]);
    }
};

// Sums' table (off_v, off_ms): the f16 pieces h, m, l of the D components and
// the one of source s, in the rows of its 32-source block, at the position that
// matches the K-slots of a pair of 16x16 tiles: lane group g holds sources
// 4 g + r of the first tile in slots r and of the second in slots 4 + r.  Rows:
//   D <= 3   h, m, l / 2 of four components (the one is component 3); one
//            MFMA takes them all, its last four rows l / 2 again
//   D = 4    h, m, l of four components, then the one; one MFMA
//   above    h, m, l / 2 of eight components (the one is component 7); one
//            MFMA takes h and m, another l / 2 in either half of its rows
// (so that every lane reads a row of values and steps from block to block by
// the same distance).
template <int D> __device__ __forceinline__ void put_sum_row(unsigned char *smem, int base, int s, const float (&v)[D], float one)
{
    constexpr int C = D <= 4 ? 4 : 8, kOne = D <= 3 ? 3 : D == 4 ? 12 : 7;
    const int pos = ((s >> 2) & 3) * 8 + ((s >> 4) & 1) * 4 + (s & 3);
    _Float16 *d = (_Float16 *)(smem + base + (s >> 5) * (sum_rows(D) * 64)) + pos;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const _Float16 h = (_Float16)v[c];
        const float r = v[c] - (float)h;
        const _Float16 m = (_Float16)r;
        d[c * 32] = h;
        d[(C + c) * 32] = m;
        d[(2 * C + c) * 32] = (_Float16)((r - (float)m) * (D == 4 ? 1.f : 0.5f));
    }
    d[kOne * 32] = (_Float16)one;
    if constexpr (D != 4) d[(kOne + C) * 32] = d[(kOne + 2 * C) * 32] = (_Float16)0.f;
}
// A lane's operands of the table from source block blk on
template <int D> struct SumRows {
    uint32_t o0, o1;
    __device__ __forceinline__ void init(const unsigned char *smem, int table, int blk, int lane)
    {
        const int r = lane & 15;
        const uint32_t at = (uint32_t)(table + (lane >> 4) * 16 + blk * (sum_rows(D) * 64));
        o0 = lds_address(smem, at + (uint32_t)(D <= 3 && r >= 12 ? r - 4 : r) * 64u);
        if (D > 4) o1 = lds_address(smem, at + (uint32_t)(16 + (r & 7)) * 64u);
    }
    // the operands of this block; on to the next
    __device__ __forceinline__ void load(u32x4 &a0, u32x4 &a1)
    {
        a0 = lds_read<u32x4>(o0);
        o0 += sum_rows(D) * 64;
        if constexpr (D > 4) {
            a1 = lds_read<u32x4>(o1);
            o1 += sum_rows(D) * 64;
        }
    }
};

// power of two that brings values of magnitude up to `bound` below 2^bits
__device__ __forceinline__ float f16_scale(float bound, int bits)
{
    const int e = min(max((int)(__float_as_uint(bound) >> 23) & 0xff, 20), 250);  // 2^(e - 127) <= bound < 2^(e - 126)
    return __uint_as_float((uint32_t)(253 + bits - e) << 23);
}
// the inverse of a power of two
__device__ __forceinline__ float inverse_scale(float scale) { return __uint_as_float(0x7f000000u - __float_as_uint(scale)); }
// whether too many of a wave's `count` values are below 2 (zeros aside)
__device__ __forceinline__ bool many_tiny(float v, int count)
{
    const bool tiny = (__float_as_uint(v) & 0x7fffffffu) - 1u < 0x3fffffffu;
    return kTinyShare * __builtin_popcountll(__builtin_amdgcn_ballot_w64(tiny)) > count;
}

// Sum over the lane groups that hold a component's pieces, and a transpose:
// given O[q] of the four (two) 16-target tiles of a task (register i of lane
// group g holds row 4 g + i of target 16 q + l % 16), lane l receives the
// components of target l (l < 32 with two tiles): lo and hi the sums over the
// even and the odd lane groups.
template <int QT>
__device__ __forceinline__ void collect_groups(const float (&o)[QT], float &lo, float &hi)
{
    uint32_t u, w;
    if constexpr (QT == 4) {
        auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0]), __float_as_uint(o[2]), false, false);
        auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[1]), __float_as_uint(o[3]), false, false);
        // lane groups 0, 1: target tile 0 (1), rows g and g + 2; groups 2, 3: tile 2 (3)
        u = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
        w = __float_as_uint(__uint_as_float(b[0]) + __uint_as_float(b[1]));
    } else {
        auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0]), __float_as_uint(o[1]), false, false);
        // lane groups 0, 1: target tile 0; groups 2, 3: tile 1, brought below
        u = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
        auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        u = b[0];
        w = b[1];
    }
    auto c = __builtin_amdgcn_permlane16_swap(u, w, false, false);
    lo = __uint_as_float(c[0]);
    hi = __uint_as_float(c[1]);
}
template <int D, int QT>
__device__ __forceinline__ void collect_rows(const f32x4 (&O)[QT], float (&out)[D <= 3 ? 4 : 8])
{
    float o[QT], lo, hi;
    if constexpr (D == 4) {
        // the one's sums: register 0 of the last lane group
        const bool last = (threadIdx.x & 63) >= 48;
#pragma unroll
        for (int q = 0; q < QT; ++q) o[q] = last ? O[q][0] : 0.f;
        collect_groups<QT>(o, lo, hi);
        out[7] = hi;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
            o[q] = D == 4 && (threadIdx.x & 63) >= 48 ? 0.f : O[q][i];
        collect_groups<QT>(o, lo, hi);
        if constexpr (D <= 4) {
            out[i] = lo + hi;
            if constexpr (D == 4) if (i < 3) out[4 + i] = 0.f;
        } else {
            out[i] = lo;
            out[4 + i] = hi;
        }
    }
}

// One wave's walk over its share of the distances of the pairs k > i: the
// 32x32 blocks (targets 32 I.., sources 32 K.., K >= I) listed row by row and
// cut into as many equal runs as there are waves (in the multi-workgroup mode
// the waves of all its workgroups).  The results are half the squared
// distances (exact powers of two apart).  In a diagonal block the lanes that
// hold no pair k > i get +inf (as the products' addend); pad particles have
// half norms of 2^126.  Two tiles of targets share each source operand: with
// one the walk took twice the LDS reads, which bounded it.
template <bool K4> struct BlockWalker {
    const unsigned char *smem;
    int base;
    int rows, nb, g, col, I, K, left;
    SourceRows<K4> src;

    // blocks [p0, p1) of the list
    __device__ void start(const unsigned char *lds, int x_base, int npad, int ones, int lane, int p0, int p1)
    {
        smem = lds;
        base = x_base;
        rows = npad;
        g = lane >> 4;
        col = lane & 15;
        src.init(lds, x_base, npad, ones, g, col);
        nb = npad / 32;
        left = p1 - p0;
        I = 0;
        while (p0 >= nb - I) {
            p0 -= nb - I;
            ++I;
        }
        K = I + p0;
    }
    // B operand of target tile t: [-x_i, 1], constant |x_i|^2 / 2 - origin
    __device__ __forceinline__ void target(int t, float origin, u32x4 &b0, u32x4 &b1) const
    {
        constexpr int W = PieceRow<K4>::W;
        PieceRow<K4> p;
        p.load(smem, base, rows, t * 16 + col);
        const float half = p.at(K4 ? 3 : 7);
#pragma unroll
        for (int q = 0; q < W; ++q) {
            p.h[q] ^= 0x80008000u;
            p.m[q] ^= 0x80008000u;
            p.l[q] ^= 0x80008000u;
        }
        p.h[W - 1] = (p.h[W - 1] & 0xffffu) | 0x3f800000u;
        p.m[W - 1] &= 0xffffu;
        p.l[W - 1] &= 0xffffu;
        target_operand<K4>(p.h, p.m, p.l, half - origin, g, b0, b1);
    }
    // fn(D) for every block of the share: its four tiles' distances, relative
    // to `origin` (subtracted within the products' sum)
    template <typename Fn> __device__ __forceinline__ void visit_all(float origin, Fn &&fn)
    {
        const float inf = __builtin_huge_valf();
        for (; left > 0; ++I, K = I) {
            u32x4 b00, b01, b10, b11;
            target(2 * I, origin, b00, b01);
            target(2 * I + 1, origin, b10, b11);
            const int end = min(nb, K + left);
            left -= end - K;
            SourceRows<K4> at = src;
            at.skip(2 * K);
            f32x4 diag = {0.f, 0.f, 0.f, 0.f}, all = diag;
            if (K == I) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    diag[r] = 4 * g + r > col ? 0.f : inf;
                    all[r] = inf;
                }
            }
            // the next block's operands are read one block ahead (the last
            // reads run past the table into the one behind it, unused)
            u32x4 a00, a01, a10, a11;
            at.load(0, a00, a01);
            at.load(1, a10, a11);
            for (; K < end; ++K) {
                f32x4 D[4];
                D[0] = SourceRows<K4>::dot(a00, a01, b00, b01, diag);
                D[1] = SourceRows<K4>::dot(a00, a01, b10, b11, all);
                D[2] = SourceRows<K4>::dot(a10, a11, b00, b01);
                D[3] = SourceRows<K4>::dot(a10, a11, b10, b11, diag);
                at.skip(2);
                at.load(0, a00, a01);
                at.load(1, a10, a11);
                diag = all = f32x4{0.f, 0.f, 0.f, 0.f};
                fn(D);
            }
        }
    }
};

// One digit of a radix selection: wave 0 finds the histogram bin holding
// `rank` (red[0]) and the rank within it (red[1]).
__device__ __forceinline__ void radix_digit(const uint32_t *hist, uint32_t rank, uint32_t *red, int lane)
{
    constexpr int per = kBins / kWave;
    uint32_t cnt = 0;
    for (int q = 0; q < per; ++q) cnt += hist[lane * per + q];
    const uint32_t incl = wave_incl_scan(cnt, lane);
    const uint32_t excl = incl - cnt;
    if (lane == 0) { red[0] = 0; red[1] = 0; }
    __builtin_amdgcn_wave_barrier();
    if (rank >= excl && rank < incl) {
        uint32_t r = rank - excl;
        for (int q = 0; q < per; ++q) {
            const uint32_t h = hist[lane * per + q];
            if (r < h) { red[0] = (uint32_t)(lane * per + q); red[1] = r; break; }
            r -= h;
        }
    }
}

// Exact order statistic r of the n values of buf, all in [lo, hi], by a radix
// selection of the whole workgroup on the key offsets key - key(lo), 8 bits
// per pass, as many passes as the span needs.
__device__ float buffer_select(const float *buf, uint32_t n, uint32_t r, float lo, float hi, uint32_t *hist,
                               uint32_t *red)
{
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = wave_id();
    const uint32_t key_lo = __float_as_uint(lo), span = __float_as_uint(hi) - key_lo;
    const int bits = span == 0 ? 1 : 32 - __clz(span);
    uint32_t prefix = 0, pmask = 0;
    for (int p = (bits + 7) / 8 - 1; p >= 0; --p) {
        const int shift = 8 * p;
        for (int q = tid; q < 256; q += nt) hist[q] = 0;
        __syncthreads();
        for (uint32_t s = tid; s < n; s += nt) {
            const uint32_t k = __float_as_uint(buf[s]) - key_lo;
            if ((k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & 0xffu], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            uint32_t c[4];
            uint32_t cnt = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) { c[q] = hist[lane * 4 + q]; cnt += c[q]; }
            const uint32_t incl = wave_incl_scan(cnt, lane);
            const uint32_t excl = incl - cnt;
            if (r >= excl && r < incl) {
                uint32_t rr = r - excl;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (rr < c[q]) { red[8] = (uint32_t)(lane * 4 + q); red[9] = rr; break; }
                    rr -= c[q];
                }
            }
        }
        __syncthreads();
        prefix |= red[8] << shift;
        r = red[9];
        pmask |= 0xffu << shift;
        __syncthreads();
    }
    return __uint_as_float(key_lo + prefix);
}

// The same by one wave, for up to 64 S values (kept in registers).  The
// window is narrow, so its values are spread nearly evenly: a pivot placed by
// the rank's share of the values between two known counts (ballot counts)
// leaves the rank next to a pivot after three or four of them, and the answer
// is then the least value above it or the largest below.  Ties are settled
// bit by bit below the common prefix of the window's ends.
template <int S> __device__ __forceinline__ float window_select(const float *buf, uint32_t n, uint32_t r, float lo, float hi)
{
    const uint32_t lane = threadIdx.x & 63;
    float v[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const uint32_t at = lane + (uint32_t)q * kWave;
        v[q] = at < n ? buf[at] : __builtin_huge_valf();
    }
    auto count_below = [&](float t) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < S; ++q) c += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(v[q] < t));
        return c;
    };
    float a = lo, b = hi;
    uint32_t ca = 0, cb = n;
    for (int k = 0; k < 10; ++k) {
        const float t = a + (b - a) * (((float)(r - ca) + 0.5f) * __builtin_amdgcn_rcpf((float)(cb - ca)));
        const uint32_t c = count_below(t);
        if (c == r || c == r + 1) {
            uint32_t best = c == r ? 0x7f800000u : 0u;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const uint32_t u = __float_as_uint(v[q]);
                if (c == r) best = v[q] < t ? best : min(best, u);
                else best = v[q] < t ? max(best, u) : best;
            }
            if (c == r) best = wave_reduce(best, [](uint32_t x, uint32_t y) { return x < y ? x : y; });
            else best = wave_reduce(best, [](uint32_t x, uint32_t y) { return x > y ? x : y; });
            return __uint_as_float(best);
        }
        if (c < r) { a = t; ca = c; }
        else { b = t; cb = c; }
    }
    const uint32_t klo = __float_as_uint(lo), diff = klo ^ __float_as_uint(hi);
    const int top = diff ? 31 - __builtin_clz(diff) : -1;
    uint32_t prefix = top >= 31 ? 0u : klo & ~((1u << (top + 1)) - 1u);
    for (int bit = top; bit >= 0; --bit) {
        const uint32_t t = prefix | (1u << bit);
        if (count_below(__uint_as_float(t)) <= r) prefix = t;
    }
    return __uint_as_float(prefix);
}
constexpr uint32_t kSelectMax = 1024;   // most values the one-wave selection takes
__device__ float window_select(const float *buf, uint32_t n, uint32_t r, float lo, float hi)
{
    if (n <= 2 * kWave) return window_select<2>(buf, n, r, lo, hi);
    if (n <= 4 * kWave) return window_select<4>(buf, n, r, lo, hi);
    return window_select<kSelectMax / kWave>(buf, n, r, lo, hi);
}

// Median tracker across the iterations of one step (of half the squared
// distances).  The previous two medians, extrapolated, predict a window
// [lo, hi).  While the particles are unchanged the waves visit every distance
// once, counting those below lo and keeping those inside the window; the
// median is the matching order statistic of the kept ones.
// The half width is the larger of kWinTarget / 2 distances at the density of
// the last window and three times the recent error of the prediction (the
// largest, fading by 0.8 an iteration).  On the workloads' runs (N = 256 and
// 512, 50 and 100 iterations) that keeps 130 to 150 distances on average and
// misses the median in none of the iterations after the first two; windows of
// three times the median's last move kept 500 to 650 (4,000 at 1024 particles
// of the arm, where nine tiles in ten then held one) and missed 1%.
// Without a prediction, or when the window misses the rank or overflows,
// histogram passes over the distances narrow the range to one of few enough
// values (MedianRange).  The result is the exact lower median of the distances
// as the pass that ran rounds them: the window's pass subtracts lo within the
// products' sum, the others nothing, so the median may differ in its last bits
// with the path taken, and that with the buffer's capacity (workgroup shape,
// multi-workgroup mode).
constexpr int kWinTarget = 128;
constexpr int kMaxHistPasses = 4;
struct MedianTracker {
    float med1, med2, density, pred, err;
    int have;        // number of medians recorded (0, 1, 2, 3+)
    float lo, width; // the window [lo, lo + width)
    uint32_t below;  // per lane: distances below lo

    __device__ void reset()
    {
        med1 = med2 = density = pred = err = 0.f;
        have = 0;
    }

    // window of this iteration among M pairs; false without a prediction
    __device__ bool plan(uint32_t M, uint32_t cap)
    {
        if (have == 0 || !(med1 > 0.f)) return false;
        const float move = fabsf(med1 - med2);
        const float target = fminf((float)kWinTarget, fmaxf((float)(M / 64), 32.f));
        float w = density > 0.f ? 0.5f * target / density : 1e-3f * med1;
        pred = have >= 2 ? med1 + (med1 - med2) : med1;
        // one median: as wide as the buffer holds (at the densest, 0.7 of the
        // pairs per unit of relative distance), up to a hundredth
        if (have == 1) w = fminf(1e-2f, 0.6f * (float)cap / (float)M) * med1;
        else w = fmax_(w, have == 2 ? 0.5f * move : 3.f * err);
        w = fmax_(w, 2e-5f * med1);
        pred = uniform(pred);
        lo = uniform(fmax_(pred - w, 0.f));
        width = uniform(pred + w - lo);
        return true;
    }
    __device__ void record(float med)
    {
        if (have >= 2) err = fmax_(fabsf(med - pred), 0.8f * err);
        med2 = med1;
        med1 = uniform(med);
        err = uniform(err);
        have = have < 3 ? have + 1 : 3;
    }

    // A block's distances, relative to lo.  The common case: the sign bits of
    // a lane's sixteen values are shifted together and counted (those below
    // lo; a -0 counts as one), and one test tells that none lies in the
    // window: as bit patterns the least is not below the width (negative ones
    // are larger; a NaN is in neither).  Window distances are appended to the
    // common list while they fit (the order does not matter).
    __device__ __forceinline__ void visit(const f32x4 (&D)[4], float *list, uint32_t cap, uint32_t *counter)
    {
        uint32_t signs = 0, least = 0xffffffffu;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t d = __float_as_uint(D[r >> 2][r & 3]);
            signs = __builtin_amdgcn_alignbit(signs, d, 31);
            least = min(least, d);
        }
        below += (uint32_t)__builtin_popcount(signs);
        const uint32_t w = __float_as_uint(width);
        if (least < w) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float d = D[r >> 2][r & 3];
                if (__float_as_uint(d) < w) {
                    const uint32_t at = atomicAdd(counter, 1u);
                    if (at < cap) list[at] = lo + d;
                }
            }
        }
    }
};

// The range of the distances that holds the median's rank, narrowed by linear
// histograms of 2048 bins.  It starts at [0, top) with top four times the mean
// of |x|^2 / 2: the mean half squared distance is at most twice that mean,
// and a median is at most twice the mean.  (A radix selection on the bit
// patterns, whose first digit puts nearly all distances into a few bins, takes
// three passes and 240 us at 1024 particles of the arm; a histogram pass and a
// window pass about half of that.)
struct MedianRange {
    float a, b;          // the range
    __device__ float scale() const { return (float)kBins / (b - a); }
    // counts a block's distances of the range, and (per lane) those below it
    __device__ __forceinline__ void visit(const f32x4 (&D)[4], uint32_t *hist, float sc, uint32_t &below) const
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float d = fmax_(D[r >> 2][r & 3], 0.f);
            below += d < a ? 1u : 0u;
            if (d >= a && d < b) atomicAdd(&hist[min((int)((d - a) * sc), kBins - 1)], 1u);
        }
    }
    // narrows to a bin and a quarter of one on either side
    __device__ void narrow(uint32_t bin)
    {
        const float w = (b - a) / (float)kBins;
        const float na = a + ((float)bin - 0.25f) * w, nb = a + ((float)bin + 1.25f) * w;
        a = fmax_(na, 0.f);
        b = nb;
    }
};

// ---- multi-workgroup mode ---------------------------------------------
// The G workgroups of one sequence each own npad / G consecutive particles as
// their targets and hold every particle in LDS.  Per
// SVGD iteration they exchange, through global memory, the score rows of
// their targets and their share of the median's window pass (barrier 1),
// then their moved particles (barrier 2); every workgroup then holds the
// same state, and every selection they make from the exchanged data (the
// median, the radix fallback) is the same.  The layout of one sequence's
// exchange area, host and device:
constexpr int kCoopWinCap = 2048;     // window buffer of a workgroup (floats; MfmaLds::win_cap)
constexpr uint32_t kCoopSpinLimit = 1u << 24;  // barrier wait bound (polls)

struct CoopLayout {
    long off_ctr, off_x, off_s, off_info, off_vals, off_rhist, bytes;
    __host__ __device__ CoopLayout(int npad, int G)
    {
        long o = 0;
        off_ctr = o; o += 256;
        off_x = o; o += align16((long)npad * 8 * 4);
        off_s = o; o += align16((long)npad * 8 * 4);
        // two buffers each, used in turn
        off_info = o; o += align16((long)2 * G * 2 * 4);
        off_vals = o; o += align16((long)2 * G * kCoopWinCap * 4);
        off_rhist = o; o += align16((long)2 * G * kBins * 4);
        bytes = (o + 255) / 256 * 256;
    }
};

struct CoopArgs {
    char *base;     // exchange area of sequence 0; sequence b at base + b * stride
    long stride;
    int G;          // workgroups per sequence
    int gi;         // this workgroup's index within its sequence (set by the kernel)
};

// Barrier among the G workgroups of a sequence: thread 0 makes the
// workgroup's global writes visible at device scope, arrives on the counter
// and waits for epoch * G arrivals (bounded: past the bound the stall bit is
// set and the wait ends, and once it is set no barrier of the run waits),
// then acquires before the workgroup reads what the others wrote.
__device__ __forceinline__ void coop_barrier(uint32_t *ctr, uint32_t target, uint32_t *status)
{
    // every wave waits for its own global stores to complete, so they sit in
    // the L2 before the workgroup barrier; thread 0's device-scope release
    // then writes them back, and its acquire (before the second workgroup
    // barrier) invalidates the caches the other waves read through: one
    // write-back and one invalidation per workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicAdd(ctr, 1u);
        uint32_t polls = 0;
        // after one stall no later barrier waits (the run is flagged already)
        const bool stalled = (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & STATUS_STALLED) != 0;
        while (!stalled && __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(2);
            if (++polls > kCoopSpinLimit) {
                atomicOr(status, STATUS_STALLED);
                break;
            }
        }
        __threadfence();
    }
    __syncthreads();
}
// Step arguments in the constant address space (a kernel's own arguments, or a
// plan's items, which an earlier launch wrote): read by scalar loads where they
// are used.  As ordinary references the compiler copied them to scratch and
// read them lane by lane.
using ConstStepArgs = const __attribute__((address_space(4))) StepArgs<float>;

// SPLIT: the layout splits the sources of each task among waves (MfmaLds
// split); a separate instantiation, so the unsplit path keeps its
// registers.  COOP (with SPLIT): one of the G workgroups of sequence b in
// the multi-workgroup mode (cx).
// One sequence's time step (b: its index in the strided batch of `a`).  The
// workgroup owns the sequence: all state in LDS, every barrier block-wide.
// Thread tid owns particles tid + ts nt: it keeps their scores in registers
// from the score pass to the bandwidth, and moves them.  In the passes a wave
// covers a task of 64 targets, one per lane once its sums are collected.
template <int KIND, int D, int TS, bool SPLIT, bool COOP = false, bool CHUNKED = false>
__device__ __forceinline__ void step_mfma_body(ConstStepArgs *const ap, const int b, const CoopArgs cx = CoopArgs{})
{
    const StepArgs<float> &a = *(const StepArgs<float> *)ap;
    using F = Family<float, KIND, D>;
    using R = RealOps<float>;
    static_assert(D <= 7, "component 7 carries the norms");
    extern __shared__ __align__(16) unsigned char smem[];
    static_assert(!COOP || (SPLIT && TS == 1), "the multi-workgroup mode splits the sources");
    static_assert(!CHUNKED || (TS == 1 && !COOP), "chunks: one task a wave, one workgroup");
    // d <= 3: rows of four components, one MFMA per tile instead of two
    constexpr bool K4 = D <= 3;
    constexpr int NC = K4 ? 4 : 8;      // components of a table row
    constexpr int kLast = NC - 1;       // the norm, constant or ones component
    constexpr int kPart = NC + 1;       // floats of a split's partial sums per particle
    const int n = a.n, np = a.n_prev;
    const int G = COOP ? cx.G : 1, gi = COOP ? cx.gi : 0;
    constexpr int QT = SPLIT ? 2 : 4;   // 16-target tiles of a task
    constexpr int kTask = 16 * QT;
    const int npad0 = (n + 63) / 64 * 64;
    const MfmaLds L(D, n, np, (int)(blockDim.x >> 6), COOP ? npad0 / G : 0, CHUNKED ? MfmaLds::kMaxChunks : 1);
    const int npad = L.npad, chunk = L.chunk;   // (chunk: every source but for CHUNKED)
    float *PART = (float *)(smem + L.off_part); // [ns_max][targets][kPart] partial sums of the splits
    // the workgroup's targets: particles [tbase, tbase + ntl) (all of them outside COOP)
    const int tbase = gi * L.ntasks * kTask;
    // exchange area of this sequence (COOP)
    const CoopLayout CL(npad, G);
    char *cbase = COOP ? cx.base + (long)b * cx.stride : nullptr;
    uint32_t *cctr = (uint32_t *)(cbase + CL.off_ctr);
    float *cX = (float *)(cbase + CL.off_x);
    float *cS = (float *)(cbase + CL.off_s);
    uint32_t *cinfo = (uint32_t *)(cbase + CL.off_info);
    float *cvals = (float *)(cbase + CL.off_vals);
    uint32_t *crhist = (uint32_t *)(cbase + CL.off_rhist);
    uint32_t epoch = 0;  // barriers passed (the same count in every workgroup)
    float *WIN = (float *)(smem + L.off_win);                    // median window buffer, radix histogram
    uint32_t *whist = (uint32_t *)(smem + L.off_win) + L.win_cap;  // 256 bins of buffer_select
    float *sz = (float *)(smem + L.off_z);
    uint32_t *red = (uint32_t *)(smem + L.off_red);
    float *redf = (float *)(smem + L.off_red + 256);

    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = wave_id(), nwaves = nt >> 6;
    const DevModel<float> &m = a.m;
    const float *xprev = a.x_prev + (long)b * a.x_prev_stride;
    float *xg = a.x + (long)b * a.x_stride;
    const float inf = R::inf();
    float neg1 = -1.f;
    asm("" : "+s"(neg1));  // see split_f16

    if (tid == 0) *(u32x4 *)(smem + L.off_ones) = u32x4{0x3f803f80u, 0x3f80u, 0u, 0u};
    // red[12] what stands against a table just written (kRescale, kDirect);
    // [16 + c] largest |2 mh_c|, [24 + c] largest |v_c| where scales are set.
    // The scales themselves: redf[32 + c] of 2 mh, redf[40 + c] of v.
    constexpr uint32_t kRescale = 1, kDirect = 2;
    if (tid >= 12 && tid < 32) red[tid] = 0;
    const float *const ms_scale = redf + 32, *const v_scale = redf + 40;
    for (int o = tid; o < m.obs_dim; o += nt) sz[o] = a.z[(long)b * a.z_stride + o];
    static_assert(kMaxObs <= kWave, "one lane per element of an observation");
    const bool on = lane < m.n_obs && (!a.mask || a.mask[(long)b * a.mask_stride + lane]);
    const ObsBits mk{__builtin_amdgcn_ballot_w64(on)};
    float rs[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) rs[c] = c < D ? m.rs[c] : 0.f;

    float half_irs[D];   // 2 mh back to the state's units
#pragma unroll
    for (int c = 0; c < D; ++c) half_irs[c] = uniform(0.5f / rs[c]);

    // reference point: mean of the transition means
    float ref[D];
    for (int c = 0; c < D; ++c) {
        float part = 0.f;
        for (int j = tid; j < np; j += nt) {
            float xp[D], mu[D];
#pragma unroll
            for (int q = 0; q < D; ++q) xp[q] = xprev[(long)j * D + q];
            F::mean(m, a.t, xp, mu);
            part += mu[c];
        }
        part = wave_sum(part);
        if (lane == 0) redf[wave] = part;
        __syncthreads();
        float tot = 0.f;
        for (int w = 0; w < nwaves; ++w) tot += redf[w];
        ref[c] = uniform(tot / (float)np);
        __syncthreads();
    }

    // transition means, centred and log2-scaled: row j = [2 mh_j, c'_j] with
    // c'_j = log2 w_j - |mh_j|^2; pad sources and those of weight zero get a
    // logit that counts for nothing
    float mmax[D];
#pragma unroll
    for (int c = 0; c < D; ++c) mmax[c] = 0.f;
    // the table of the sources from `first` on
    auto build_vt = [&](int first) {
        for (int r = tid; r < chunk; r += nt) {
            const int j = first + r;
            float row[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) row[c] = 0.f;
            row[kLast] = kNoSource;
            if (j < np) {
                float xp[D], mu[D];
#pragma unroll
                for (int q = 0; q < D; ++q) xp[q] = xprev[(long)j * D + q];
                F::mean(m, a.t, xp, mu);
                float nrm = 0.f;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const float mh = (mu[c] - ref[c]) * rs[c];
                    row[c] = 2.f * mh;
                    mmax[c] = fmax_(mmax[c], fabsf(row[c]));
                    nrm += mh * mh;
                }
                const float lw = a.log_w ? a.log_w[(long)b * a.log_w_stride + j] : -R::log_((float)np);
                const float cj = lw * (float)kLog2e - nrm;
                row[kLast] = cj < kNoSource ? kNoSource : cj;
            }
            put_row<K4>(smem, L.off_vt, chunk, r, row);
        }
    };
    for (int ch = 0; ch < (CHUNKED ? L.chunks : 1); ++ch) build_vt(ch * chunk);
    // scales of the f16 pieces, from the largest magnitude of each component of
    // a wave's values
    auto note_max = [&](const float (&v)[D], int slot) {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float mx = wave_max_abs(fabsf(v[c]));
            if (lane == 0) atomicMax(&red[slot + c], __float_as_uint(mx));
        }
    };
    note_max(mmax, 16);
    __syncthreads();
    if (tid < D) redf[32 + tid] = f16_scale(__uint_as_float(red[16 + tid]), 15);
    __syncthreads();
    // the sums' table of the transition means, from its rows
    auto build_ms = [&](bool first, int from) {
        for (int j = tid; j < chunk; j += nt) {
            PieceRow<K4> p;
            p.load(smem, L.off_vt, chunk, j);
            float v[D];
            bool tiny = false;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                v[c] = p.at(c) * ms_scale[c];
                tiny |= first && many_tiny(v[c], min(kWave, max(np - from - (j & ~(kWave - 1)), 0)));  // (pads are zero)
            }
            if (tiny) red[12] = kDirect;
            put_sum_row<D>(smem, L.off_ms, j, v, 1.f);
        }
    };
    for (int ch = 0; ch < (CHUNKED ? L.chunks : 1); ++ch) {
        if (CHUNKED) build_vt(ch * chunk);  // (a thread's rows are its own in both tables)
        build_ms(true, ch * chunk);
    }
    const int ntl = L.ntasks * kTask;
    // score operand of particle i (at its place in a row), where it is one of
    // the workgroup's targets and they are kept
    auto put_score_target = [&](int i, const float (&x)[NC]) {
        if (!SPLIT || !L.b_table || i < tbase || i >= tbase + ntl) return;
        float v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = c == kLast ? 1.f : c < D ? x[c] * rs[c] : 0.f;
        put_target<K4>(smem, L.off_b, ntl, i - tbase, v, 0.f);
    };
    // initial particles, centred
    for (int i = tid; i < npad; i += nt) {
        float xi[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) xi[c] = 0.f;
        if (i < n) {
            if (a.init_given) {
#pragma unroll
                for (int c = 0; c < D; ++c) xi[c] = xg[(long)i * D + c] - ref[c];
            } else {
                float xp[D], mu[D];
                const int j = i % np;
#pragma unroll
                for (int c = 0; c < D; ++c) xp[c] = xprev[(long)j * D + c];
                F::mean(m, a.t, xp, mu);
                double nz[D];
                normals<D>(a.seed, a.seq_offset + (uint32_t)b, (uint32_t)a.t, (uint32_t)i, nz);
#pragma unroll
                for (int c = 0; c < D; ++c) xi[c] = (mu[c] + m.sqrt_q[c] * (float)nz[c]) - ref[c];
            }
        }
        float nrm = 0.f;
#pragma unroll
        for (int c = 0; c < kLast; ++c) nrm += xi[c] * xi[c];
        xi[kLast] = i < n ? 0.5f * nrm : kPadHalfNorm;
        put_row<K4>(smem, L.off_x, npad, i, xi);
        put_score_target(i, xi);
    }
    if (tid < 2) red[10 + tid] = 0;
    __syncthreads();
    const bool score_on_valu = __builtin_amdgcn_readfirstlane((int)red[12]) != 0;

    // mean of the centred transition means (literal score reading)
    float mbar_all[D];
#pragma unroll
    for (int c = 0; c < D; ++c) mbar_all[c] = 0.f;
    if (a.do_svgd && a.trans_mode == 1) {
        for (int c = 0; c < D; ++c) {
            float part = 0.f;
            for (int j = tid; j < np; j += nt) {
                if constexpr (CHUNKED) {
                    float xp[D], mu[D];
#pragma unroll
                    for (int q = 0; q < D; ++q) xp[q] = xprev[(long)j * D + q];
                    F::mean(m, a.t, xp, mu);
                    part += mu[c] - ref[c];
                } else {
                    PieceRow<K4> p;
                    p.load(smem, L.off_vt, chunk, j);
                    part += p.at(c) * half_irs[c];
                }
            }
            part = wave_sum(part);
            if (lane == 0) redf[wave] = part;
            __syncthreads();
            float tot = 0.f;
            for (int w = 0; w < nwaves; ++w) tot += redf[w];
            mbar_all[c] = uniform(tot / (float)np);
            __syncthreads();
        }
    }

    __syncthreads();
    if (tid == 0) red[12] = 0;  // (read above; used again past the next barrier)
    const int ntasks = L.ntasks;   // target tasks of this workgroup
    // every workgroup of the sequence has read its inputs before any writes
    // its outputs (the x array may hold the initial particles)
    if (COOP) coop_barrier(cctr, ++epoch * (uint32_t)G, a.status);
    const float inv_n = 1.f / (float)n;
    float h = 1.f;
    MedianTracker tracker;
    tracker.reset();
    // the softmax references of this wave's tasks, negated, one target per
    // lane, kept from one iteration to the next
    float negref[TS];
    bool have_ref = false;
    bool have_scale = false;  // of v

    // This thread's index, opaque to the compiler: addresses derived from it in
    // a pass are formed there instead of being kept (and spilled) across all
    // of them.
    auto fresh_tid = [&]() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    // The model, likewise: read again by scalar loads instead of held.
    auto fresh_model = [&]() -> const DevModel<float> & {
        ConstStepArgs *q = ap;
        asm volatile("" : "+s"(q));
        return ((const StepArgs<float> *)q)->m;
    };
    // O[q] = the sums over the source blocks [blk0, blk1) of 2^(exponent) times
    // the rows of a sums' table (at byte `table`), for the 16-target
    // tiles of a task (operands b0, b1).  A wave's instructions issue in order
    // and a SIMD has four waves, so the loop is pipelined by hand: while one
    // target tile's exponentials and their splits run on the vector ALU, the
    // matrix cores form the exponents of the tile after it and the sums of the
    // tile before it, one MFMA every four vector instructions; nothing waits
    // for a result of its own step.
    auto weighted_sums = [&](const SourceRows<K4> &src, int table, const u32x4 (&b0)[QT],
                             const u32x4 (&b1)[QT], int blk0, int blk1, f32x4 (&O)[QT]) {
        constexpr int kQ = QT;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        SumRows<D> sums;
        sums.init(smem, table, blk0, fresh_tid() & 63);
        u32x4 a00, a01, a10, a11, eh = {0u, 0u, 0u, 0u}, el = eh, av = eh, aw = eh;
        SourceRows<K4> at = src;
        at.skip(2 * blk0);
        at.load(0, a00, a01);
        at.load(1, a10, a11);
        f32x4 T0 = SourceRows<K4>::dot(a00, a01, b0[0], b1[0]), T1 = SourceRows<K4>::dot(a10, a11, b0[0], b1[0]);
#pragma unroll
        for (int q = 0; q < kQ; ++q) O[q] = zero;
        for (int blk = blk0; blk < blk1; ++blk) {
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int qn = (q + 1) % kQ, qp = (q + kQ - 1) % kQ;
                f32x4 N0, N1, S;
                if (K4) {
                    N0 = mfma_bf16(a00, b0[qn], zero);
                    S = mfma_f16(av, el, zero);
                    N1 = mfma_bf16(a10, b0[qn], zero);
                    S = mfma_f16(av, eh, S);
                } else {
                    N0 = mfma_bf16(a01, b1[qn], zero);
                    S = mfma_f16(av, el, zero);
                    N1 = mfma_bf16(a11, b1[qn], zero);
                    if (D > 4) S = mfma_f16(aw, eh, S);
                    N0 = mfma_bf16(a00, b0[qn], N0);
                    S = mfma_f16(av, eh, S);
                    N1 = mfma_bf16(a10, b0[qn], N1);
                }
                if (q == 0) sums.load(av, aw);
                if (q == kQ - 2) {
                    // the exponents of the next block start at the next step
                    // (past the last one: into the table behind, unused)
                    at.skip(2);
                    at.load(0, a00, a01);
                    at.load(1, a10, a11);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    T0[r] = R::exp2_(T0[r]);
                    T1[r] = R::exp2_(T1[r]);
                }
                uint32_t hi, lo;
                split_f16(T0[0], T0[1], neg1, hi, lo); eh[0] = hi; el[0] = lo;
                split_f16(T0[2], T0[3], neg1, hi, lo); eh[1] = hi; el[1] = lo;
                split_f16(T1[0], T1[1], neg1, hi, lo); eh[2] = hi; el[2] = lo;
                split_f16(T1[2], T1[3], neg1, hi, lo); eh[3] = hi; el[3] = lo;
                O[qp] += S;
                T0 = N0;
                T1 = N1;
            }
        }
        f32x4 S = mfma_f16(av, el, zero);
        if (D > 4) S = mfma_f16(aw, eh, S);
        O[kQ - 1] += mfma_f16(av, eh, S);
    };

    // components of the target operands: [x_k in log2 units, 1] of the scores,
    // [2 beta x_i, -2 beta] of the Stein direction
    auto score_target = [&](const float (&xt)[D], float (&v)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = c == kLast ? 1.f : c < D ? xt[c < D ? c : 0] * rs[c] : 0.f;
    };
    auto target_row = [&](const float (&v)[NC], float cst, int g, u32x4 &b0, u32x4 &b1) {
        uint32_t ph[NC / 2], pm[NC / 2], pl[NC / 2];
#pragma unroll
        for (int w = 0; w < NC / 2; ++w) {
            const Pieces3 s = w == NC / 2 - 1 ? split3_last(v[2 * w], v[2 * w + 1]) : split3(v[2 * w], v[2 * w + 1]);
            ph[w] = s.h; pm[w] = s.m; pl[w] = s.l;
        }
        target_operand<K4>(ph, pm, pl, cst, g, b0, b1);
    };
    // coordinates of particle k
    auto target_x = [&](int k, float (&xt)[D]) {
        PieceRow<K4> p;
        p.load(smem, L.off_x, npad, k);
#pragma unroll
        for (int c = 0; c < D; ++c) xt[c] = p.at(c);
    };
    // score_sums on the vector ALU, whatever the logits' magnitude: the
    // exponentials stay in FP32, relative to the largest logit so far
    int first_source = 0;   // of the tables
    auto score_direct = [&](int kbase, int blk0, int blk1, float &nref, float (&os)[NC]) {
        float xs[D], mx = kNoSource, sum = 0.f, acc[D];
        target_x(kbase + (fresh_tid() & (kTask - 1)), xs);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            xs[c] *= rs[c];
            acc[c] = 0.f;
        }
        const int j1 = min(32 * blk1, np - first_source);
        for (int j = 32 * blk0; j < j1; ++j) {
            PieceRow<K4> p;
            p.load(smem, L.off_vt, chunk, j);
            float logit = p.at(kLast);
#pragma unroll
            for (int c = 0; c < D; ++c) logit += p.at(c) * xs[c];
            const float nm = logit > mx ? logit : mx;
            const float sf = R::exp2_(mx - nm), e = logit > 0.1f * kNoSource ? R::exp2_(logit - nm) : logit - logit;
            mx = nm;
            sum = sum * sf + e;
#pragma unroll
            for (int c = 0; c < D; ++c) acc[c] = acc[c] * sf + e * p.at(c);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) os[c] = c == kLast ? sum : c < D ? acc[c < D ? c : 0] * ms_scale[c < D ? c : 0] : 0.f;
        nref = mx > 0.1f * kNoSource ? -mx : 0.f;
    };
    // os[c] = sum_j e_kj [2 mh_j, 1] (times ms_scale[c] but for the last) over the
    // source blocks [blk0, blk1) for this lane's particle kbase + lane,
    // e_kj = exp2(logit_kj - sref)
    auto score_sums = [&](int kbase, int blk0, int blk1, float &nref, float (&os)[NC], float &sref) {
        const int lane = fresh_tid() & 63, g = lane >> 4, col = lane & 15;
        u32x4 b0[QT], b1[QT];
        SourceRows<K4> src;
        src.init(smem, L.off_vt, chunk, L.off_ones, g, col);
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const float cst = have_ref ? __shfl(nref, 16 * q + col, kWave) : 0.f;
            b1[q] = u32x4{0u, 0u, 0u, 0u};
            if (SPLIT && L.b_table) {
                load_target<K4>(smem, L.off_b, ntl, kbase - tbase + 16 * q + col, g, b0[q], b1[q]);
                target_constant<K4>(cst, g, b0[q], b1[q]);
            } else {
                PieceRow<K4> p;
                p.load(smem, L.off_x, npad, kbase + 16 * q + col);
                float v[NC];
                float xt[D];
#pragma unroll
                for (int c = 0; c < D; ++c) xt[c] = p.at(c);
                score_target(xt, v);
                target_row(v, cst, g, b0[q], b1[q]);
            }
        }
        bool from_max = !have_ref;
        for (;;) {
            if (score_on_valu) {
                score_direct(kbase, blk0, blk1, nref, os);
                break;
            }
            if (from_max) {
                // references from the largest logits of the sources
                float mx[QT];
#pragma unroll
                for (int q = 0; q < QT; ++q) {
                    mx[q] = -inf;
                    target_constant<K4>(0.f, g, b0[q], b1[q]);
                }
                for (int jt = 2 * blk0; jt < 2 * blk1; ++jt) {
                    u32x4 a0, a1;
                    src.load(jt, a0, a1);
#pragma unroll
                    for (int q = 0; q < QT; ++q) {
                        const f32x4 T = SourceRows<K4>::dot(a0, a1, b0[q], b1[q]);
                        mx[q] = fmax_(mx[q], fmax_(fmax_(T[0], T[1]), fmax_(T[2], T[3])));
                    }
                }
#pragma unroll
                for (int q = 0; q < QT; ++q) {
                    // no source at all (padding, or weights of zero): reference 0
                    const float gm = group_max4(mx[q]);
                    const float nr = gm > 0.1f * kNoSource ? kRefShift - gm : 0.f;
                    target_constant<K4>(nr, g, b0[q], b1[q]);
                    if (g == q) nref = nr;
                }
            }
            f32x4 O[QT];
            weighted_sums(src, L.off_ms, b0, b1, blk0, blk1, O);
            collect_rows<D, QT>(O, os);
            const float s = os[kLast];
            const bool ok = lane >= kTask || (s >= kRefMinSum && s < 1e30f) || (nref == 0.f && s == 0.f);
            if (!__builtin_amdgcn_ballot_w64(!ok)) break;
            if (from_max) {  // (logits so large that their rounding overflows a piece)
                score_direct(kbase, blk0, blk1, nref, os);
                break;
            }
            from_max = true;
        }
        sref = -nref;
        if (os[kLast] > 0.f && os[kLast] < 1e30f) nref += kRefShift - __builtin_amdgcn_logf(os[kLast]);
        else if (nref == 0.f) sref = kNoSource;  // nothing to merge
    };
    // score row of a particle: the observation's gradient, then the transition
    // term from its softmax sums
    auto score_grad = [&](const float (&xt)[D], float (&s)[D]) {
        float xa[D];
#pragma unroll
        for (int c = 0; c < D; ++c) xa[c] = xt[c] + ref[c];
        F::grad(fresh_model(), sz, mk, xa, s);
    };
    auto score_transition = [&](const float *os, const float (&xt)[D], float (&s)[D]) {
        const DevModel<float> &m = fresh_model();
        if (a.trans_mode == 0) {
            const float inv_sum = 1.f / os[kLast];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float mb = os[c] * inv_sum * (inverse_scale(ms_scale[c]) * half_irs[c]);
                s[c] -= (xt[c] - mb) * m.inv_q[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < D; ++c) s[c] -= (xt[c] - mbar_all[c]) * m.inv_q[c];
        }
    };
    // the splits' partial sums of target kl, merged in split order (softmax
    // sums rebased to their largest reference)
    auto merge_part = [&](int kl, int ns, bool softmax, float (&os)[NC]) {
        float mx = -inf;
        for (int sp = 0; softmax && sp < ns; ++sp) mx = fmax_(mx, PART[(sp * ntl + kl) * kPart + NC]);
#pragma unroll
        for (int c = 0; c < NC; ++c) os[c] = 0.f;
        for (int sp = 0; sp < ns; ++sp) {
            const float *pp = PART + (sp * ntl + kl) * kPart;
            const float w = softmax ? R::exp2_(pp[NC] - mx) : 1.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) os[c] += pp[c] * w;
        }
    };

    // ---- exact lower median of the half squared distances ----
    const uint32_t M = (uint32_t)((long)n * (n - 1) / 2);
    const uint32_t rank = M > 0 ? (M - 1) / 2 : 0u;
    const uint32_t cap = (uint32_t)L.win_cap;
    uint32_t *hist = (uint32_t *)WIN;  // histograms use the window buffer
    // red[10], red[11]: values in the window, values below it (of this
    // workgroup; red[10] beyond `cap` where they do not fit)
    // a walk over this wave's share of the distances
    const int nblocks = npad / 32 * (npad / 32 + 1) / 2;
    auto walk = [&](float origin, auto &&fn) {
        const int v = gi * nwaves + wave, nv = G * nwaves;
        BlockWalker<K4> walker;
        walker.start(smem, L.off_x, npad, L.off_ones, fresh_tid() & 63, nblocks * v / nv, nblocks * (v + 1) / nv);
        walker.visit_all(origin, fn);
    };
    // adds the lanes' counts of distances below the window or range
    auto add_below = [&](uint32_t count) {
        count = wave_count(count);
        if (lane == 0) atomicAdd(&red[11], count);
    };
    auto window_walk = [&]() {
        tracker.below = 0;
        walk(tracker.lo, [&](const f32x4 (&Dv)[4]) { tracker.visit(Dv, WIN, cap, &red[10]); });
        add_below(tracker.below);
    };
    // COOP: this workgroup's counts and kept values to the exchange area ...
    int parity = 0;  // of the exchange buffers: a workgroup may still read the last ones
    auto publish_window = [&]() {
        const uint32_t kept = red[10];
        float *vals = cvals + ((long)parity * G + gi) * kCoopWinCap;
        for (uint32_t q = tid; q < min(kept, cap); q += nt) vals[q] = WIN[q];
        if (tid == 0) {
            cinfo[(parity * G + gi) * 2 + 0] = kept;
            cinfo[(parity * G + gi) * 2 + 1] = red[11];
        }
    };
    // ... and, past a barrier of the sequence's workgroups, everybody's into
    // this workgroup's (red[10] beyond `cap` where they do not fit)
    auto collect_window = [&]() {
        uint32_t *ci = (uint32_t *)redf;  // [32]
        if (tid < 2 * G) ci[tid] = cinfo[parity * G * 2 + tid];
        __syncthreads();
        uint32_t kept = 0, below = 0;
        for (int q = 0; q < G; ++q) {
            const uint32_t c = ci[2 * q];
            kept = c > cap || kept > cap ? cap + 1 : kept + c;
            below += ci[2 * q + 1];
        }
        if (kept <= cap) {
            for (uint32_t e = tid; e < kept; e += nt) {
                uint32_t off = 0;
                int q = 0;
                while (e >= off + ci[2 * q]) off += ci[2 * q++];
                WIN[e] = cvals[((long)parity * G + q) * kCoopWinCap + (e - off)];
            }
        }
        if (tid == 0) {
            red[10] = kept;
            red[11] = below;
        }
        parity ^= 1;
        __syncthreads();
    };
    // a histogram over every workgroup's distances (COOP)
    auto share_hist = [&]() {
        if constexpr (COOP) {
            uint32_t *rh = crhist + (long)parity * G * kBins;
            for (int q = tid; q < kBins; q += nt) rh[(long)gi * kBins + q] = hist[q];
            if (tid == 0) cinfo[(parity * G + gi) * 2 + 1] = red[11];
            coop_barrier(cctr, ++epoch * (uint32_t)G, a.status);
            uint32_t below = 0;
            for (int q = 0; q < G; ++q) below += cinfo[(parity * G + q) * 2 + 1];
            for (int q = tid; q < kBins; q += nt) {
                uint32_t c = 0;
                for (int gg = 0; gg < G; ++gg) c += rh[(long)gg * kBins + q];
                hist[q] = c;
            }
            if (tid == 0) red[11] = below;
            parity ^= 1;
            __syncthreads();
        }
    };
    auto clear_counts = [&]() {
        __syncthreads();
        if (tid < 2) red[10 + tid] = 0;
    };
    // whether the window of the last walk holds the median
    auto in_window = [&]() { return rank >= red[11] && rank - red[11] < red[10] && red[10] <= cap; };
    // the median from the window's values: by the last wave (up to kSelectMax
    // values), or by all
    auto select_by_wave = [&]() {
        const float v = window_select(WIN, red[10], rank - red[11], tracker.lo, tracker.lo + tracker.width);
        if (lane == 0) red[5] = __float_as_uint(v);
    };
    // without a window: histogram passes, then a window; a radix selection
    // (digits of 11, 11 and 10 bits) where values tie too heavily for those
    auto median_from_range = [&]() {
        float hsum = 0.f;
        for (int i = lane; i < n; i += kWave) {
            PieceRow<K4> p;
            p.load(smem, L.off_x, npad, i);
            hsum += p.at(kLast);
        }
        MedianRange rg;
        rg.a = 0.f;
        rg.b = uniform(4.004f * wave_sum(hsum) / (float)n + 1e-37f);
        for (int pass = 0; pass < kMaxHistPasses; ++pass) {
            clear_counts();
            for (int q = tid; q < kBins; q += nt) hist[q] = 0;
            __syncthreads();
            const float sc = rg.scale();
            uint32_t below = 0;
            walk(0.f, [&](const f32x4 (&Dv)[4]) { rg.visit(Dv, hist, sc, below); });
            add_below(below);
            __syncthreads();
            share_hist();
            if (rank < red[11]) break;
            if (wave == 0) radix_digit(hist, rank - red[11], red, lane);
            __syncthreads();
            const uint32_t bin = red[0], count = hist[red[0]];
            rg.narrow(bin);
            if (2 * count <= cap) {
                tracker.lo = uniform(rg.a);
                tracker.width = uniform(rg.b - rg.a);
                clear_counts();
                __syncthreads();
                window_walk();
                __syncthreads();
                if constexpr (COOP) {
                    publish_window();
                    coop_barrier(cctr, ++epoch * (uint32_t)G, a.status);
                    collect_window();
                }
                if (!in_window()) break;
                return buffer_select(WIN, red[10], rank - red[11], tracker.lo, tracker.lo + tracker.width, whist, red);
            }
        }
        uint32_t prefix = 0, pmask = 0, rk = rank;
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
            const uint32_t dmask = pass == 2 ? 0x3ffu : 0x7ffu;
            __syncthreads();
            for (int q = tid; q < kBins; q += nt) hist[q] = 0;
            __syncthreads();
            walk(0.f, [&](const f32x4 (&Dv)[4]) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t key = __float_as_uint(fmax_(Dv[r >> 2][r & 3], 0.f));
                    if ((key & pmask) == prefix) atomicAdd(&hist[(key >> shift) & dmask], 1u);
                }
            });
            __syncthreads();
            share_hist();
            if (wave == 0) radix_digit(hist, rk, red, lane);
            __syncthreads();
            prefix |= red[0] << shift;
            rk = red[1];
            pmask |= dmask << shift;
        }
        tracker.density = 0.f;  // no window to measure it in
        return __uint_as_float(prefix);
    };

    for (int it = 0; a.do_svgd && it < a.n_iter; ++it) {
        const bool need_median = (a.bw_mode == 0 || it == 0) && M > 0;
        const bool window = need_median && tracker.plan(M, cap);
        float srow[TS][D];        // scores of this thread's particles

        // (1) scores
        float os[NC], sref = 0.f;
        const int sp = SPLIT ? wave / ntasks : 0;
        if constexpr (CHUNKED) {
            // chunk by chunk, each relative to its own largest logit; the sums so
            // far move to the larger reference
            float tot[NC], tref = kNoSource;
#pragma unroll
            for (int c = 0; c < NC; ++c) tot[c] = 0.f;
            for (int ch = 0; a.trans_mode == 0 && ch < L.chunks; ++ch) {
                first_source = ch * chunk;
                __syncthreads();
                build_vt(first_source);
                build_ms(false, first_source);
                __syncthreads();
                const int nb = chunk / 32;
                if (sp >= L.ns_sc) continue;
                score_sums(tbase + wave % ntasks * kTask, sp * nb / L.ns_sc, (sp + 1) * nb / L.ns_sc, negref[0], os, sref);
                const float top = fmax_(tref, sref), w0 = R::exp2_(tref - top), w1 = R::exp2_(sref - top);
#pragma unroll
                for (int c = 0; c < NC; ++c) tot[c] = tot[c] * w0 + os[c] * w1;
                tref = top;
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) os[c] = tot[c];
            sref = tref;
        }
        if constexpr (SPLIT) {
            // this wave's split of its task's sources
            if (!CHUNKED && a.trans_mode == 0 && sp < L.ns_sc) {
                const int nb = chunk / 32;
                score_sums(tbase + wave % ntasks * kTask, sp * nb / L.ns_sc, (sp + 1) * nb / L.ns_sc, negref[0], os, sref);
            }
        } else {
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                const int task = wave + ts * nwaves;
                if (task >= ntasks) break;
                if (!CHUNKED && a.trans_mode == 0) score_sums(task * kTask, 0, chunk / 32, negref[ts], os, sref);
                const int k = task * kTask + (fresh_tid() & 63);
                if (k < n) {
                    float xt[D];
                    target_x(k, xt);
                    score_grad(xt, srow[ts]);
                    score_transition(os, xt, srow[ts]);
                }
            }
        }
        have_ref = !CHUNKED;

        // (2) the bandwidth needs the exact lower median of the squared
        // distances of the current particles: their window pass
        if (window) window_walk();
        // (the multi-workgroup mode keeps the partial sums over the sums' tables)
        if (COOP) __syncthreads();
        if constexpr (SPLIT) {
            // partial sums of the splits to LDS
            if (a.trans_mode == 0 && sp < L.ns_sc && lane < kTask) {
                float *pp = PART + (sp * ntl + wave % ntasks * kTask + lane) * kPart;
#pragma unroll
                for (int c = 0; c < NC; ++c) pp[c] = os[c];
                pp[NC] = sref;
            }
        }
        __syncthreads();
        bool found = !COOP && window && in_window();
        // the last wave ranks the window's values while the first ones merge
        // the splits
        if (found && red[10] <= kSelectMax && wave == nwaves - 1) select_by_wave();
        if constexpr (SPLIT) {
            const int il = fresh_tid();
            if (il < ntl && tbase + il < n) {
                if (a.trans_mode == 0) merge_part(il, L.ns_sc, true, os);
                float xt[D];
                target_x(tbase + il, xt);
                score_grad(xt, srow[0]);
                score_transition(os, xt, srow[0]);
            }
        }
        if constexpr (COOP) {
            // this workgroup's score rows and its share of the window pass to
            // the exchange area
            if (tid < ntl) {
                float *cs = cS + (long)(tbase + tid) * 8;
#pragma unroll
                for (int c = 0; c < D; ++c) cs[c] = tbase + tid < n ? srow[0][c] : 0.f;
            }
            if (window) publish_window();
            coop_barrier(cctr, ++epoch * (uint32_t)G, a.status);
            // every score row: thread tid takes particle tid
            if (tid < n) {
#pragma unroll
                for (int c = 0; c < D; ++c) srow[0][c] = cS[(long)tid * 8 + c];
            }
            if (window) {
                collect_window();
                found = in_window();
                if (found && red[10] <= kSelectMax && wave == nwaves - 1) select_by_wave();
            }
        }
        __syncthreads();
        if (need_median || it == 0) {
            float med = __builtin_nanf("");
            if (need_median) {
                if (window) tracker.density = uniform((float)min(red[10], cap) / tracker.width);
                if (found && red[10] <= kSelectMax) med = __uint_as_float(red[5]);
                else if (found) med = buffer_select(WIN, red[10], rank - red[11], tracker.lo, tracker.lo + tracker.width, whist, red);
                else med = median_from_range();
                med = uniform(med);
                tracker.record(med);
            }
            h = uniform(bandwidth_from_median(2.f * med, n, a.bw_scale));
        }
        if (a.h_out && tid == 0 && gi == 0) a.h_out[(long)b * a.h_stride + it] = h;
        const float beta = uniform((float)kLog2e / h);

        // (3) Stein direction
        //   phi_i = (sum_k kappa_ki v_k + c2 x_i sum_k kappa_ki) / n,
        //   v_k = s_k - c2 x_k, c2 = 2 / h
        // (the kernel-gradient term of the update folded into the score
        // rows, so one contraction of kappa with [v, 1] gives both sums).
        const float twob = 2.f * beta;
        const float c2 = 2.f / h;
        // B = [2 beta x_i, -2 beta], constant kKapShift - beta n_i: a tile holds the
        // exponent kKapShift - beta |x_k - x_i|^2
        auto stein_target = [&](const PieceRow<K4> &p, float (&v)[NC], float &cst) {
#pragma unroll
            for (int c = 0; c < NC; ++c) v[c] = c == kLast ? -twob : c < D ? twob * p.at(c) : 0.f;
            const float half = p.at(kLast);
            cst = kKapShift - (half < 0.5f * kPadHalfNorm ? twob * half : 0.f);
        };
        const float k_inv = inv_n / kKapScale;
        // What the matrix cores cannot take (kMaxProductExponent, kTinyShare): the
        // table holds the score rows in FP32, and differences are formed.
        bool direct = false;
        float *const srows = (float *)(smem + L.off_v);
        auto put_scores = [&]() {
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                const int k = fresh_tid() + ts * nt;
                if (k >= npad) break;
#pragma unroll
                for (int c = 0; c < D; ++c) srows[k * D + c] = k < n ? srow[ts][c] : 0.f;
            }
        };
        // v of this thread's ts-th particle k
        auto vector = [&](int ts, int k, const PieceRow<K4> &p, float (&w)[D]) {
#pragma unroll
            for (int c = 0; c < D; ++c) w[c] = k < n ? srow[ts][c] - c2 * p.at(c) : 0.f;
        };
        // scales from the largest values (a block-wide barrier before and after)
        auto set_scales = [&]() {
            __syncthreads();
            float mx[D];
#pragma unroll
            for (int c = 0; c < D; ++c) mx[c] = 0.f;
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                const int k = fresh_tid() + ts * nt;
                if (k >= n) break;
                PieceRow<K4> p;
                float w[D];
                p.load(smem, L.off_x, npad, k);
                vector(ts, k, p, w);
#pragma unroll
                for (int c = 0; c < D; ++c) mx[c] = fabsf(w[c]) > mx[c] || w[c] != w[c] ? fabsf(w[c]) : mx[c];
            }
            note_max(mx, 24);
            __syncthreads();
            if (tid < D) {
                redf[40 + tid] = f16_scale(__uint_as_float(red[24 + tid]), 14);
                red[24 + tid] = 0;
            }
            if (tid == 0) red[12] = 0;
            have_scale = true;
            __syncthreads();
        };
        if (!have_scale) set_scales();
        // the table and what stands against it
        auto put_vectors = [&]() {
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                const int k = fresh_tid() + ts * nt;
                if (k >= npad) break;
                PieceRow<K4> p;
                float w[D];
                p.load(smem, L.off_x, npad, k);
                vector(ts, k, p, w);
                bool off = false, tiny = false;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    w[c] *= v_scale[c];
                    off |= !(fabsf(w[c]) < kScaledMax);
                    tiny |= many_tiny(w[c], min(kWave, n - (k & ~(kWave - 1))));
                }
                const bool far = k < n && !(twob * p.at(kLast) <= kMaxProductExponent);
                const uint32_t bad = (tiny || __builtin_amdgcn_ballot_w64(off) ? kRescale : 0u) |
                                     (__builtin_amdgcn_ballot_w64(far) ? kDirect : 0u);
                if (bad) atomicOr(&red[12], bad);
                put_sum_row<D>(smem, L.off_v, k, w, k < n ? 1.f : 0.f);
            }
        };
        put_vectors();
        // (a workgroup that splits has two threads or more per particle: the
        // second puts the target operands)
        constexpr bool kOther = SPLIT && !COOP;
#pragma unroll
        for (int ts = 0; ts < TS; ++ts) {
            const int k = fresh_tid() + ts * nt;
            PieceRow<K4> p;
            float v[NC], cst;
            const int r = kOther ? k - npad : k;
            if (SPLIT && L.b_table && r >= tbase && r < tbase + ntl) {
                p.load(smem, L.off_x, npad, r);
                stein_target(p, v, cst);
                put_target<K4>(smem, L.off_b, ntl, r - tbase, v, cst);
            }
        }
        __syncthreads();
        if (tid < 2) red[10 + tid] = 0;  // the next walk's counters (past the last read)
        uint32_t against = red[12];
        if (__builtin_amdgcn_readfirstlane((int)against)) {
            if (!(against & kDirect)) {
                set_scales();
                put_vectors();
                __syncthreads();
            }
            if (red[12]) {
                direct = true;
                __syncthreads();
                if (tid == 0) red[12] = 0;
                have_scale = false;
                put_scores();
                __syncthreads();
            }
        }
        // sums over the source blocks [blk0, blk1) for the targets of a task
        auto stein_sums = [&](int ibase, int blk0, int blk1, float (&so)[NC]) {
            const int lane = fresh_tid() & 63, g = lane >> 4, col = lane & 15;
            if (direct) {  // (the kernel-gradient term included; no sum of kappa)
                float xi[D], acc[D];
                target_x(ibase + (lane & (kTask - 1)), xi);
#pragma unroll
                for (int c = 0; c < D; ++c) acc[c] = 0.f;
                const int k1 = min(32 * blk1, n);
                for (int k = 32 * blk0; k < k1; ++k) {
                    float df[D], dd = 0.f;
                    target_x(k, df);
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        df[c] = xi[c] - df[c];
                        dd += df[c] * df[c];
                    }
                    const float kap = R::exp2_(-beta * dd);
#pragma unroll
                    for (int c = 0; c < D; ++c) acc[c] += kap * (srows[k * D + c] + c2 * df[c]);
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) so[c] = c < D ? acc[c < D ? c : 0] : 0.f;
                return;
            }
            u32x4 b0[QT], b1[QT];
            f32x4 O[QT];
            SourceRows<K4> src;
            src.init(smem, L.off_x, npad, L.off_ones, g, col);
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                b1[q] = u32x4{0u, 0u, 0u, 0u};
                if (SPLIT && L.b_table) {
                    load_target<K4>(smem, L.off_b, ntl, ibase - tbase + 16 * q + col, g, b0[q], b1[q]);
                } else {
                    PieceRow<K4> p;
                    p.load(smem, L.off_x, npad, ibase + 16 * q + col);
                    float v[NC], cst;
                    stein_target(p, v, cst);
                    target_row(v, cst, g, b0[q], b1[q]);
                }
            }
            weighted_sums(src, L.off_v, b0, b1, blk0, blk1, O);
            collect_rows<D, QT>(O, so);
        };
        // the moved particle and half its squared norm
        auto move = [&](int i, const float *so, float (&xn)[NC]) {
            PieceRow<K4> p;
            p.load(smem, L.off_x, npad, i);
            float nrm = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) xn[c] = 0.f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float xc = p.at(c);
                const float v = xc + a.step * (so[c] * (direct ? inv_n : k_inv * inverse_scale(v_scale[c])) + c2 * xc * (so[kLast] * k_inv));
                xn[c] = v;
                nrm += v * v;
            }
            xn[kLast] = 0.5f * nrm;
        };
        float so[TS][NC];
        if constexpr (SPLIT) {
            const int nb = npad / 32;
            if (sp < L.ns_st)
                stein_sums(tbase + wave % ntasks * kTask, sp * nb / L.ns_st, (sp + 1) * nb / L.ns_st, so[0]);
            if (COOP) __syncthreads();
            if (sp < L.ns_st && lane < kTask) {
                float *pp = PART + (sp * ntl + wave % ntasks * kTask + lane) * kPart;
#pragma unroll
                for (int c = 0; c < NC; ++c) pp[c] = so[0][c];
            }
        } else {
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) {
                const int task = wave + ts * nwaves;
                if (task >= ntasks) break;
                stein_sums(task * kTask, 0, npad / 32, so[ts]);
            }
        }
        __syncthreads();
        // synchronous update: every thread its particles (SPLIT: the first
        // threads, from the splits' partial sums; the next ones in line move
        // the same particles for the score operands)
        if constexpr (SPLIT && !COOP) {
            const int il = fresh_tid(), i = il < ntl ? il : il - ntl;
            const bool mine = i < n && (il < ntl || L.b_table);
            float xn[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) xn[c] = 0.f;
            if (mine) {
                merge_part(i, L.ns_st, false, so[0]);
                move(i, so[0], xn);
            }
            __syncthreads();
            if (mine && il < ntl) put_row<K4>(smem, L.off_x, npad, i, xn);
            // (a pad's Stein operand makes way for its score operand)
            if (il >= ntl && i < ntl) put_score_target(i, xn);
        } else
#pragma unroll
        for (int ts = 0; ts < TS; ++ts) {
            const int il = fresh_tid() + ts * nt;
            const int i = tbase + il;
            if (il >= ntl) break;
            if (SPLIT && L.b_table && i >= n) {
                const float none[NC] = {};
                put_score_target(i, none);
            }
            if (i >= n) break;
            if (SPLIT) merge_part(il, L.ns_st, false, so[ts]);
            float xn[NC];
            move(i, so[ts], xn);
            put_score_target(i, xn);
            if constexpr (COOP) {
#pragma unroll
                for (int c = 0; c < NC; ++c) cX[(long)i * 8 + c] = xn[c];
            } else {
                put_row<K4>(smem, L.off_x, npad, i, xn);
            }
        }
        if constexpr (COOP) {
            // every workgroup's moved particles
            coop_barrier(cctr, ++epoch * (uint32_t)G, a.status);
            if (tid < n) {
                float xn[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) xn[c] = cX[(long)tid * 8 + c];
                put_row<K4>(smem, L.off_x, npad, tid, xn);
            }
        }
        // the sums' tables share their region where LDS is short
        if (!CHUNKED && L.ms_shared) build_ms(false, 0);
        __syncthreads();
    }

    // rows [mh_j, phi_{t-1}(j)] of the forward recursion over the sums' tables
    // (dead by now; chunks: from the previous particles, over every table of
    // theirs), before the particles are written, which may take the previous
    // ones' place
    float *VF = (float *)(smem + (CHUNKED ? L.off_vt : L.off_v));
    for (int j = tid; a.do_viterbi && j < np; j += nt) {
        if constexpr (CHUNKED) {
            float xp[D], mu[D];
#pragma unroll
            for (int c = 0; c < D; ++c) xp[c] = xprev[(long)j * D + c];
            F::mean(m, a.t, xp, mu);
#pragma unroll
            for (int c = 0; c < kLast; ++c) VF[j * NC + c] = c < D ? (mu[c < D ? c : 0] - ref[c < D ? c : 0]) * rs[c] : 0.f;
        } else {
            PieceRow<K4> p;
            p.load(smem, L.off_vt, chunk, j);
#pragma unroll
            for (int c = 0; c < kLast; ++c) VF[j * NC + c] = 0.5f * p.at(c);
        }
        VF[j * NC + kLast] = a.phi_prev ? a.phi_prev[(long)b * a.phi_prev_stride + j] : 0.f;
    }
    __syncthreads();

    bool bad = false;
    const int i_lo = COOP ? tbase : 0, i_hi = COOP ? min(n, tbase + ntl) : n;
    for (int i = i_lo + tid; a.do_svgd && i < i_hi; i += nt) {
        PieceRow<K4> p;
        p.load(smem, L.off_x, npad, i);
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float v = p.at(c) + ref[c];
            bad |= !R::finite(v);
            xg[(long)i * D + c] = v;
        }
    }

    if (a.do_viterbi) {
        for (int i = i_lo + tid; i < i_hi; i += nt) {
            float xs[D], xa[D];
            PieceRow<K4> p;
            p.load(smem, L.off_x, npad, i);
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const float xt = p.at(c);
                xs[c] = xt * rs[c];
                xa[c] = xt + ref[c];
            }
            ArgBest<float> ab{-inf, -inf, 0};
            bool nan_seen = false;
            for (int j = 0; j < np; ++j) {
                float mj[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) mj[c] = VF[j * NC + c];
                float q2 = 0.f;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const float r = xs[c] - mj[c];
                    q2 += r * r;
                }
                const float A = m.log_z - (float)kLn2 * q2;
                const float cij = A + mj[kLast];
                nan_seen |= (cij != cij);
                if (j == 0) { ab.best = cij; ab.arg = 0; }
                else argbest_push(ab, cij, j);
            }
            const float ell = F::loglik(m, sz, mk, xa);
            const float ph = ab.best + ell;
            nan_seen |= (ph != ph);
            bad |= nan_seen;
            a.phi[(long)b * a.phi_stride + i] = ph;
            a.psi[(long)b * a.psi_stride + i] = ab.arg;
            if (a.flags) {
                const float mag = ab.best < 0 ? -ab.best : ab.best;
                const float sc_ = mag > 1.f ? mag : 1.f;
                a.flags[(long)b * a.flags_stride + i] = (np > 1 && ab.second >= ab.best - a.tie_tol * sc_) ? 1 : 0;
            }
        }
    }
    if (bad) atomicOr(a.status, STATUS_NONFINITE);
}

// the step's arguments, the first of its kernel's
__device__ __forceinline__ ConstStepArgs *kernel_args()
{
    return (ConstStepArgs *)__builtin_amdgcn_kernarg_segment_ptr();
}

template <int KIND, int D, bool SPLIT, bool CHUNKED = false>
__global__ __launch_bounds__(kMaxWaves * 64) void k_step_mfma(StepArgs<float> a)
{
    step_mfma_body<KIND, D, kMaxParticles / 64 / kMaxWaves, SPLIT, false, CHUNKED>(kernel_args(), blockIdx.x);
}

// Multi-workgroup step: workgroup blockIdx.x is group blockIdx.x % G of
// sequence blockIdx.x / G (a cooperative launch: all resident at once).
template <int KIND, int D>
__global__ __launch_bounds__(kMaxWaves * 64) void k_step_mfma_coop(StepArgs<float> a, CoopArgs c)
{
    c.gi = (int)(blockIdx.x % (unsigned)c.G);
    step_mfma_body<KIND, D, 1, true, true>(kernel_args(), (int)(blockIdx.x / (unsigned)c.G), c);
}

} // namespace smsq
