// device_common.h — device building blocks of the particle filter (gfx950).
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) keyed by the
// run seed; every draw is a pure function of its logical coordinates, so results
// do not depend on the launch shape. Counter layout:
//   flows       (particle j, filter i, k<<16 | t, 1<<24 | draw b<<16 | call a)
//   PF resample (0, filter i, k<<16 | t, 2<<24); multinomial: slots 2p, 2p+1 from
//                (p, filter i, k<<16 | t, 2<<24 | 1<<16)
//   prior       (sample i, 0, 1<<16, 3<<24 | coordinate d)
//   RW normal   (sample i, 0, k<<16, 4<<24 | coordinate d)
//   outer resample (0, 0, k<<16, 5<<24)
//   learned proposal: initial parameter p (p, 0, 0, 6<<24); training permutation
//   (k, epoch, which, 7<<24)
//   linear-Gaussian state noise (particle j, filter i, k<<16 | t, 8<<24); t = 0 draws
//   the initial state
// Uniforms: u24(x) = (2(x>>9)+1) 2^-24 (exact in FP32); u53 = (2(x64>>12)+1) 2^-53.
//
// Precision: the particle filter works in `real` (float or double). Every
// transcendental is defined as its FP64 value rounded to `real`, every other
// operation is one IEEE operation in `real` (the library is built with
// -ffp-contract=off), so a reimplementation that follows the same definitions
// reproduces each integer decision. Two pieces reach the same result in FP32: the
// square root (correctly rounded) and the BTRS final test's decision (FP32 with an
// error bound, FP64 near the boundary).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fast_fp64.h"

namespace smc2 {

enum : uint32_t { S_PF_PROP = 1u, S_PF_RS = 2u, S_PRIOR = 3u, S_RW = 4u, S_OUTER_RS = 5u, S_MLP_INIT = 6u,
                  S_MLP_PERM = 7u, S_LG = 8u };

struct W4 {
    uint32_t x, y, z, w;
};

// a ^ b ^ c. With V3 on the device, one three-input bitwise vector instruction (truth
// table 0x96) instead of two XORs; it is a vector instruction even for uniform inputs, so
// it is meant for counters that differ per lane, where the XORs are vector work anyway.
template <bool V3> __host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (V3) return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#endif
    return a ^ b ^ c;
}

// V3: the round XORs as three-input vector instructions (per-lane counters)
template <bool V3 = false>
__host__ __device__ __forceinline__ W4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                                uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3<V3>((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3<V3>((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return W4{c0, c1, c2, c3};
}

// (2 (x >> 9) + 1) 2^-24. One funnel shift puts k = x >> 9 under the exponent of 1.0,
// giving 1 + k 2^-23; subtracting 1 - 2^-24 leaves (2k + 1) 2^-24 exactly (the operands
// lie within a factor of two of each other, so the difference is exact).
__device__ __forceinline__ float u24(uint32_t x)
{
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, x, 9u)) - 0x1.fffffep-1f;
}

__host__ __device__ __forceinline__ double u53(uint32_t lo, uint32_t hi)
{
    const uint64_t x = ((uint64_t)hi << 32) | lo;
    return (double)(2ull * (x >> 12) + 1ull) * 0x1p-53;
}

// Box-Muller on one Philox call, first output.
__device__ __forceinline__ double normal_key(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                             uint32_t k1)
{
    const W4 w = philox10(c0, c1, c2, c3, k0, k1);
    const double r = sqrt(-2.0 * log(u53(w.x, w.y)));
    return r * cos(6.283185307179586 * u53(w.z, w.w));
}

__device__ __forceinline__ double normal_call(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint64_t seed)
{
    return normal_key(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ----------------------------------------------------------- precision helpers
// a / b correctly rounded, for positive normal operands whose quotient needs no range
// scaling: a >= 2^-100, b in [2^-100, 2^100], a / b below 2^100. Then the scale steps of
// the general division sequence leave the operands unchanged and its fix-up step passes
// the value through, so the core below gives the same bits as the general division: Markstein's
// scheme (IBM J. Res. Dev. 34, 1990), a reciprocal refined by Newton steps, the quotient and
// its residual corrections, all FMAs.
template <typename real> __device__ __forceinline__ real rdiv_inrange(real a, real b);
template <> __device__ __forceinline__ float rdiv_inrange<float>(float a, float b)
{
    const float y0 = __builtin_amdgcn_rcpf(b);
    const float e = fmaf(-b, y0, 1.0f);
    const float y1 = fmaf(e, y0, y0);
    const float q0 = a * y1;
    const float r0 = fmaf(-b, q0, a);
    const float q1 = fmaf(r0, y1, q0);
    const float r1 = fmaf(-b, q1, a);
    return fmaf(r1, y1, q1);
}
template <> __device__ __forceinline__ double rdiv_inrange<double>(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(fma(-b, y, 1.0), y, y);
    y = fma(fma(-b, y, 1.0), y, y);
    const double q = a * y;
    return fma(fma(-b, q, a), y, q);
}
// Square root correctly rounded, x in [2^-60, 2^60]: in FP32 x times the hardware reciprocal
// root and one residual correction, the general sequence without its scaling and special
// cases (equal to it on every mantissa of [1, 4), checked exhaustively). With the in-range
// division the BTRS set-up takes 39 vector instructions for 55 (1000 SEIR filters, N_x = 1000,
// 150 days: 6.92 -> 6.65 ms; Langevin sampler 12.4 -> 12.1 ms; age-structured sampler 294 ->
// 286 ms).
template <typename real> __device__ __forceinline__ real rsqrt_inrange(real x);
template <> __device__ __forceinline__ float rsqrt_inrange<float>(float x)
{
    const float y = __builtin_amdgcn_rsqf(x);
    const float s = x * y, h = 0.5f * y;
    return fmaf(fmaf(-s, s, x), h, s);
}
template <> __device__ __forceinline__ double rsqrt_inrange<double>(double x)
{
    // Goldschmidt's coupled iteration for the root g and half its reciprocal h, then two
    // residual corrections
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}
// (int) floor(t), saturating at the limits of int32
template <typename real> __device__ __forceinline__ int32_t floor_sat(real t);
template <> __device__ __forceinline__ int32_t floor_sat<float>(float t)
{
    int32_t k;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(k) : "v"(t));
    return k;
}
template <> __device__ __forceinline__ int32_t floor_sat<double>(double t)
{
    int32_t k;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(k) : "v"(floor(t)));
    return k;
}

// Stream of one binomial draw: flows counter without the call index.
struct DrawStream {
    uint32_t j, i, kt, b;
    uint32_t k0, k1;
    __device__ __forceinline__ W4 call(uint32_t a) const
    {
        return philox10<true>(j, i, kt, (S_PF_PROP << 24) | (b << 16) | a, k0, k1);
    }
};

// ----------------------------------------------------------- binomial sampler
// 1/m for m = 1..128, correctly rounded in each precision (compile-time division).
template <typename real> struct RcpTable {
    real v[128];
    constexpr RcpTable() : v()
    {
        for (int i = 0; i < 128; ++i) v[i] = (real)1 / (real)(i + 1);
    }
};
static __constant__ RcpTable<float> c_rcp_f32;
static __constant__ RcpTable<double> c_rcp_f64;
template <typename real> __device__ __forceinline__ real rcp_int(int m);
template <> __device__ __forceinline__ float rcp_int<float>(int m) { return c_rcp_f32.v[m - 1]; }
template <> __device__ __forceinline__ double rcp_int<double>(int m) { return c_rcp_f64.v[m - 1]; }

// Sequential-search inversion of the Binomial(n, p) CDF for p <= 1/2, n p < 10:
// f_0 = (1-p)^n, f_{k+1} = f_k ((n-k) r) / (k+1), r = p/(1-p); stops at the first k
// whose running sum reaches u, when adding a term no longer changes the sum, or
// at k = min(n, 127).
// l1p = log1p(-p) in FP64 (hoisted by callers whose p is fixed per filter), NaN when the
// caller does not have it.
//
// f_0 by the library functions: 42 vector instructions, and 135 more for log1p.
template <typename real> __device__ __forceinline__ real inversion_first(int32_t n, real p, double l1p)
{
    const double lq = (l1p == l1p) ? l1p : log1p(-(double)p);
    return (real)exp((double)n * lq);
}
// FP32: 25 and 18 instructions (age-structured SEIR, 2048 filters x 2048 x 365, two
// iterations: 325 -> 310 ms with leave_prob4)
// n = 1: the value is 1 - p, which for one FP32 p in four lies halfway between two FP32
// values, where nothing short decides: the callers that hoist l1p hoist it too (f1)
__device__ __forceinline__ float inversion_first_fast(int32_t n, float p, double l1p, float f1)
{
    const double lq = (l1p == l1p) ? l1p : log1m_half((double)p);
    float f;
    bool ok = round_safe(exp_neg((double)n * lq), f);
    const bool one = (n == 1) & (l1p == l1p);
    f = one ? f1 : f;
    if (!(ok | one)) f = inversion_first<float>(n, p, l1p);
    return f;
}

template <typename real>
__device__ __forceinline__ int32_t binom_inversion(int32_t n, real p, double l1p, real f1, uint32_t word)
{
    const real u = (real)u24(word);
    const real q = (real)1 - p;
    // in range: p below 2^-100 gives f_0 = 1 > u, whatever the ratio
    const real r = rdiv_inrange<real>(p, q);
    real f;
    if constexpr (sizeof(real) == 4) f = inversion_first_fast(n, p, l1p, f1);
    else f = inversion_first<real>(n, p, l1p);
    real F = f;
    int32_t k = 0;
    const int32_t kcap = n < 127 ? n : 127;
    while (u > F && k < kcap) {
        real t = (real)(n - k) * r;
        t = t * rcp_int<real>(k + 1);
        f = f * t;
        k = k + 1;
        const real Fn = F + f;
        if (Fn == F) break;
        F = Fn;
    }
    return k;
}

// log(x!) for integer-valued x >= 0 in FP64: exact table below 16, Stirling's series
// for log Gamma(x+1) with terms up to (x+1)^-7 above (truncation error < 1e-14).
static __constant__ double c_lfact_tab[16] = {
    0.0, 0.0, 0.69314718055994530942, 1.7917594692280550008, 3.1780538303479456196, 4.7874917427820459942,
    6.5792512120101009951, 8.5251613610654143002, 10.604602902745250228, 12.801827480081469611,
    15.104412573075515295, 17.502307845873885839, 19.98721449566188615, 22.552163853123422886,
    25.1912211827386815, 27.899271383840891566};

__device__ __forceinline__ double lfact(double x)
{
    if (x < 16.0) return c_lfact_tab[(int)x];
    const double z = x + 1.0;
    const double r = 1.0 / z, r2 = r * r;
    const double series = r * (1.0 / 12.0 - r2 * (1.0 / 360.0 - r2 * (1.0 / 1260.0 - r2 * (1.0 / 1680.0))));
    return ((x + 0.5) * log(z) - z) + 0.91893853320467274178 + series;
}

// BTRS transformed rejection (W. Hoermann, J. Stat. Comput. Simul. 46, 1993) for
// p <= 1/2, n p >= 10. Constants, proposal index and squeeze in `real`; the centre
// n p + 1/2 split in FP64 into integer and fraction; the final acceptance test is
// defined in FP64 on log-factorials (btrs_final) and decided FP32-first with an error
// bound (btrs_final_fast, btrs_decide). Attempt e uses words 2(e&1), 2(e&1)+1 of call e>>1.
// The pieces below are shared by the sequential sampler (binom_btrs), the filter's per-draw
// schedule (btrs_first, then the wave's open draws) and its pooled one, which defers final
// tests; all take identical decisions because each piece is a pure function of (n, p, k, words).
template <typename real> struct BtrsConst {
    real spq, bb, aa, vr, cf;
    int32_t ci;
};

// The set-up given its two costly values, spq = sqrt(n p q) and vr = 0.92 - 4.2 / bb.
template <typename real>
__device__ __forceinline__ BtrsConst<real> btrs_setup_from(int32_t n, real p, real spq, real vr)
{
    BtrsConst<real> c;
    c.spq = spq;
    c.bb = (real)1.15 + (real)2.53 * c.spq;
    c.aa = ((real)-0.0873 + (real)0.0248 * c.bb) + (real)0.01 * p;
    c.vr = vr;
    const double cc = (double)n * (double)p + 0.5;
    c.ci = (int32_t)cc;
    c.cf = (real)__builtin_amdgcn_fract(cc);
    return c;
}

template <typename real> __device__ __forceinline__ BtrsConst<real> btrs_setup(int32_t n, real p)
{
    // n p >= 10, p <= 1/2, n < 2^30: n p q in [5, 2^30), bb in [6, 2^17)
    const real spq = rsqrt_inrange<real>(((real)n * p) * ((real)1 - p));
    const real bb = (real)1.15 + (real)2.53 * spq;
    return btrs_setup_from<real>(n, p, spq, (real)0.92 - rdiv_inrange<real>((real)4.2, bb));
}

enum : int { BTRS_OUT = 0, BTRS_ACCEPT = 1, BTRS_FINAL = 2 };

// One attempt from the uniform words (wu, wv): the candidate k, and whether it lies
// outside [0, n], is accepted by the squeeze, or needs the final test.
template <typename real>
__device__ __forceinline__ int btrs_try(const BtrsConst<real>& c, int32_t n, uint32_t wu, uint32_t wv, int32_t& k)
{
    const real u = (real)u24(wu) - (real)0.5;
    const real v = (real)u24(wv);
    const real us = (real)0.5 - (real)fabs((double)u);
    real t = (real)2 * c.aa;
    // in range: 2a with a = -0.0873 + 0.0248 b + 0.01 p in [0.12, 1100] (b = 1.15 + 2.53 sqrt(npq),
    // npq > 9, n < 2^30), over us in [2^-24, 1/2]
    t = rdiv_inrange<real>(t, us);
    t = t + c.bb;
    t = t * u;
    t = t + c.cf;
    // beyond 2^30 in magnitude the candidate lies outside [0, n] (n < 2^30), and so does the
    // sum when the conversion saturates: above it exceeds n or wraps below 0
    k = (int32_t)((uint32_t)c.ci + (uint32_t)floor_sat<real>(t));
    if (k < 0 || k > n) return BTRS_OUT;
    if (us >= (real)0.07 && v <= c.vr) return BTRS_ACCEPT;
    return BTRS_FINAL;
}

// The final acceptance test of candidate k (FP64).
template <typename real>
__device__ __forceinline__ bool btrs_final(const BtrsConst<real>& c, int32_t n, real p, int32_t k, uint32_t wu,
                                           uint32_t wv)
{
    const real u = (real)u24(wu) - (real)0.5;
    const real v = (real)u24(wv);
    const real us = (real)0.5 - (real)fabs((double)u);
    const real q = (real)1 - p;
    const double alpha = (2.83 + 5.1 / (double)c.bb) * (double)c.spq;
    const double lpq = log((double)p / (double)q);
    const double m = floor((double)(n + 1) * (double)p);
    const double h = lfact(m) + lfact((double)n - m);
    const double lhs = log((double)v * alpha / ((double)c.aa / ((double)us * (double)us) + (double)c.bb));
    const double rhs = ((h - lfact((double)k)) - lfact((double)(n - k))) + ((double)k - m) * lpq;
    return lhs <= rhs;
}

// The same test evaluated in FP32 with a bound on its distance from the FP64
// evaluation above; returns 1 (accept), -1 (reject), or 0 when the FP32 value is
// too close to the boundary to decide (then the FP64 test decides). Exact algebra
// on the test: with m = floor((n+1)p), d = k - m, M = m+1, N = n-m+1, A = k+1 = M+d,
// B = n-k+1 = N-d and lfact(x) = (x+1/2) log(x+1) - (x+1) + log(2 pi)/2 + fc(x), the FP64
// right-hand side is
//   -(A-1/2) log(A/M) - (B-1/2) log(B/N) + d log(pN/(qM)) + fc(m) + fc(n-m) - fc(k) - fc(n-k).
// With u1 = d/M, u2 = -d/N and h(u) = (1+u) log(1+u) - u, A log(A/M) = M h(u1) + d and
// B log(B/N) = N h(u2) - d: the linear parts cancel exactly and
//   rhs = -M h(u1) - N h(u2) + log((A/M)(B/N))/2 + d L0 + fc(m) + fc(n-m) - fc(k) - fc(n-k),
// L0 = log(pN/(qM)). Both h are non-negative; for |u| <= 1/8, h(u) = u^2 entropy_curve(u),
// beyond it A log(A/M) - d (and B log(B/N) + d), whose cancelling parts of size |d| enter
// the bound. L0 = log1p(y0), y0 = (pN - qM)/(qM), pN - qM = fr + p - 1 + ((1-p) - q) M with
// fr = (n+1)p - m (q is 1 - p rounded to the filter's precision, as in the FP64 test; its
// error is formed exactly). Reciprocals and base-2 logarithms are the hardware instructions
// (relative error below 2^-22 on gfx950), so every piece carries a relative error of a few
// tens of FP32 units at most and 2^-17 times the sum of the magnitudes bounds the FP32
// error; for n < 2^23, n 2^-41 bounds the FP64 evaluation's own error (terms of size n ln n,
// a few roundings each: 2^-46 (n+1)(1 + log2(n+2))). A decision taken outside both bounds is
// the FP64 decision. Needs n < 2^23 (integers exact in FP32). For the FP64 filters the set-up
// values and p enter rounded to FP32, one more unit each.
// The test is bound by instruction issue, and a wave runs it whenever one lane needs it: 2.5
// times a draw when each attempt runs in place. What depends on (n, p) alone is therefore computed
// once a draw (BtrsFinal, 50 vector instructions), leaving about 90 a test, against 735 for the
// FP64 test (FP64 SIR sampler, 1024 filters x 500 x 30, ten iterations: 10.3 -> 7.8 ms; the
// age-structured sampler, 140 a test -> this: 287 -> 257 ms, Langevin 12.1 -> 11.4 ms).
// Reciprocals and logarithms issue at a quarter of the rate: products share one reciprocal and the
// two logarithms that always enter are one, five of them a test for eight and two a set-up for
// four (1000 SEIR filters, N_x = 1000, 150 days: 5.29 -> 5.16 ms; 50 age-structured filters,
// N_x = 1500, 200 days: 10.2 -> 9.9 ms).
static __constant__ float c_fc_tab[4] = {0.081061466795327f, 0.041340695955409f, 0.027677925684998f,
                                        0.020790672103766f};

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_ln(float x) { return __builtin_amdgcn_logf(x) * 0.693147181f; }

// fc(x), x >= 4, from r = 1 / (x + 1): the Stirling series 1/(12z) - 1/(360z^3), z = x+1
// (the next term, 1/(1260 z^5), is below 2.6e-7)
__device__ __forceinline__ float btrs_fc(float r) { return r * fmaf(r * r, -0.00277777778f, 0.0833333333f); }

// (log1p(x) - x) / x^2 for |x| <= 1/8: the Chebyshev interpolant of degree 5 (relative
// error below 2^-24.9)
__device__ __forceinline__ float log1p_curve(float x)
{
    float h = 0.14549927f;
    h = fmaf(h, x, -0.16963811f);
    h = fmaf(h, x, 0.19998446f);
    h = fmaf(h, x, -0.24998252f);
    h = fmaf(h, x, 0.33333334f);
    return fmaf(h, x, -0.5f);
}

// ((1+u) log(1+u) - u) / u^2 for |u| <= 1/8: the Chebyshev interpolant of degree 4 (relative
// error below 2^-23.2)
__device__ __forceinline__ float entropy_curve(float u)
{
    float h = 0.03368553f;
    h = fmaf(h, u, -0.05046931f);
    h = fmaf(h, u, 0.08333196f);
    h = fmaf(h, u, -0.16666482f);
    return fmaf(h, u, 0.5f);
}

// What the FP32 final test needs of (n, p) alone
struct BtrsFinal {
    float rM, rN;   // 1 / (m+1), 1 / (n-m+1)
    float L0;       // log(p (n-m+1) / (q (m+1)))
    float fmn;      // fc(m) + fc(n-m)
    float alpha;    // (2.83 + 5.1 / b) sqrt(n p q)
    int32_t m;
};

template <typename real> __device__ __forceinline__ BtrsFinal btrs_final_setup(const BtrsConst<real>& c, int32_t n, real p)
{
    BtrsFinal s;
    const real q = (real)1 - p;
    const double mp = (double)(n + 1) * (double)p;  // FP32 p: exact
    s.m = (int32_t)mp;
    const float fr = (float)__builtin_amdgcn_fract(mp);
    const float M = (float)(s.m + 1), N = (float)(n - s.m + 1);
    const float pf = (float)p, qf = (float)q;
    const float qM = qf * M, qN = qf * N;
    const float r = fast_rcp(qM * N);  // all three reciprocals from one
    s.rM = r * qN;
    s.rN = r * qM;
    const float dq = (float)(((real)1 - q) - p);
    const float y0 = fmaf(dq, M, (fr + pf) - 1.0f) * (r * N);
    s.L0 = fabsf(y0) <= 0.125f ? fmaf(y0 * y0, log1p_curve(y0), y0) : fast_ln(1.0f + y0);
    s.fmn = btrs_fc(s.rM) + btrs_fc(s.rN);
    // 5.1 / b from v_r = 0.92 - 4.2 / b (its rounding, 2^-25, is small beside 2.83)
    s.alpha = fmaf(0.92f - (float)c.vr, 5.1f / 4.2f, 2.83f) * (float)c.spq;
    return s;
}

template <typename real>
__device__ __forceinline__ int btrs_final_fast(const BtrsConst<real>& c, const BtrsFinal& s, int32_t n, int32_t k,
                                               uint32_t wu, uint32_t wv)
{
    if (n >= (1 << 23)) return 0;
    const float u = u24(wu) - 0.5f;
    const float v = u24(wv);
    const float us = 0.5f - fabsf(u);
    const float df = (float)(k - s.m);
    const float A = (float)(k + 1), B = (float)(n - k + 1);
    const float u1 = df * s.rM, u2 = -df * s.rN;
    const float a1 = A * s.rM, b1 = B * s.rN;
    float h1 = (df * u1) * entropy_curve(u1), h2 = (-df * u2) * entropy_curve(u2), wide = 0.0f;
    if (fmaxf(fabsf(u1), fabsf(u2)) > 0.125f) {
        if (fabsf(u1) > 0.125f) h1 = fmaf(A, fast_ln(a1), -df);
        if (fabsf(u2) > 0.125f) h2 = fmaf(B, fast_ln(b1), df);
        wide = fabsf(df);
    }
    const float rAB = fast_rcp(A * B);
    float fk = btrs_fc(rAB * B), fnk = btrs_fc(rAB * A);
    if (k < 4) fk = c_fc_tab[k];
    if (n - k < 4) fnk = c_fc_tab[n - k];
    const float f = s.fmn - (fk + fnk);
    // log((A/M)(B/N)) / 2 less the left-hand side log(v alpha / (aa / us^2 + bb)), as one logarithm
    // (beyond its range infinite, and undecided)
    const float us2 = us * us;
    const float y = fmaf((float)c.bb, us2, (float)c.aa) * fast_rcp((v * s.alpha) * us2);
    const float lg = 0.5f * fast_ln((a1 * b1) * (y * y));
    const float hs = h1 + h2;
    const float D = (fmaf(df, s.L0, lg) - hs) + f;
    const float S = ((hs + wide) + fabsf(df * s.L0)) + (fabsf(lg) + 1.0f);
    const float E = fmaf((float)n, 0x1p-41f, 0x1p-17f * S);
    return D > E ? 1 : (D < -E ? -1 : 0);
}

// btrs_final as a call, for the per-draw sampler: the FP64 test is taken only near the
// boundary of the FP32 one, and kept out of line its registers do not weigh on the
// draw loop around it.
template <typename real>
__device__ __attribute__((noinline)) bool btrs_final_call(const BtrsConst<real> c, int32_t n, real p, int32_t k,
                                                          uint32_t wu, uint32_t wv)
{
    return btrs_final<real>(c, n, p, k, wu, wv);
}

// The acceptance decision of a candidate that needs the final test: FP32 first, the
// FP64 test only when the FP32 value cannot decide.
template <typename real>
__device__ __forceinline__ bool btrs_decide(const BtrsConst<real>& c, int32_t n, real p, int32_t k, uint32_t wu,
                                            uint32_t wv)
{
    const int f = btrs_final_fast<real>(c, btrs_final_setup<real>(c, n, p), n, k, wu, wv);
    bool acc = f > 0;
    if (f == 0) acc = btrs_final_call<real>(c, n, p, k, wu, wv);
    return acc;
}

// the value returned when 256 attempts were all rejected: the mode
template <typename real> __device__ __forceinline__ int32_t btrs_mode(int32_t n, real p)
{
    return (int32_t)floor((double)(n + 1) * (double)p);
}

template <typename real>
__device__ __forceinline__ int32_t binom_btrs(int32_t n, real p, const DrawStream& s)
{
    const BtrsConst<real> c = btrs_setup<real>(n, p);
    const BtrsFinal fs = btrs_final_setup<real>(c, n, p);
    W4 w{0u, 0u, 0u, 0u};
    for (int e = 0; e < 256; ++e) {
        if ((e & 1) == 0) w = s.call((uint32_t)(e >> 1));
        const uint32_t wu = (e & 1) ? w.z : w.x;
        const uint32_t wv = (e & 1) ? w.w : w.y;
        int32_t k = 0;
        const int r = btrs_try<real>(c, n, wu, wv, k);
        // The acceptance is merged as a flag and k is returned after the branch: the
        // form "if (quick || final(...)) return k" was miscompiled for gfx950 (the
        // register holding k was reused inside the final test on the accepting path).
        bool acc = r == BTRS_ACCEPT;
        if (r == BTRS_FINAL) {
            const int f = btrs_final_fast<real>(c, fs, n, k, wu, wv);
            acc = f > 0;
            if (f == 0) acc = btrs_final_call<real>(c, n, p, k, wu, wv);
        }
        if (acc) return (int32_t)k;
    }
    return btrs_mode<real>(n, p);
}

// A draw's attempts 0 and 1, one Philox call, as far as one final test goes: attempt 0's when
// attempt 0 needs it, attempt 1's when attempt 0 lies outside [0, n]. True when that settles
// the draw (k is set, the same value as binom_btrs gives): the test runs once for the whole
// wave instead of once an attempt, and one draw in fourteen stays open (from attempt 1 on).
template <typename real>
__device__ __forceinline__ bool btrs_first(int32_t n, real p, const DrawStream& s, int32_t& k)
{
    const BtrsConst<real> c = btrs_setup<real>(n, p);
    const W4 w = s.call(0u);
    int32_t k0 = 0, k1 = 0;
    const int t0 = btrs_try<real>(c, n, w.x, w.y, k0), t1 = btrs_try<real>(c, n, w.z, w.w, k1);
    const bool out = t0 == BTRS_OUT;
    const int t = out ? t1 : t0;
    k = out ? k1 : k0;
    bool acc = t == BTRS_ACCEPT;
    if (t == BTRS_FINAL) acc = btrs_decide<real>(c, n, p, k, out ? w.z : w.x, out ? w.w : w.y);
    const bool second = !acc & !out & (t1 == BTRS_ACCEPT);
    k = second ? k1 : k;
    return acc | second;
}

// Binomial(n, p). l1p, when not NaN, is log1p(-min(p, 1-p)) precomputed in FP64, and f1
// its exponential rounded to `real`.
template <typename real>
__device__ __forceinline__ int32_t binomial(int32_t n, real p, const DrawStream& s, double l1p = NAN, real f1 = (real)0)
{
    if (n <= 0 || !(p > (real)0)) return 0;
    if (p >= (real)1) return n;
    const bool flip = p > (real)0.5;
    const real pp = flip ? (real)1 - p : p;
    int32_t k;
    if ((real)n * pp < (real)10) {
        k = binom_inversion<real>(n, pp, l1p, f1, s.call(0u).x);
    } else {
        k = binom_btrs<real>(n, pp, s);
    }
    return flip ? n - k : k;
}

// The same value, or 0 with open set when its first attempts (btrs_first) leave it open.
template <typename real>
__device__ __forceinline__ int32_t binomial_first(int32_t n, real p, const DrawStream& s, double l1p, real f1, bool& open)
{
    open = false;
    if (n <= 0 || !(p > (real)0)) return 0;
    if (p >= (real)1) return n;
    const bool flip = p > (real)0.5;
    const real pp = flip ? (real)1 - p : p;
    int32_t k = 0;
    if ((real)n * pp < (real)10) {
        k = binom_inversion<real>(n, pp, l1p, f1, s.call(0u).x);
    } else if (!btrs_first<real>(n, pp, s, k)) {
        open = true;
        return 0;
    }
    return flip ? n - k : k;
}

// Probability 1 - exp(-x) of leaving a compartment within a day at hazard x: the FP64 value
// rounded to `real`. FP32: from the short evaluation where that rounds safely (24 vector
// instructions), else the library's expm1 (53; also for x outside [0, 16)).
template <typename real> __device__ __forceinline__ real leave_prob(real x);
template <> __device__ __forceinline__ double leave_prob<double>(double x) { return -expm1(-x); }
template <> __device__ __forceinline__ float leave_prob<float>(float x)
{
    float p;
    const bool ok = round_safe(one_minus_exp_neg((double)x), p);
    if (!(ok & (x >= 0.0f) & (x < 16.0f))) p = (float)(-expm1(-(double)x));
    return p;
}
// four at once, in one block: four independent chains hide each other's latency and share the
// coefficients' scalar moves
template <typename real> __device__ __forceinline__ void leave_prob4(const real (&x)[4], real (&p)[4])
{
    if constexpr (sizeof(real) == 4) {
        // bitwise: a logical and would branch between the chains
        bool ok = true;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            ok = ok & round_safe(one_minus_exp_neg((double)x[g]), p[g]) & (x[g] >= 0.0f) & (x[g] < 16.0f);
        if (!ok) {
#pragma unroll
            for (int g = 0; g < 4; ++g) p[g] = (float)(-expm1(-(double)x[g]));
        }
    } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) p[g] = leave_prob<real>(x[g]);
    }
}

// ----------------------------------------------------------- observations (FP64)
enum : int { OBS_POIS_PREV = 0, OBS_POIS_INC = 1, OBS_NB_INC = 2, OBS_GAUSS = 3 };

// The observation log-pmf split into a per-day constant (no particle dependence)
// and a per-particle part, both FP64:
//   Poisson  log g = [y log(lambda) - lambda] + [-lgamma(y+1)]
//   NB       log g = -[y log1p(r/mu) + r log1p(mu/r)] + [lgamma(y+r) - lgamma(r) - lgamma(y+1)]
// The constant scales every weight equally: it leaves the normalised weights
// unchanged and enters the likelihood increment once per day. The per-particle
// parts have no cancellation, so their rounding to the filter precision is well
// defined. A zero mean gives 0 for y = 0 and -inf otherwise.
__device__ __forceinline__ double obs_const(int obs, int32_t y, double r)
{
    if (obs == OBS_NB_INC) return (lgamma((double)y + r) - lgamma(r)) - lgamma((double)y + 1.0);
    return -lgamma((double)y + 1.0);
}

template <int OBS> __device__ __forceinline__ double obs_part(int32_t y, int32_t cnt, double r)
{
    if (cnt <= 0) return (y == 0) ? 0.0 : -INFINITY;
    const double mu = (double)cnt;
    if (OBS == OBS_NB_INC) return -((double)y * log1p(r / mu) + r * log1p(mu / r));
    return (double)y * log(mu) - mu;
}

// ----------------------------------------------------------- wave / block primitives
// Values that every thread of a workgroup computes identically (block reductions,
// items read from LDS) live in vector registers, so the compiler cannot tell that a
// branch on them is uniform; around workgroup barriers it may then restructure the
// control flow per lane (a persistent work loop was split so that threads other than
// the one that fetches the next item looped without it). Reading such a value through
// readfirstlane makes it a scalar, and branches on it uniform.
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ bool uniform_bool(bool v) { return __builtin_amdgcn_readfirstlane((int)v) != 0; }
__device__ __forceinline__ float uniform_f32(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform_f64(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// true in every lane of the workgroup's first wave, as a scalar (uniform) condition
__device__ __forceinline__ bool first_wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x) == 0; }
template <typename real> __device__ __forceinline__ real uniform_real(real v);
template <> __device__ __forceinline__ float uniform_real<float>(float v) { return uniform_f32(v); }
template <> __device__ __forceinline__ double uniform_real<double>(double v) { return uniform_f64(v); }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }
__device__ __forceinline__ int wave_id() { return (int)(threadIdx.x >> 6); }

// Exchanges between the lanes of a wave, on the vector ALU. Through LDS (ds_bpermute, what a
// shuffle compiles to) a step waits about 60 cycles on top of its issue; six of them per
// reduction, and several reductions a day, set the pace of a small filter (the reductions,
// scans and sums of a day below: 100 linear-Gaussian filters, N_x = 257, 100 days,
// 586 -> 485 us; 1000 SEIR filters, N_x = 1000, 150 days, 7.50 -> 6.92 ms).
// A 32-bit word from another lane by a data-parallel primitive (CTRL); lanes without a source,
// and rows outside ROWS, get 0.
template <int CTRL, int ROWS = 0xF> __device__ __forceinline__ uint32_t dpp_word(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, true);
}
template <int CTRL, int ROWS = 0xF, typename T> __device__ __forceinline__ T dpp(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two words");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp_word<CTRL, ROWS>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = dpp_word<CTRL, ROWS>((uint32_t)u), hi = dpp_word<CTRL, ROWS>((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, lo | (hi << 32));
    }
}
// op of lane l's value and lane l ^ O's, O = 32 or 16: the swap of half waves (of odd and even
// rows) leaves the pair's two values in two registers of both lanes
template <int O, typename T, typename F> __device__ __forceinline__ T swap_step(T v, F op)
{
    const auto sw = [](uint32_t x, uint32_t& a, uint32_t& b) {
        const auto r = O == 32 ? __builtin_amdgcn_permlane32_swap(x, x, false, false)
                               : __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    };
    uint32_t a0, b0;
    if constexpr (sizeof(T) == 4) {
        sw(__builtin_bit_cast(uint32_t, v), a0, b0);
        return op(__builtin_bit_cast(T, a0), __builtin_bit_cast(T, b0));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        uint32_t a1, b1;
        sw((uint32_t)u, a0, b0);
        sw((uint32_t)(u >> 32), a1, b1);
        return op(__builtin_bit_cast(T, (uint64_t)a0 | ((uint64_t)a1 << 32)),
                  __builtin_bit_cast(T, (uint64_t)b0 | ((uint64_t)b1 << 32)));
    }
}
// the butterfly steps 8, 4, 2, 1 within a row of 16 lanes. After step 8 the values repeat
// every 8 lanes, so a rotation by 4 brings lane l ^ 4's value.
template <typename T, typename F> __device__ __forceinline__ T row_reduce(T v, F op)
{
    v = op(v, dpp<0x128>(v));  // rotate by 8
    v = op(v, dpp<0x124>(v));  // rotate by 4
    v = op(v, dpp<0x4E>(v));   // quad lanes 2, 3, 0, 1
    return op(v, dpp<0xB1>(v));  // quad lanes 1, 0, 3, 2
}
template <typename T, typename F> __device__ __forceinline__ T wave_reduce(T v, F op)
{
    return row_reduce(swap_step<16>(swap_step<32>(v, op), op), op);
}

// all 64 lanes active; the butterfly's order of additions (lanes 32, 16, 8, 4, 2, 1 apart)
template <typename T> __device__ __forceinline__ T wave_max(T v)
{
    return wave_reduce(v, [](T x, T u) { return u > x ? u : x; });
}
template <typename T> __device__ __forceinline__ T wave_sum(T v)
{
    return wave_reduce(v, [](T x, T u) { return x + u; });
}

// inclusive scan within a row of 16 lanes, and within a wave (all 64 lanes active)
__device__ __forceinline__ uint64_t row_incl_scan(uint64_t v)
{
    v += dpp<0x111>(v);  // from 1, 2, 4, 8 lanes below in the row
    v += dpp<0x112>(v);
    v += dpp<0x114>(v);
    v += dpp<0x118>(v);
    return v;
}
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v)
{
    v = row_incl_scan(v);
    v += dpp<0x142, 0xA>(v);  // each odd row adds the last lane of the row below it
    v += dpp<0x143, 0xC>(v);  // the upper half adds lane 31
    return v;
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) { return __builtin_bit_cast(uint64_t, uniform_f64(__builtin_bit_cast(double, v))); }

}  // namespace smc2
