// fast_fp64.h — short FP64 evaluations whose result is wanted in FP32 (gfx950).
//
// The FP32 filters define a transcendental as its FP64 value rounded to FP32. The library
// functions give that FP64 value to the last bit, at 50 to 280 instructions (without FP
// contraction a log1p is 135 vector instructions); an FP32 result needs 24 of those bits.
// Each function here evaluates in FP64 with a relative error below 2^-41 and returns the
// FP32 value only when every number within 2^-40 of the evaluation rounds to it; then the
// library's value rounds to it too. Otherwise (about one call in 2^15) the caller takes
// the library function. The FP32 results are therefore the same bits.
//
// FP64 instructions issue at the FP32 rate on gfx950, so instructions are what counts.
// Two forms keep them few: polynomial steps whose coefficient sits in a scalar register
// pair (the compiler otherwise moves every coefficient into a vector pair first, two more
// vector instructions a step), and quotients from the hardware reciprocal with one Newton
// step (measured relative error below 2^-47) in place of the correctly rounded division.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace smc2 {

// a b + c, a + c, a c with the coefficient c in scalar registers
__device__ __forceinline__ double fma_s(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}
__device__ __forceinline__ double fma_m(double a, double c, double b)  // a c + b
{
    double d;
    asm("v_fma_f64 %0, %1, %3, %2" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}
__device__ __forceinline__ double add_s(double a, double c)
{
    double d;
    asm("v_add_f64 %0, %1, %2" : "=v"(d) : "v"(a), "s"(c));
    return d;
}
__device__ __forceinline__ double mul_s(double a, double c)
{
    double d;
    asm("v_mul_f64 %0, %1, %2" : "=v"(d) : "v"(a), "s"(c));
    return d;
}

// a / b for normal operands and quotient: hardware reciprocal and one Newton step
__device__ __forceinline__ double quot_fast(double a, double b)
{
    const double y0 = __builtin_amdgcn_rcp(b);
    const double e = fma(-b, y0, 1.0);
    return a * fma(e, y0, y0);
}

// 2 atanh(s) for |s| <= 1/3: s times a polynomial of degree 7 in s^2, the Chebyshev
// interpolant on [0, 1/9] (relative error below 2^-43.7)
__device__ __forceinline__ double atanh2_third(double s)
{
    const double z = s * s;
    double p = fma_s(z, 0x1.9afeeeabf4dc1p-3, 0x1.202b4d748c2edp-3);
    p = fma_s(p, z, 0x1.76fd5c92728f9p-3);
    p = fma_s(p, z, 0x1.c6f8ad632fa9ep-3);
    p = fma_s(p, z, 0x1.2492cc4fabee3p-2);
    p = fma_s(p, z, 0x1.999997c399b24p-2);
    p = fma_s(p, z, 0x1.5555555694e91p-1);
    p = fma_s(p, z, 0x1.ffffffffffdc7p+0);
    return s * p;
}

// expm1(r) for |r| <= 0.35: r times a polynomial of degree 8, the Chebyshev interpolant
// (relative error below 2^-43.2)
__device__ __forceinline__ double expm1_reduced(double r)
{
    double p = fma_s(r, 0x1.72cbc2d115ac0p-19, 0x1.a160af3a7fe30p-16);
    p = fma_s(p, r, 0x1.a019aa4cb1c39p-13);
    p = fma_s(p, r, 0x1.6c164950be7a3p-10);
    p = fma_s(p, r, 0x1.1111111cf461cp-7);
    p = fma_s(p, r, 0x1.555555760904bp-5);
    p = fma_s(p, r, 0x1.555555555395fp-3);
    p = fma_s(p, r, 0x1.fffffffff6629p-2);
    p = fma(p, r, 1.0);
    return r * p;
}

// 1 - exp(-x), 0 <= x < 16: exp(-x) = 2^k exp(r) with |r| <= log(2) / 2, so the value is
// (1 - 2^k) - 2^k expm1(r); for k = 0 it is -expm1(r) and keeps its relative accuracy
__device__ __forceinline__ double one_minus_exp_neg(double x)
{
    const double k = rint(mul_s(x, -0x1.71547652b82fep+0));
    const double q = expm1_reduced(fma_m(k, -0x1.62e42fefa39efp-1, -x));
    const double sc = __builtin_amdgcn_ldexp(1.0, (int)k);
    return fma(-sc, q, 1.0 - sc);
}

// exp(t), -700 < t <= 0
__device__ __forceinline__ double exp_neg(double t)
{
    const double k = rint(mul_s(t, 0x1.71547652b82fep+0));
    const double q = expm1_reduced(fma_m(k, -0x1.62e42fefa39efp-1, t));
    return __builtin_amdgcn_ldexp(1.0 + q, (int)k);
}

// log1p(-p), 0 < p <= 1/2: -2 atanh(p / (2 - p)), the argument within 1/3 (degree 8,
// relative error below 2^-47 with the quotient's)
__device__ __forceinline__ double log1m_half(double p)
{
    const double s = quot_fast(p, 2.0 - p);
    const double z = s * s;
    double a = fma_s(z, 0x1.802a101eedabfp-3, 0x1.e113009e29adap-4);
    a = fma_s(a, z, 0x1.3ee359d54f9bep-3);
    a = fma_s(a, z, 0x1.741ba33d08379p-3);
    a = fma_s(a, z, 0x1.c71f002282a8cp-3);
    a = fma_s(a, z, 0x1.2492420132b9cp-2);
    a = fma_s(a, z, 0x1.999999ad7f31fp-2);
    a = fma_s(a, z, 0x1.555555554ab02p-1);
    a = fma_s(a, z, 0x1.0000000000007p+1);
    return -(s * a);
}

// log(x) + c for x > 0 normal: x = f 2^e with f in [1/2, 1), log x = e log 2 + log sqrt(1/2)
// + 2 atanh((f - sqrt(1/2)) / (f + sqrt(1/2))), the last argument within 0.1716 (degree 5,
// error below 2^-45); c1 = c + log sqrt(1/2). Absolute error below 2^-44 (1 + |result|).
__device__ __forceinline__ double log_plus(double x, double c1)
{
    constexpr double R = 0x1.6a09e667f3bcdp-1;
    const double f = __builtin_amdgcn_frexp_mant(x);
    const double e = (double)__builtin_amdgcn_frexp_exp(x);
    const double s = quot_fast(add_s(f, -R), add_s(f, R));
    const double z = s * s;
    double p = fma_s(z, 0x1.9193ad28d294dp-3, 0x1.c620e125f3027p-3);
    p = fma_s(p, z, 0x1.24943845c8aa0p-2);
    p = fma_s(p, z, 0x1.9999962baa8c9p-2);
    p = fma_s(p, z, 0x1.55555556716d9p-1);
    p = fma_s(p, z, 0x1.fffffffffff12p+0);
    return fma(s, p, fma(e, 0x1.62e42fefa39efp-1, c1));
}

// the FP32 rounding of every number within 2^-40 of x (x >= 0 or +inf), in lo when it is
// one value; false when it is not (or x is NaN)
__device__ __forceinline__ bool round_safe(double x, float& lo)
{
    lo = (float)mul_s(x, 1.0 - 0x1p-40);
    return lo == (float)mul_s(x, 1.0 + 0x1p-40);
}

// y log1p(r / mu) + r log1p(mu / r), the particle's part of minus the negative-binomial
// log-pmf, for mu >= 1, y >= 0 and r in [2^-30, 2^30] (lr1 = log sqrt(1/2) - log r). With
// L1 = log1p(min / max) = 2 atanh(min / (2 max + min)) and L2 = |log mu - log r| the two
// logarithms are L1 and L1 + L2, so the sum is (y + r) L1 + (mu > r ? r : y) L2: every
// term is non-negative and nothing cancels.
__device__ __forceinline__ double nb_cost(double y, double mu, double r, double lr1)
{
    const double mx = fmax(mu, r), mn = fmin(mu, r);
    const double l1 = atanh2_third(quot_fast(mn, fma(2.0, mx, mn)));
    const double l2 = fabs(log_plus(mu, lr1));
    return fma(y + r, l1, (mu > r ? r : y) * l2);
}

}  // namespace smc2
