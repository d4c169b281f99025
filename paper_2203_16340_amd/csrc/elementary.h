// log and log1p in fp64 for the kernels that evaluate one per entry and step length (entropy regulariser, logistic loss).
//
// Those kernels are bound by instructions, and the runtime's logarithm, which carries two-word arithmetic throughout, takes
// 116 of them (76 in fp64), its log1p 152 (113).  These take 84 (39) and 101 (51), a load, a store and the constants included,
// and are more accurate.  Method (the classical one, as in
// fdlibm's e_log.c and s_log1p.c; coefficients and rounding corrections are this file's own): x = 2^e m with m in
// [sqrt(1/2), sqrt(2)), f = m - 1 (exact), s = 2 f / (2 + f), log(1 + f) = log((1 + s/2)/(1 - s/2)) = s + s^3 P(s^2) with
// P(z) = 1/12 + z/80 + z^2/448 + ...  The quotient s is held in two words, its first sum with e log 2 is kept with what its
// rounding takes away, and everything else is small against the result (1 % of it at most), so that only the last sum rounds at
// the result's size.
// P: the polynomial through the series at the 8 Chebyshev nodes of [0, 4 ((sqrt(2)-1)/(sqrt(2)+1))^2] (relative error of the
// logarithm 2^-60.7).  log 2 in two words, the first a multiple of 2^-32, so that e times it is exact.
// Every rounding above is meant to happen: contraction into fused multiply-adds is off where it would change one.
// Largest error on the device, units in the last place, over 2 10^6 arguments per range, runtime / these: log on [1/2, 2]
// 0.635 / 0.550, on [1e-300, 1e300] 0.625 / 0.523; log1p on [-1/2, 1] 0.638 / 0.571, +-[1e-16, 1e-6] 0.500 / 0.500.
#pragma once

#include <cmath>
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define LB_BOTH __host__ __device__ __forceinline__
#else
#define LB_BOTH inline
#endif
#ifdef __clang__
#define LB_NO_CONTRACTION _Pragma("clang fp contract(off)")
#else
#define LB_NO_CONTRACTION   // (the host's tests are compiled with -ffp-contract=off)
#endif

namespace lb {

// 1/z to about 24 bits (the hardware's: 2^-24.4 over [0.8, 3]; the host's, which stands in for it in tests, is worse: 2^-23)
LB_BOTH double reciprocal_seed(double z) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcp(z);
#else
    return (double)(1.0f / (float)z) * (1.0 - 0x1p-24);
#endif
}

// log(u + rest) for finite u > 0.  REST false: rest is zero; else what the rounding of u took away, so at most half a unit of
// u's last place, and |log| is at least 2^-36 (s and its second word are then far apart).
template <bool REST>
LB_BOTH double log_of_sum(double u, double rest) {
    LB_NO_CONTRACTION
#ifdef __HIP_DEVICE_COMPILE__
    double m = __builtin_amdgcn_frexp_mant(u);
    int e = __builtin_amdgcn_frexp_exp(u);
#else
    int e;
    double m = std::frexp(u, &e);
#endif
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, f_rest = REST ? __builtin_ldexp(rest, -e) : 0.0;
    // z + z_rest = 1 + (f + f_rest)/2
    const double z = __builtin_fma(0.5, f, 1.0);
    double z_rest = __builtin_fma(0.5, f, 1.0 - z);
    if (REST) z_rest = __builtin_fma(0.5, f_rest, z_rest);
    // (two steps: with one, the 2^-48 that s would be off count in s^3)
    double y = reciprocal_seed(z);
    y = __builtin_fma(__builtin_fma(-z, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-z, y, 1.0), y, y);
    // s + s_rest = (f + f_rest) / (z + z_rest)
    const double s = f * y;
    double r = __builtin_fma(-s, z_rest, __builtin_fma(-s, z, f));
    if (REST) r += f_rest;
    const double s_rest = r * y, ss = s * s;
    double p = 0x1.0c051669ed052p-20;
    p = __builtin_fma(p, ss, 0x1.0fbe71adfbddap-18);
    p = __builtin_fma(p, ss, 0x1.3b1c36b44161bp-16);
    p = __builtin_fma(p, ss, 0x1.745cf8fe32a46p-14);
    p = __builtin_fma(p, ss, 0x1.c71c720168523p-12);
    p = __builtin_fma(p, ss, 0x1.2492492476c42p-9);
    p = __builtin_fma(p, ss, 0x1.9999999999a38p-7);
    p = __builtin_fma(p, ss, 0x1.5555555555555p-4);
    const double de = (double)e;
    const double k = de * 0x1.62e42fee00000p-1, b = k + s, b_rest = (k - b) + s;   // (k is zero or the larger of the two)
    const double tail = __builtin_fma(de, 0x1.a39ef35793c76p-33, __builtin_fma(s * ss, p, s_rest));
    return b + (b_rest + tail);
}

// a/z for z in [1, 2] and |a| <= 1: one Newton step on the reciprocal, then the quotient corrected by its own residue, which
// leaves 2^-90 (without the scaling that a quotient of any two numbers needs, 6 instructions for 11; the same bits as the
// division in each of 2 10^6 values of the logistic function)
LB_BOTH double quotient_d(double a, double z) {
    double y = reciprocal_seed(z);
    y = __builtin_fma(__builtin_fma(-z, y, 1.0), y, y);
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-z, q, a), y, q);
}

LB_BOTH double log_d(double x) {
    const double r = log_of_sum<false>(x, 0.0);
    // (zero, infinite, negative or no number: -infinity, infinity, no number)
    return x > 0.0 && x < INFINITY ? r : (x == 0.0 ? -INFINITY : (x > 0.0 ? x : NAN));
}

LB_BOTH double log1p_d(double x) {
    LB_NO_CONTRACTION
    const double u = 1.0 + x, big = u - 1.0;
    const double rest = (1.0 - (u - big)) + (x - big);           // (1 + x) - u, exactly
    double r = log_of_sum<true>(u, rest);
    // (the series; the next term is 2^-71 of x)
    r = std::fabs(x) < 0x1p-35 ? __builtin_fma(-0.5 * x, x, x) : r;
    return u > 0.0 && u < INFINITY ? r : (u == 0.0 ? -INFINITY : (u > 0.0 ? u : NAN));
}

}  // namespace lb
