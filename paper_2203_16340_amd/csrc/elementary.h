// log and log1p in fp64 for the kernels that evaluate one per entry and step length (entropy regulariser, logistic loss).
//
// Those kernels are bound by instructions, and the runtime's logarithm, which carries two-word arithmetic throughout, takes
// 118 of them (76 in fp64), its log1p 154 (113).  These take 60 and 70.  Method: x = 2^e m with m in [sqrt(1/2), sqrt(2)),
// f = m - 1 (exact), s = f / (2 + f), log(1 + f) = log((1 + s)/(1 - s)) = f - f^2/2 + s (f^2/2 + R), R = s^2 P(s^2) with
// P(z) = 2/3 + 2 z/5 + 2 z^2/7 + ...  Everything but f is small against f, so only the last sums round at the result's size.
// P: the polynomial through the series at the 8 Chebyshev nodes of [0, ((sqrt(2)-1)/(sqrt(2)+1))^2] (relative error of the
// logarithm 2^-60.7).  log 2 in two words, the first a multiple of 2^-32, so that e times it is exact.
// Largest error found over 2 10^7 arguments in each of nine ranges: 0.67 units in the last place.
#pragma once

#include <cmath>
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define LB_BOTH __host__ __device__ __forceinline__
#else
#define LB_BOTH inline
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

// log(u) + small for finite u > 0; small: what the rounding of u took away, divided by u
LB_BOTH double log_and_rest(double u, double small) {
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
    const double f = m - 1.0, z2 = 2.0 + f;
    double y = reciprocal_seed(z2);
    y = __builtin_fma(__builtin_fma(-z2, y, 1.0), y, y);
    double s = f * y;
    s = __builtin_fma(__builtin_fma(-z2, s, f), y, s);
    const double z = s * s;
    double p = 0x1.0c051669ed052p-3;
    p = __builtin_fma(p, z, 0x1.0fbe71adfbddap-3);
    p = __builtin_fma(p, z, 0x1.3b1c36b44161bp-3);
    p = __builtin_fma(p, z, 0x1.745cf8fe32a46p-3);
    p = __builtin_fma(p, z, 0x1.c71c720168523p-3);
    p = __builtin_fma(p, z, 0x1.2492492476c42p-2);
    p = __builtin_fma(p, z, 0x1.9999999999a38p-2);
    p = __builtin_fma(p, z, 0x1.5555555555555p-1);
    const double half_ff = 0.5 * f * f, de = (double)e;
    // de log2 + f - f^2/2 with what the rounding of each step takes away, then the rest
    const double ff_rest = __builtin_fma(0.5 * f, f, -half_ff);
    const double a = f - half_ff, a_rest = (f - a) - half_ff;
    const double k = de * 0x1.62e42fee00000p-1, b = k + a, b_rest = (k - b) + a;   // (k is zero or the larger of the two)
    const double tail = __builtin_fma(s, __builtin_fma(z, p, half_ff), __builtin_fma(de, 0x1.a39ef35793c76p-33, small));
    return b + (b_rest + (a_rest + (tail - ff_rest)));
}

// a/z for z in [1, 2] and |a| <= 1: one Newton step on the reciprocal, then the quotient corrected by its own residue (off by at
// most 0.51 units in the last place; without the scaling that a quotient of any two numbers needs, 6 instructions for 11)
LB_BOTH double quotient_d(double a, double z) {
    double y = reciprocal_seed(z);
    y = __builtin_fma(__builtin_fma(-z, y, 1.0), y, y);
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-z, q, a), y, q);
}

LB_BOTH double log_d(double x) {
    const double r = log_and_rest(x, 0.0);
    // (zero, infinite, negative or no number: -infinity, infinity, no number)
    return x > 0.0 && x < INFINITY ? r : (x == 0.0 ? -INFINITY : (x > 0.0 ? x : NAN));
}

LB_BOTH double log1p_d(double x) {
    const double u = 1.0 + x, big = u - 1.0;
    const double rest = (1.0 - (u - big)) + (x - big);           // (1 + x) - u, exactly
    // rest / u: for small x as large as x itself, so it needs every bit (with the bare seed log1p was off by 10^-8 at 10^-10)
    double y = reciprocal_seed(u);
    y = __builtin_fma(__builtin_fma(-u, y, 1.0), y, y);
    double small = rest * y;
    small = __builtin_fma(__builtin_fma(-u, small, rest), y, small);
    const double r = log_and_rest(u, small);
    return u > 0.0 && u < INFINITY ? r : (u == 0.0 ? -INFINITY : (u > 0.0 ? u : NAN));
}

}  // namespace lb
