// FP64 exponentials, shorter than the device library's (about 45 instructions).
//
// Both take an integer power of two out by adding 1.5 * 2^52, whose low word is
// then the nearest integer (v_cvt_i32_f64 issues at half rate), and a polynomial
// in the remainder.
#pragma once
#include <hip/hip_runtime.h>

namespace smc {

constexpr double kRound64 = 6755399441055744.0;        // 1.5 * 2^52

__device__ __forceinline__ int low_word(double r) {
    return static_cast<int>(__builtin_bit_cast(long long, r));
}

// 2^t for |t| < 2^31 (0 below the FP64 range, NaN for NaN), 14 instructions: the
// least-squares fit of the relative error of 2^f at Chebyshev nodes of [-1/2, 1/2]
// with the constant term 1, degree 10. Its error is below 2.5e-16 and the function's
// below 3.5e-16 (over 10^6 arguments); the likelihoods' is no larger for a higher
// degree.
__device__ __forceinline__ double exp2_fp64(double t) {
    const double r = t + kRound64;
    const double f = t - (r - kRound64);
    double p = 7.041923263577725e-09;
    p = fma(p, f, 1.020852183362834e-07);
    p = fma(p, f, 1.3215629590371928e-06);
    p = fma(p, f, 1.5252658206764617e-05);
    p = fma(p, f, 0.0001540353004830873);
    p = fma(p, f, 0.0013333558228392813);
    p = fma(p, f, 0.0096181291079336);
    p = fma(p, f, 0.05550410866446);
    p = fma(p, f, 0.2402265069590925);
    p = fma(p, f, 0.6931471805599497);
    p = fma(p, f, 1.0);
    return __builtin_amdgcn_ldexp(p, low_word(r));
}

// e^x for x < 709 (0 below -746 and for -infinity, NaN for NaN), 24 instructions.
// The remainder f = x - n ln2 takes ln2 in two parts, the first of 42 bits so that
// its product with n is exact; e^f = 1 + (f + f^2 q(f)), q of degree 10 through
// Chebyshev nodes (3e-19), and 1 + f is kept with its rounding error, so that only
// the last addition's rounding is left: relative error below 1.3e-16 over 10^6
// arguments, where the device library's exp has 1.4e-16 (a form in 2^f with the
// product x log2(e) in two parts has 1.9e-16).
__device__ __forceinline__ double exp_fp64(double x) {
    constexpr double kLn2Hi = 0.6931471805598903;      // ln2 to 42 bits
    constexpr double kLn2Lo = 5.497923018708371e-14;   // and the rest
    const double r = fma(x, 1.4426950408889634, kRound64);
    const double n = r - kRound64;
    const double f = fma(n, -kLn2Lo, fma(n, -kLn2Hi, x));
    double p = 2.09147553258932e-09;
    p = fma(p, f, 2.5105312729622103e-08);
    p = fma(p, f, 2.755727347871858e-07);
    p = fma(p, f, 2.755725517000089e-06);
    p = fma(p, f, 2.480158732567746e-05);
    p = fma(p, f, 0.0001984126987500228);
    p = fma(p, f, 0.0013888888888883711);
    p = fma(p, f, 0.008333333333326084);
    p = fma(p, f, 0.04166666666666667);
    p = fma(p, f, 0.1666666666666667);
    p = fma(p, f, 0.5);
    const double s = 1.0 + f;
    const double e = f - (s - 1.0);
    return x < -746.0 ? 0.0 : __builtin_amdgcn_ldexp(s + fma(f * f, p, e), low_word(r));
}

}  // namespace smc
