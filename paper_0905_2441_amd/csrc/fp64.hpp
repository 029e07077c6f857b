// FP64 exponentials, shorter than the device library's (about 45 instructions).
//
// Both take an integer power of two out by adding 1.5 * 2^52, whose low word is
// then the nearest integer (v_cvt_i32_f64 issues at half rate), and a polynomial
// in the remainder f in [-1/2, 1/2]: the least-squares fit of the relative error
// of 2^f at Chebyshev nodes with the constant term 1, rounded to FP64.
#pragma once
#include <hip/hip_runtime.h>

namespace smc {

constexpr double kRound64 = 6755399441055744.0;        // 1.5 * 2^52

__device__ __forceinline__ int low_word(double r) {
    return static_cast<int>(__builtin_bit_cast(long long, r));
}

// 2^t for |t| < 2^31 (0 below the FP64 range, NaN for NaN): degree 10, relative
// error below 2.5e-16, 14 instructions.
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

// e^x for x < 709 (0 below -746 and for -infinity, NaN for NaN): the product
// x log2(e) is carried in two parts, degree 11, relative error below 4e-17 before
// the evaluation's own rounding; 20 instructions.
__device__ __forceinline__ double exp_fp64(double x) {
    constexpr double kL = 1.4426950408889634;          // log2(e) in two parts
    constexpr double kLlo = 2.0355273740931033e-17;
    const double r = fma(x, kL, kRound64);
    double f = fma(x, kL, -(r - kRound64));
    f = fma(x, kLlo, f);
    double p = 4.4307278984014654e-10;
    p = fma(p, f, 7.073810155099862e-09);
    p = fma(p, f, 1.0178229258049394e-07);
    p = fma(p, f, 1.3215435106247474e-06);
    p = fma(p, f, 1.5252733412140717e-05);
    p = fma(p, f, 0.00015403530457518835);
    p = fma(p, f, 0.0013333558146874727);
    p = fma(p, f, 0.009618129107593736);
    p = fma(p, f, 0.05550410866481954);
    p = fma(p, f, 0.24022650695910133);
    p = fma(p, f, 0.6931471805599453);
    p = fma(p, f, 1.0);
    return x < -746.0 ? 0.0 : __builtin_amdgcn_ldexp(p, low_word(r));
}

}  // namespace smc
