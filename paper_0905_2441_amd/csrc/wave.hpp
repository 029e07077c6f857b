// Wavefront (64-lane) and workgroup reductions and scans.
//
// Every reduction here combines values in one fixed order that depends only on
// lane and block indices, so a result is bit-reproducible across launches.
#pragma once
#include <hip/hip_runtime.h>

#include <climits>

#include "dd.hpp"

namespace smc {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / kWave; }

// Orders the wave's LDS accesses before the call against those after it (for
// data one lane writes and other lanes of the same wave read).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The largest and smallest of the wave's 64 values of v, in every lane, by
// DPP row shifts and row broadcasts (no LDS round trips). Floats are compared
// through integer keys that keep their order (a NaN comes out largest or
// smallest, by its sign bit).
__device__ __forceinline__ int float_order_key(float v) {
    const int b = __builtin_bit_cast(int, v);
    return b >= 0 ? b : b ^ 0x7fffffff;
}
__device__ __forceinline__ float float_of_order_key(int k) {
    return __builtin_bit_cast(float, k >= 0 ? k : k ^ 0x7fffffff);
}
template <bool MAX, int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_extreme_step(int v) {
    // a lane whose DPP source is outside its row, or whose row is masked off,
    // reads the operation's identity (so the DPP move folds into the min/max)
    constexpr int kId = MAX ? INT_MIN : INT_MAX;
    const int o = __builtin_amdgcn_update_dpp(kId, v, CTRL, ROW_MASK, 0xf, false);
    return MAX ? (v > o ? v : o) : (v < o ? v : o);
}
template <bool MAX>
__device__ __forceinline__ int wave_extreme_key(int v) {
    v = dpp_extreme_step<MAX, 0x111, 0xf>(v);   // row_shr:1
    v = dpp_extreme_step<MAX, 0x112, 0xf>(v);   // row_shr:2
    v = dpp_extreme_step<MAX, 0x114, 0xf>(v);   // row_shr:4
    v = dpp_extreme_step<MAX, 0x118, 0xf>(v);   // row_shr:8
    v = dpp_extreme_step<MAX, 0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_extreme_step<MAX, 0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ float wave_max_dpp(float v) {
    return float_of_order_key(wave_extreme_key<true>(float_order_key(v)));
}
__device__ __forceinline__ float wave_min_dpp(float v) {
    return float_of_order_key(wave_extreme_key<false>(float_order_key(v)));
}

// The sum of the wave's 64 values of v, in every lane: an inclusive scan within
// each row of 16 lanes by DPP row shifts (a source outside the row reads 0),
// then the row totals carried up by row broadcasts, so lane 63 ends with the
// total. The order of the additions is fixed.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add_step(float v) {
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf,
                                              true);
    return v + __builtin_bit_cast(float, o);
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
    v = dpp_add_step<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add_step<0x112, 0xf>(v);   // row_shr:2
    v = dpp_add_step<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add_step<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add_step<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add_step<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// FP64 values through the same DPP moves, two dwords each. A lane whose source is
// outside its row, or whose row is masked off, gets `id`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v, double id) {
    const long long b = __builtin_bit_cast(long long, v);
    const long long i = __builtin_bit_cast(long long, id);
    const int lo = __builtin_amdgcn_update_dpp(static_cast<int>(i), static_cast<int>(b), CTRL,
                                               ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(static_cast<int>(i >> 32),
                                               static_cast<int>(b >> 32), CTRL, ROW_MASK, 0xf,
                                               false);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) |
                                          static_cast<long long>(static_cast<unsigned>(lo)));
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), lane);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) |
                                          static_cast<long long>(static_cast<unsigned>(lo)));
}

// The wave's sum and maximum in every lane, in the order of an inclusive scan
// (about 150 cycles; a butterfly of lane shuffles goes through LDS, 12 dependent
// accesses of about 130 cycles).
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0x111, 0xf>(v, 0.0);   // row_shr:1
    v += dpp_move<0x112, 0xf>(v, 0.0);   // row_shr:2
    v += dpp_move<0x114, 0xf>(v, 0.0);   // row_shr:4
    v += dpp_move<0x118, 0xf>(v, 0.0);   // row_shr:8
    v += dpp_move<0x142, 0xa>(v, 0.0);   // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v, 0.0);   // row_bcast:31 into rows 2 and 3
    return read_lane(v, kWave - 1);
}
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move<0x111, 0xf>(v, -INFINITY));
    v = fmax(v, dpp_move<0x112, 0xf>(v, -INFINITY));
    v = fmax(v, dpp_move<0x114, 0xf>(v, -INFINITY));
    v = fmax(v, dpp_move<0x118, 0xf>(v, -INFINITY));
    v = fmax(v, dpp_move<0x142, 0xa>(v, -INFINITY));
    v = fmax(v, dpp_move<0x143, 0xc>(v, -INFINITY));
    return read_lane(v, kWave - 1);
}

// Inclusive double-double scan over the wave's lanes.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ dd dpp_scan_step(dd v) {
    const dd up{dpp_move<CTRL, ROW_MASK>(v.hi, 0.0), dpp_move<CTRL, ROW_MASK>(v.lo, 0.0)};
    return dd_add(up, v);
}
__device__ __forceinline__ dd wave_scan(dd v) {
    v = dpp_scan_step<0x111, 0xf>(v);
    v = dpp_scan_step<0x112, 0xf>(v);
    v = dpp_scan_step<0x114, 0xf>(v);
    v = dpp_scan_step<0x118, 0xf>(v);
    v = dpp_scan_step<0x142, 0xa>(v);
    return dpp_scan_step<0x143, 0xc>(v);
}

}  // namespace smc
