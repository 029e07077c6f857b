// Device helpers shared by the mixture likelihood kernels (VALU and MFMA forms).
#pragma once
#include <type_traits>

#include "cdf_search.hpp"
#include "fp64.hpp"
#include "internal.hpp"
#include "philox.hpp"
#include "wave.hpp"

namespace smc {

constexpr double kLn2 = 0.6931471805599453;
constexpr double kLog2e = 1.4426950408889634;

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int PREC>
__device__ __forceinline__ double finish_loglik(double acc, int n, const GmmDev& g) {
    const double body = (PREC == SMC_PREC_FP32) ? kLn2 * acc : acc;
    return static_cast<double>(n) * g.cst + body;
}

// Sum over data j in [j0, j1) of log2 sum_i 2^{a_ij}, a_ij = log2 w_i - s^2 ||y_j - mu_i||^2
// (FP32 per-datum arithmetic, FP64 result). Per-datum factors are multiplied
// into a running FP32 product that is renormalised (frexp) after each block of
// data, its exponents summed as integers. Three forms:
//  - pivot (1-D data with a staging row, slices of at least kPivotMinData
//    data): the slice goes window by window, 64 data at a time. In a window
//    with midpoint c and half-width h, each particle takes as its pivot p the
//    component with the largest exponent at c. The difference of two
//    exponents is linear in y, so
//      log2 sum_i 2^{a_ij} = a_pj + log2(1 + sum_{i != p} 2^{t_ij}),
//      t_ij = dX_i + dB_i (y_j - c),  dX_i = a_i(c) - a_p(c) <= 0,
//      dB_i = 2 s^2 (mu_i - mu_p),
//    and sum_j a_pj over the window follows in FP64 from two sums over the
//    window's data (of y_j - c and of its square) that every particle shares.
//    Per datum and particle that is at most K-1 FMAs, K-1 exp2, K-2 adds and
//    one FMA into the product: each particle orders its other components by
//    the largest t_ij the window can hold, and the wave takes only as many as
//    its neediest particle has that can reach 2^kPivotSkip (near the data
//    mostly the one or two nearest neighbours of the pivot; the terms left out
//    are below the factor's FP32 resolution). Every factor is at least 1, so
//    the product cannot
//    underflow; a window is taken when, for every particle of the wave, every
//    dX_i + |dB_i| h (the largest t_ij the window can hold) is at most
//    pivot_over_max<K>(), which keeps a block of 8 factors below 2^128. A window
//    that some particle fails (components far apart across a wide window, a
//    datum or parameter not finite) goes through the plain forms below. On
//    data in ascending order the windows are narrow and nearly all are
//    taken; on unordered data nearly none are;
//  - direct (weights of total mass <= 1): e_j = sum_i 2^{a_ij}. Every factor
//    is then <= 1, so the partial products only fall, and a block of 8 whose
//    product ends at or above 2^-100 had no factor or partial product in the
//    FP32 subnormal range: it is as accurate as the shifted form;
//  - shifted: each datum's sum is taken relative to its largest term
//    m_j = max_i a_ij (blocks of 16), and the m_j are added apart.
// The plain forms: a wave starts in the direct form when every lane's `near`
// hint holds (the caller's guess that the particle sits near the data, from
// its current log-likelihood) and, at the first block where any of its lanes
// ends below 2^-100 (a particle far from these data, or a NaN), drops that
// block and takes the shifted form for the rest of its slice; otherwise it
// takes the shifted form throughout. All forms are within the FP32 error
// bound; which one a particle's data went through depends on the wave it
// shares (fixed for a given launch shape, population and data order). j0 and
// j1 must be the same in every lane of the wave, and every lane of the wave
// must take part (the forms use cross-lane operations, scalar loads and the
// wave's LDS row). With form_ctr set (kFormCounts arrays of kFormSlots
// counters), a wave adds to slot `slot` of each array (one atomic per nonzero
// count, slots spread so that waves rarely share one): [0] the number of data
// it took in the plain shifted form, counted up to the last full block of 8
// of each range the plain forms took (a whole slice, or a refused window; the
// fewer than 8 data after such a range's last full block always take the
// shifted form and are not counted); [1] the number of data it took in the
// pivot form; [2] the sum over those data of the number of other components
// the pivot form evaluated for them.
constexpr int kFormSlots = 1024;
constexpr int kFormCounts = 3;
// Data per window of the pivot form (one per lane), and the floats of a wave's
// staging row (two windows).
constexpr int kPivotWin = kWave;
constexpr int kPivotRow = 2 * kPivotWin;
// Shortest slice that takes the pivot form. Short slices come from short data
// (the paper's runs have 100 observations), whose windows of 64 span most of
// the data's range: the pivot form refuses nearly all of them, and trying cost
// 5-8% there.
constexpr int kPivotMinData = 128;
// Largest t_ij a window of the pivot form may hold with K components: a
// factor is then below 1 + (K-1) 2^T, and a block of 8 factors times a
// mantissa below 1 stays below the FP32 overflow at 2^128:
// (1 + 3 * 2^14)^8 < 2^125 for K <= 4, (1 + 7 * 2^13)^8 < 2^127 for K <= 8.
template <int K>
constexpr float pivot_over_max() {
    static_assert(K <= 8, "pivot_over_max assumes at most 8 components");
    return K <= 4 ? 14.0f : 13.0f;
}
static_assert(SMC_KMAX <= 8, "pivot_over_max assumes at most 8 components");
// A component other than the pivot whose t_ij stays below this in a window
// for every particle of the wave is left out there: its term is below 2^-25,
// under half the relative resolution of the product update p (1 + e) it would
// join (at most 7 such terms, so a datum's log2 factor is short by less than
// 3.1e-7, of the order of that update's own rounding).
constexpr float kPivotSkip = -25.0f;

// Calls f(std::integral_constant<int, m>) for a wave-uniform m in [0, M].
template <int M, class F>
__device__ __forceinline__ void with_count(int m, F&& f) {
    if constexpr (M == 0) {
        f(std::integral_constant<int, 0>{});
    } else {
        if (m == M) f(std::integral_constant<int, M>{});
        else with_count<M - 1>(m, f);
    }
}

// A wave's staging for the pivot form: its LDS row of kPivotRow floats
// (nullptr: plain forms only) and, when `pre` is set, each lane's datum
// y[j0 + lane] of its slice already loaded where j0 + lane < j1 (a caller may
// issue that load early, ahead of other work).
struct PivotStage {
    float* row = nullptr;
    float y0 = 0.0f;
    bool pre = false;
};

// The data slice [j0, j1) of slice sl out of nsl over n data (the same in
// every lane). Slices of at least 64 data start on multiples of 8, the FP32
// forms' blocks, so that only a slice ending at n can end in a partial block.
__device__ __forceinline__ void slice_bounds(int n, int sl, int nsl, int& j0, int& j1) {
    const int a = static_cast<int>((static_cast<int64_t>(n) * sl) / nsl);
    const int b = static_cast<int>((static_cast<int64_t>(n) * (sl + 1)) / nsl);
    const bool blocks = static_cast<int64_t>(n) >= static_cast<int64_t>(64) * nsl;
    j0 = wave_uniform(blocks ? a & ~7 : a);
    j1 = wave_uniform(blocks && sl + 1 < nsl ? b & ~7 : b);
}

// Data counts of one wave's slice by form (the form counters of partial_fp32).
struct FormCount {
    int shifted = 0;           // in the plain shifted form (up to full blocks of 8)
    int pivot = 0;             // in the pivot form
    int terms = 0;             // other components evaluated, summed over pivot data
};

// The pivot form over the 1-D slice [j0, j1) (see partial_fp32): adds the
// slice's terms to prod, expo and msum and its data counts to fc. nms[i] =
// -s mu_i in FP32; plain(ja, jb) runs the plain forms over [ja, jb) and
// returns the count of data they took in the shifted form.
template <int K, class Plain>
__device__ __forceinline__ void pivot_slice(const float* __restrict__ y, int j0, int j1,
                                            const double (&mu)[K], const GmmDev& g,
                                            const float (&nms)[K], const PivotStage& st,
                                            float& prod, int& expo, double& msum, FormCount& fc,
                                            Plain&& plain) {
    constexpr double kLog2eD = 1.4426950408889634;
    constexpr int KO = K > 1 ? K - 1 : 1;
    const int lane = lane_id();
    const float s = g.s32;
    const double s2 = g.inv2s2 * kLog2eD;
    float* row = st.row;
    float beta[K];
#pragma unroll
    for (int i = 0; i < K; ++i) beta[i] = static_cast<float>(2.0 * s2 * mu[i]);
    // each lane's datum of the current window and of the next one, loaded a
    // window ahead of their use
    float ycur = st.pre ? st.y0 : (j0 + lane < j1 ? y[j0 + lane] : 0.0f);
    float ynext = j0 + kPivotWin + lane < j1 ? y[j0 + kPivotWin + lane] : 0.0f;
    // the pivot of each lane for a window with midpoint c and half-width h:
    // the others' offsets dX, slopes dB and largest offsets ub, and the pivot's
    // mean and log-weight; ok when no lane's ub passes pivot_over_max<K>() (and h is
    // finite)
    float dX[KO], dB[KO], ub[KO];
    double mp = 0.0, lwp = 0.0;
    auto choose = [&](float c, float h) {
        float a[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const float t = __builtin_fmaf(c, s, nms[i]);
            a[i] = __builtin_fmaf(-t, t, g.lw2[i]);
        }
        int piv = 0;
        float best = a[0];
#pragma unroll
        for (int i = 1; i < K; ++i) {
            const bool up = a[i] > best;
            best = up ? a[i] : best;
            piv = up ? i : piv;
        }
        float bp = beta[0];
        mp = mu[0];
        lwp = g.lw[0];
#pragma unroll
        for (int i = 1; i < K; ++i) {
            const bool at = piv == i;
            bp = at ? beta[i] : bp;
            mp = at ? mu[i] : mp;
            lwp = at ? g.lw[i] : lwp;
        }
        bool ok = h <= 3.0e38f;               // false for a datum not finite
#pragma unroll
        for (int o = 0; o + 1 < K; ++o) {
            const bool up = o >= piv;
            dX[o] = (up ? a[o + 1] : a[o]) - best;
            dB[o] = (up ? beta[o + 1] : beta[o]) - bp;
            ub[o] = __builtin_fmaf(fabsf(dB[o]), h, dX[o]);
            ok &= ub[o] <= pivot_over_max<K>();
        }
        return __all(ok);
    };
    // while it works, two windows at a time share one choice of pivots
    bool pairs = true;
    for (int wb = j0; wb < j1;) {
        const int left = j1 - wb;
        const int nw0 = wave_uniform(left < kPivotWin ? left : kPivotWin);
        const int nw1 = wave_uniform(left > kPivotWin ? (left - kPivotWin < kPivotWin
                                                             ? left - kPivotWin : kPivotWin) : 0);
        const float v0 = ycur, v1 = ynext;
        const bool in0 = lane < nw0, in1 = lane < nw1;
        int nw = 0;
        float c = 0.0f, S1 = 0.0f, S2 = 0.0f;
        if (pairs && nw1 > 0) {
            // the pair's range and its data sums about its midpoint (all lanes)
            const int k0 = float_order_key(v0);
            const int k1 = in1 ? float_order_key(v1) : INT_MAX;
            const int k1x = in1 ? float_order_key(v1) : INT_MIN;
            const float lo = float_of_order_key(wave_extreme_key<false>(k0 < k1 ? k0 : k1));
            const float hi = float_of_order_key(wave_extreme_key<true>(k0 > k1x ? k0 : k1x));
            c = 0.5f * lo + 0.5f * hi;
            const float h = 0.5f * hi - 0.5f * lo;
            if (choose(c, h)) {
                const float d0 = v0 - c;
                const float d1 = in1 ? v1 - c : 0.0f;
                S1 = wave_sum_dpp(d0 + d1);
                S2 = wave_sum_dpp(__builtin_fmaf(d1, d1, d0 * d0));
                wave_sync();                  // the previous window's reads come first
                row[lane] = d0;
                row[kPivotWin + lane] = d1;
                // the next two windows' data, in flight while these are consumed
                // (issued after these are used, so that no wait covers them)
                const int jn = wb + 2 * kPivotWin + lane;
                ycur = jn < j1 ? y[jn] : 0.0f;
                ynext = jn + kPivotWin < j1 ? y[jn + kPivotWin] : 0.0f;
                wave_sync();                  // the windows are written before they are read
                nw = nw0 + nw1;
            } else {
                pairs = false;
            }
        }
        if (nw == 0) {
            // one window: its range and data sums about its midpoint
            const float lo = wave_min_dpp(in0 ? v0 : INFINITY);
            const float hi = wave_max_dpp(in0 ? v0 : -INFINITY);
            c = 0.5f * lo + 0.5f * hi;
            const float h = 0.5f * hi - 0.5f * lo;
            const bool take = choose(c, h);
            const float d0 = in0 ? v0 - c : 0.0f;
            if (take) {
                S1 = wave_sum_dpp(d0);
                S2 = wave_sum_dpp(d0 * d0);
                wave_sync();
                row[lane] = d0;
            }
            // the window after next, in flight
            const int jn = wb + 2 * kPivotWin + lane;
            ycur = v1;
            ynext = jn < j1 ? y[jn] : 0.0f;
            if (!take) {
                fc.shifted += plain(wb, wb + nw0);
                wb += nw0;
                continue;
            }
            wave_sync();
            nw = nw0;
        }
        fc.pivot += nw;
        if constexpr (K > 1) {
            // each lane's others in decreasing order of ub (odd-even
            // transposition network); the wave takes as many of them as its
            // neediest lane has with ub >= kPivotSkip
#pragma unroll
            for (int r = 0; r < KO; ++r) {
#pragma unroll
                for (int o = r & 1; o + 1 < KO; o += 2) {
                    const bool sw = ub[o + 1] > ub[o];
                    const float u0 = ub[o], x0 = dX[o], b0 = dB[o];
                    ub[o] = sw ? ub[o + 1] : u0;
                    dX[o] = sw ? dX[o + 1] : x0;
                    dB[o] = sw ? dB[o + 1] : b0;
                    ub[o + 1] = sw ? u0 : ub[o + 1];
                    dX[o + 1] = sw ? x0 : dX[o + 1];
                    dB[o + 1] = sw ? b0 : dB[o + 1];
                }
            }
            int need = 0;
#pragma unroll
            for (int o = 0; o < KO; ++o) need += ub[o] >= kPivotSkip ? 1 : 0;
            int m = 0;
#pragma unroll
            for (int q = 1; q < K; ++q) m = __any(need >= q) ? q : m;
            m = wave_uniform(m);
            fc.terms += m * nw;
            with_count<KO>(m, [&](auto mc) {
                constexpr int M = decltype(mc)::value;
                if constexpr (M > 0) {
                    auto factor = [&](float p, float d) {
                        float e = __builtin_amdgcn_exp2f(__builtin_fmaf(d, dB[0], dX[0]));
#pragma unroll
                        for (int o = 1; o < M; ++o)
                            e += __builtin_amdgcn_exp2f(__builtin_fmaf(d, dB[o], dX[o]));
                        return __builtin_fmaf(p, e, p);
                    };
                    int u = 0;
                    for (; u + 8 <= nw; u += 8) {
                        float p = prod;
#pragma unroll
                        for (int q = 0; q < 8; q += 4) {
                            const float4 d4 = *reinterpret_cast<const float4*>(row + u + q);
                            p = factor(p, d4.x);
                            p = factor(p, d4.y);
                            p = factor(p, d4.z);
                            p = factor(p, d4.w);
                        }
                        expo += __builtin_amdgcn_frexp_expf(p);
                        prod = __builtin_amdgcn_frexp_mantf(p);
                    }
                    if (u < nw) {
                        float p = prod;
                        for (; u < nw; ++u) p = factor(p, row[u]);
                        expo += __builtin_amdgcn_frexp_expf(p);
                        prod = __builtin_amdgcn_frexp_mantf(p);
                    }
                }
            });
        }
        // the pivots' own terms over the window(s), in FP64
        const double d = static_cast<double>(c) - mp;
        const double sq = static_cast<double>(S2) +
                          d * (2.0 * static_cast<double>(S1) + static_cast<double>(nw) * d);
        msum += static_cast<double>(nw) * lwp * kLog2eD - s2 * sq;
        wb += nw;
    }
}

template <int K, int D>
__device__ __forceinline__ double partial_fp32(const float* __restrict__ y, int j0, int j1,
                                               const double (&mu)[K * D], const GmmDev& g,
                                               bool near, const PivotStage& st,
                                               unsigned long long* form_ctr = nullptr) {
    constexpr int UF = 8;            // direct-form block
    constexpr int US = 16;           // shifted-form block
    constexpr float kFloor = 0x1p-100f;
    const float s = g.s32;
    double msum = 0.0;
    float prod = 1.0f;
    int expo = 0;
    float nms[K * D];                // -s mu in FP32
#pragma unroll
    for (int c = 0; c < K * D; ++c) nms[c] = static_cast<float>(-(static_cast<double>(s) * mu[c]));
    auto exponents = [&](const float* yj, float (&a)[K]) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if constexpr (D == 1) {
                const float t = __builtin_fmaf(yj[0], s, nms[i]);
                a[i] = __builtin_fmaf(-t, t, g.lw2[i]);
            } else {
                float q = 0.0f;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const float t = __builtin_fmaf(yj[c], s, nms[i * D + c]);
                    q = __builtin_fmaf(t, t, q);
                }
                a[i] = g.lw2[i] - q;
            }
        }
    };
    auto shifted = [&](const float* yj, float& m_out, float& e_out) {
        float a[K];
        exponents(yj, a);
        float m = a[0];
#pragma unroll
        for (int i = 1; i < K; ++i) m = fmaxf(m, a[i]);
        float e = __builtin_amdgcn_exp2f(a[0] - m);
#pragma unroll
        for (int i = 1; i < K; ++i) e += __builtin_amdgcn_exp2f(a[i] - m);
        m_out = m;
        e_out = e;
    };
    auto direct = [&](const float* yj) {
        float a[K];
        exponents(yj, a);
        float e = __builtin_amdgcn_exp2f(a[0]);
#pragma unroll
        for (int i = 1; i < K; ++i) e += __builtin_amdgcn_exp2f(a[i]);
        return e;
    };
    // the plain forms over [ja, jb); the direct form, once left, is not taken
    // again in this slice. Returns the data taken in the shifted form up to
    // the range's last full block of 8.
    bool take_direct = g.unit_mass != 0 && __all(near);
    auto plain = [&](int ja, int jb) {
        int j = ja;
        if (take_direct) {
            for (; j + UF <= jb; j += UF) {
                const float* yb = y + (size_t)wave_uniform(j) * D;    // wave-uniform: scalar loads
                float p = prod;
#pragma unroll
                for (int u = 0; u < UF; ++u) p *= direct(yb + u * D);
                if (!__all(p >= kFloor)) {
                    take_direct = false;
                    break;
                }
                expo += __builtin_amdgcn_frexp_expf(p);
                prod = __builtin_amdgcn_frexp_mantf(p);
            }
        }
        const int counted = ((jb - ja) & ~(UF - 1)) - (j - ja);
        for (; j + US <= jb; j += US) {
            float mblk = 0.0f;
#pragma unroll 8
            for (int u = 0; u < US; ++u) {
                float m, e;
                shifted(y + (size_t)(j + u) * D, m, e);
                prod *= e;
                mblk += m;
            }
            msum += static_cast<double>(mblk);
            expo += __builtin_amdgcn_frexp_expf(prod);
            prod = __builtin_amdgcn_frexp_mantf(prod);
        }
#pragma unroll 4
        for (; j < jb; ++j) {
            float m, e;
            shifted(y + (size_t)j * D, m, e);
            prod *= e;
            msum += static_cast<double>(m);
        }
        return counted;
    };
    FormCount fc;
    if constexpr (D == 1) {
        if (st.row != nullptr && j1 - j0 >= kPivotMinData)
            pivot_slice<K>(y, j0, j1, mu, g, nms, st, prod, expo, msum, fc, plain);
        else
            fc.shifted = plain(j0, j1);
    } else {
        fc.shifted = plain(j0, j1);
    }
    if (form_ctr != nullptr && lane_id() == 0) {
        const int slot = (static_cast<int>(blockIdx.x) * (static_cast<int>(blockDim.x) >> 6) +
                          wave_id()) & (kFormSlots - 1);
        const int cnt[kFormCounts] = {fc.shifted, fc.pivot, fc.terms};
#pragma unroll
        for (int c = 0; c < kFormCounts; ++c)
            if (cnt[c] > 0)
                atomicAdd(form_ctr + c * kFormSlots + slot, static_cast<unsigned long long>(cnt[c]));
    }
    // the product's mantissa in [0.5, 1): its hardware log2 is within 2^-23 of
    // the exact value, far below the bound per slice
    expo += __builtin_amdgcn_frexp_expf(prod);
    prod = __builtin_amdgcn_frexp_mantf(prod);
    return msum + static_cast<double>(expo) + static_cast<double>(__builtin_amdgcn_logf(prod));
}

// Sum over data j in [ja, jb), at most kGeneralMax64 of them, of
// ln sum_i w_i exp(-||y_j - mu_i||^2 / (2 sigma2)) in FP64, the general form: each
// datum's sum is taken relative to its largest term (the maxima added in FP64) and
// lies in [1, K], so the sums are multiplied into a product (below 2^192) that one
// log finishes. Exponents and maxima are in natural units, so that neither log w_i
// nor 1 / (2 sigma2) is rounded again by a factor log2(e); only the differences to
// the maximum take it, on their way into 2^t. NaN for a datum that is not finite,
// for a mean that is NaN and where every mean is infinite; an infinite mean beside
// finite ones contributes a zero term. Two data at a time: FP64 issue bounds it, at
// 23 instructions per datum and component, once the chains overlap.
constexpr int kGeneralMax64 = 64;
template <int K>
__device__ __forceinline__ double general_fp64(const float* __restrict__ y, int ja, int jb,
                                               const double (&mu)[K], const GmmDev& g) {
    double msum = 0.0, prod = 1.0;
    auto datum = [&](int j, double& m, double& e) {
        double a[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const double t = static_cast<double>(y[j]) - mu[i];
            a[i] = fma(-(t * t), g.inv2s2, g.lw[i]);
        }
        m = a[0];
#pragma unroll
        for (int i = 1; i < K; ++i) m = fmax(m, a[i]);
        e = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i) e += exp2_fp64(fmax((a[i] - m) * kLog2e, -4000.0));
    };
    int j = ja;
    for (; j + 2 <= jb; j += 2) {
        double m0, m1, e0, e1;
        datum(j, m0, e0);
        datum(j + 1, m1, e1);
        msum = (msum + m0) + m1;
        prod = (prod * e0) * e1;
    }
    if (j < jb) {
        double m, e;
        datum(j, m, e);
        msum += m;
        prod *= e;
    }
    // the clamp passed over a NaN: a mean's, or that of no finite exponent at all
    bool finite = msum > -INFINITY;
#pragma unroll
    for (int i = 0; i < K; ++i) finite = finite && mu[i] == mu[i];
    return finite ? msum + kLn2 * log2(prod) : static_cast<double>(NAN);
}

// Data per window of the FP64 pivot form (one per lane): a wave's staging row
// holds one window of FP64 offsets (the room of two FP32 windows).
constexpr int kPivotWin64 = kWave;
static_assert(kPivotWin64 * sizeof(double) == kPivotRow * sizeof(float), "");
static_assert(kPivotWin64 <= kGeneralMax64, "");
// Shortest slice that takes the FP64 pivot form: choosing a window's pivots
// costs about as much as three data of the general form.
constexpr int kPivotMin64 = 8;
// A refused window of more data than this is halved if the halves are likely to hold,
// else it goes through the general form.
constexpr int kPivotLeast64 = 16;
// Largest exponent difference a window of the FP64 pivot form may hold. It bounds
// the error, not the range: a datum whose own component is 2^T above its window's
// pivot is the sum of a pivot exponent and a difference that cancel, each rounded
// at 2^-53 T, the pivot's alike for a whole window. At T = 12 the error against
// 64 bits is at most that of a term-by-term exp and log (rms over particles at
// k = 4, sigma2 = 0.55, near the modes: n = 1000 sorted 0.7e-16 against 1.6e-16,
// unsorted 0.8 against 1.7, n = 50 1.1 against 1.0); at T = 250 it is 14e-16
// unsorted and 2.6e-16 at n = 50.
constexpr double kPivotOver64 = 12.0;
// A component whose exponent difference to the pivot stays below this over a
// window is left out there: its term is below 2^-58 of a factor of at least 1,
// under a sixteenth of the resolution of the product update it would join.
constexpr double kPivotSkip64 = -58.0;

// The FP64 likelihood of the 1-D slice [j0, j1) in the pivot form (the algebra
// of the FP32 pivot form above partial_fp32, all of it in FP64): per window of
// 64 data each particle takes the component with the largest exponent at the
// window's midpoint as its pivot, whose own terms come in closed form from two
// sums over the window's data; every other component costs one FMA, one exp2
// and one add per datum, and the per-datum factors 1 + sum 2^t are multiplied
// into a product renormalised every 4 data, so no datum takes a log. Each
// particle orders its other components by the largest exponent difference the
// window can hold; the wave takes as many of them as its neediest particle
// needs, and a particle that does not need one of them adds zero for it.
// Bound by FP64 VALU issue: 16 instructions per datum and evaluated component
// plus about 270 per window. Windows of 64 data rather than 128: the narrower
// range needs fewer components, which saves more than the second choice of
// pivots costs. A window where some particle's bound fails (data that spread over
// several components, a datum or parameter not finite) is halved where that is
// likely to hold, and the next ones start from the length that held; else it goes
// through the general form. k = 4, n = 4096, N = 65536: 0.35 ms sorted, 0.70 ms
// unsorted (all general; 1.48 with an exp per term and a log per datum).
// Returns natural-log units.
template <int K>
__device__ __forceinline__ double pivot_fp64(const float* __restrict__ y, int j0, int j1,
                                             const double (&mu)[K], const GmmDev& g,
                                             const PivotStage& st) {
    constexpr int KO = K > 1 ? K - 1 : 1;
    constexpr int U = 4;
    const int lane = lane_id();
    const double s2 = g.inv2s2 * kLog2e;
    double* row = reinterpret_cast<double*>(st.row);
    double prod = 1.0, msum = 0.0, plain = 0.0;
    int expo = 0;
    float vnext = st.pre ? st.y0 : (j0 + lane < j1 ? y[j0 + lane] : 0.0f);
    int len = kPivotWin64;                           // of the next window
    // the lanes hold the 64 data from wb on; a window is nw of them from off on
    for (int wb = j0; wb < j1; wb += kPivotWin64) {
        const int held = wave_uniform(j1 - wb < kPivotWin64 ? j1 - wb : kPivotWin64);
        const float v = vnext;
        const int jn = wb + kPivotWin64 + lane;
        vnext = jn < j1 ? y[jn] : 0.0f;                  // in flight over these windows
        for (int off = 0; off < held;) {
            const int nw = wave_uniform(held - off < len ? held - off : len);
            const bool in = lane >= off && lane < off + nw;
            // the window's midpoint and half-width
            const float lo = wave_min_dpp(in ? v : INFINITY);
            const float hi = wave_max_dpp(in ? v : -INFINITY);
            const double c = static_cast<double>(0.5f * lo + 0.5f * hi);
            const double h = fmax(static_cast<double>(hi) - c, c - static_cast<double>(lo));
            // exponents at the midpoint and the pivot
            double a[K];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const double t = c - mu[i];
                a[i] = g.lw[i] - g.inv2s2 * (t * t);
            }
            int piv = 0;
            double best = a[0];
#pragma unroll
            for (int i = 1; i < K; ++i) {
                const bool up = a[i] > best;
                best = up ? a[i] : best;
                piv = up ? i : piv;
            }
            double mp = mu[0], lwp = g.lw[0];
#pragma unroll
            for (int i = 1; i < K; ++i) {
                mp = piv == i ? mu[i] : mp;
                lwp = piv == i ? g.lw[i] : lwp;
            }
            double dX[KO], dB[KO], ub[KO];
            bool ok = h <= 3.0e38 && fabs(best) <= 1.0e300;
#pragma unroll
            for (int o = 0; o + 1 < K; ++o) {
                const bool up = o >= piv;
                dX[o] = ((up ? a[o + 1] : a[o]) - best) * kLog2e;
                dB[o] = 2.0 * s2 * ((up ? mu[o + 1] : mu[o]) - mp);
                ub[o] = fma(fabs(dB[o]), h, dX[o]);
                // false for NaN; the lower bound keeps t within exp2_fp64's range
                ok &= ub[o] <= kPivotOver64 && (dX[o] >= -1.0e8 || ub[o] < kPivotSkip64);
            }
            if (!__all(ok)) {
                // half as long if the shortest such windows are likely to hold: there the
                // pivot is the best component nearby, and a difference to it at most |dB|
                // times their half-width
                const double hs = h * kPivotLeast64 / nw;
                bool half = true;
#pragma unroll
                for (int o = 0; o + 1 < K; ++o)
                    half = half && (ub[o] <= kPivotOver64 || fabs(dB[o]) * hs <= kPivotOver64);
                if (nw > kPivotLeast64 && __all(half)) {
                    len = (nw + 7) / 8 * 4;
                    continue;
                }
                plain += general_fp64<K>(y, wb + off, wb + off + nw, mu, g);
                off += nw;
                continue;
            }
            const double d = in ? static_cast<double>(v) - c : 0.0;
            const double S1 = wave_sum(d);
            const double S2 = wave_sum(d * d);
            if constexpr (K > 1) {
                wave_sync();                             // the previous window's reads come first
                row[lane] = d;
                // the others in decreasing order of ub (odd-even transposition
                // network); those a particle does not need become exact zeros
#pragma unroll
                for (int r = 0; r < KO; ++r) {
#pragma unroll
                    for (int o = r & 1; o + 1 < KO; o += 2) {
                        const bool sw = ub[o + 1] > ub[o];
                        const double u0 = ub[o], x0 = dX[o], b0 = dB[o];
                        ub[o] = sw ? ub[o + 1] : u0;
                        dX[o] = sw ? dX[o + 1] : x0;
                        dB[o] = sw ? dB[o + 1] : b0;
                        ub[o + 1] = sw ? u0 : ub[o + 1];
                        dX[o + 1] = sw ? x0 : dX[o + 1];
                        dB[o + 1] = sw ? b0 : dB[o + 1];
                    }
                }
                int m = 0;
#pragma unroll
                for (int o = 0; o < KO; ++o) {
                    const bool need = ub[o] >= kPivotSkip64;
                    dX[o] = need ? dX[o] : -4000.0;
                    dB[o] = need ? dB[o] : 0.0;
                    m = __any(need) ? o + 1 : m;
                }
                m = wave_uniform(m);
                wave_sync();                             // the window is written before it is read
                if (m > 0) {
                    int u = 0;
                    for (; u + U <= nw; u += U) {
                        double x[U], e[U];
#pragma unroll
                        for (int q = 0; q < U; ++q) x[q] = row[off + u + q];
#pragma unroll
                        for (int q = 0; q < U; ++q) e[q] = exp2_fp64(fma(x[q], dB[0], dX[0]));
#pragma unroll
                        for (int o = 1; o < KO; ++o) {
                            if (o >= m) break;
#pragma unroll
                            for (int q = 0; q < U; ++q) e[q] += exp2_fp64(fma(x[q], dB[o], dX[o]));
                        }
                        double p = prod;
#pragma unroll
                        for (int q = 0; q < U; ++q) p = fma(p, e[q], p);
                        expo += __builtin_amdgcn_frexp_exp(p);
                        prod = __builtin_amdgcn_frexp_mant(p);
                    }
                    for (; u < nw; ++u) {
                        const double x = row[off + u];
                        double e = exp2_fp64(fma(x, dB[0], dX[0]));
#pragma unroll
                        for (int o = 1; o < KO; ++o) {
                            if (o >= m) break;
                            e += exp2_fp64(fma(x, dB[o], dX[o]));
                        }
                        const double p = fma(prod, e, prod);
                        expo += __builtin_amdgcn_frexp_exp(p);
                        prod = __builtin_amdgcn_frexp_mant(p);
                    }
                }
            }
            // the pivots' own terms over the window
            const double dc = c - mp;
            const double nd = static_cast<double>(nw);
            msum += nd * lwp - g.inv2s2 * (S2 + dc * (2.0 * S1 + nd * dc));
            off += nw;
        }
        len = 2 * len < kPivotWin64 ? 2 * len : kPivotWin64;
    }
    return msum + kLn2 * (static_cast<double>(expo) + log2(prod)) + plain;
}

// Sum over data j in [j0, j1) of ln sum_i w_i exp(-||y_j - mu_i||^2 / (2 sigma2)), FP64.
// 1-D data take the pivot form where the wave has a staging row, else the
// general form; d > 1 takes the device library's exp per term and log per datum
// (its k*d means fill the register budget, and the product form measured slower).
template <int K, int D>
__device__ __forceinline__ double partial_fp64(const float* __restrict__ y, int j0, int j1,
                                               const double (&mu)[K * D], const GmmDev& g,
                                               const PivotStage& st) {
    if constexpr (D == 1) {
        if (st.row != nullptr && j1 - j0 >= kPivotMin64) return pivot_fp64<K>(y, j0, j1, mu, g, st);
        return general_fp64<K>(y, j0, j1, mu, g);
    }
    double acc = 0.0;
    for (int j = j0; j < j1; ++j) {
        const float* yj = y + (size_t)j * D;
        double a[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            double q = 0.0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const double t = static_cast<double>(yj[c]) - mu[i * D + c];
                q += t * t;
            }
            a[i] = g.lw[i] - q * g.inv2s2;
        }
        double m = a[0];
#pragma unroll
        for (int i = 1; i < K; ++i) m = fmax(m, a[i]);
        double e = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i) e += exp(a[i] - m);
        acc += m + log(e);
    }
    return acc;
}

// Whether a particle with log-likelihood l over n data sits near the data in
// the sense the FP32 direct form needs: its per-datum mixture sums average at
// least 2^-6 (blocks of 8 then stay far above 2^-100). False for NaN and -inf.
__device__ __forceinline__ bool near_data(double l, int n, const GmmDev& g) {
    return l >= static_cast<double>(n) * (g.cst - 6.0 * kLn2);
}

// The slice partial of one lane for parameters pr[0..K*D-1] (FP64 values);
// `near` is the hint of partial_fp32 (unused in FP64) and `st` the wave's staging
// for the pivot forms.
template <int K, int D, int PREC>
__device__ __forceinline__ double slice_partial(const float* __restrict__ y, int j0, int j1,
                                                const double (&pr)[K * D], const GmmDev& g,
                                                bool near = true, const PivotStage& st = {},
                                                unsigned long long* form_ctr = nullptr) {
    if constexpr (PREC == SMC_PREC_FP32) {
        return partial_fp32<K, D>(y, j0, j1, pr, g, near, st, form_ctr);
    } else {
        return partial_fp64<K, D>(y, j0, j1, pr, g, st);
    }
}

// The S slice partials of a lane's particle, added in slice order. Four rows are
// read before the first is added, so an addition does not wait on an LDS read of
// its own (a loop of single reads and adds took about 140 cycles a slice on the
// one wave that decides).
__device__ __forceinline__ double sum_slices(const double (*red)[kWave], int S) {
    const int lane = lane_id();
    double tot = 0.0;
    for (int q = 0; q < S; q += 4) {
        double v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = red[q + i < S ? q + i : S - 1][lane];
        tot = q == 0 ? v[0] : tot + v[0];
#pragma unroll
        for (int i = 1; i < 4; ++i)
            if (q + i < S) tot += v[i];
    }
    return tot;
}

// The G groups' partial sums of particle p, added in group order. All are
// requested at once (beyond G the last one again), before the caller draws its
// random numbers: one after another they took 0.6 us more a launch at G = 8.
struct GroupSums {
    double v[kMoveGroups];
    __device__ __forceinline__ GroupSums(const double* __restrict__ part, int N, int p, int G) {
#pragma unroll
        for (int q = 0; q < kMoveGroups; ++q)
            v[q] = part[static_cast<size_t>(q < G ? q : G - 1) * N + p];
    }
    __device__ __forceinline__ double total(int G) const {
        double tot = v[0];
#pragma unroll
        for (int q = 1; q < kMoveGroups; ++q)
            if (q < G) tot += v[q];
        return tot;
    }
};

// Particle p's draw from the prior, coordinate c at theta[c * N + p].
template <int KD>
__device__ __forceinline__ void prior_draw(int p, int N, uint64_t seed, const GmmDev& g,
                                           double* __restrict__ theta) {
    if (g.prior == SMC_PRIOR_GAUSS) {
        double z[KD];
        normals<KD>(seed, static_cast<uint32_t>(p), 0, kPrior, 0, z);
#pragma unroll
        for (int c = 0; c < KD; ++c) theta[static_cast<size_t>(c) * N + p] = g.pa + g.pb * z[c];
    } else {
        const double width = g.pb - g.pa;
#pragma unroll
        for (int b = 0; b < (KD + 3) / 4; ++b) {
            const Words4 w = draw(seed, static_cast<uint32_t>(p), b, 0, kPrior, 0);
            const uint32_t ws[4] = {w.w0, w.w1, w.w2, w.w3};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * b + q < KD)
                    theta[static_cast<size_t>(4 * b + q) * N + p] = g.pa + width * u01_open(ws[q]);
        }
    }
}

// This wave's staging row for the pivot form in a kernel of at most W waves
// per workgroup (a static LDS array of that kernel), or nullptr where the form
// does not apply (d > 1).
template <int PREC, int D, int W>
__device__ __forceinline__ float* pivot_row() {
    if constexpr (D == 1) {
        __shared__ __align__(16) float win[W][kPivotRow];
        return win[wave_id()];
    } else {
        return nullptr;
    }
}

// log u of the acceptance test of particle p, u from stream (p, 0, step, ACC, move).
__device__ __forceinline__ double rwmh_log_u(uint32_t p, uint32_t step, uint64_t seed, uint32_t move) {
    return log(u01_open(draw(seed, p, 0, step, kAcc, move).w0));
}

// Random-walk proposals th_src[:, a] + sd * z for the 64 particles of a
// workgroup. The ceil(KD/2) Box-Muller pairs of each particle are shared out
// over the block's nw waves (pair q: Philox block q/2, words 0-1 for even q and
// 2-3 for odd q, normals 2q and 2q+1) and exchanged through LDS, so no wave
// repeats another's draws. Cooperative: every thread of the block calls it (it
// contains one barrier); prs holds KD rows of 64 doubles. With hold set, the
// current state is kept in LDS for the decision as well: hold[c] (KD rows of 64
// doubles) gets th_src[c, a] and hold_l the current log-likelihood l_src[a]
// (read by the block's last wave), so the decision after the likelihood does
// not wait on global loads. With log_u set, log_u[lane] gets the log u of the
// move's acceptance test, one more item beside the pairs: the decision then
// starts from it instead of drawing it on one wave while the others are done.
template <int KD>
__device__ __forceinline__ void block_proposals(uint64_t seed, uint32_t index, uint32_t step,
                                                uint32_t move, const double* th_src, int N,
                                                int a, double sd, int w, int nw,
                                                double (*prs)[kWave], double (&pr)[KD],
                                                double (*hold)[kWave] = nullptr,
                                                const double* l_src = nullptr,
                                                double* hold_l = nullptr,
                                                double* log_u = nullptr) {
    constexpr int NP = (KD + 1) / 2;
    const int lane = lane_id();
    if (hold != nullptr && w == nw - 1) hold_l[lane] = l_src[a];
    for (int q = w; q < NP + (log_u != nullptr ? 1 : 0); q += nw) {
        if (q == NP) {
            log_u[lane] = rwmh_log_u(index, step, seed, move);
            break;
        }
        const int c = 2 * q;
        const double t0 = th_src[static_cast<size_t>(c) * N + a];
        const double t1 = c + 1 < KD ? th_src[static_cast<size_t>(c + 1) * N + a] : 0.0;
        const Words4 wd = draw(seed, index, static_cast<uint32_t>(q / 2), step, kProp, move);
        double z0, z1;
        if (q & 1) box_muller(wd.w2, wd.w3, z0, z1);
        else box_muller(wd.w0, wd.w1, z0, z1);
        prs[c][lane] = t0 + sd * z0;
        if (c + 1 < KD) prs[c + 1][lane] = t1 + sd * z1;
        if (hold != nullptr) {
            hold[c][lane] = t0;
            if (c + 1 < KD) hold[c + 1][lane] = t1;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < KD; ++c) pr[c] = prs[c][lane];
}

// Source of a move's current state for the arrays (theta, l) it writes.
struct MoveSource {
    const double* th;
    const double* l;
    bool write_always;         // out of place: rejected particles are copied too
};

__device__ __forceinline__ MoveSource move_source(const MoveStep& ms, double* theta, double* l) {
    const bool rs = (ms.state != nullptr) && (ms.state->resampled != 0);
    if (rs && ms.theta_alt != nullptr) return MoveSource{ms.theta_alt, ms.l_alt, true};
    const double* th = ms.theta_src ? ms.theta_src : theta;
    const double* ll = ms.l_src ? ms.l_src : l;
    return MoveSource{th, ll, th != theta};
}

// LDS doubles of fused_ancestors: chunk offsets (two halves) and ends, then the
// search's window row.
__host__ __device__ constexpr int ancestor_lds_doubles(int nchunks) {
    return nchunks > 0 ? 3 * nchunks + kCdfWin : 0;
}

// LDS bytes of the pivot forms' staging rows of `slices` waves (d = 1).
constexpr size_t rows_lds_bytes(int slices, bool rows) {
    return rows ? sizeof(float) * kPivotRow * slices : 0;
}

constexpr size_t larger(size_t a, size_t b) { return a > b ? a : b; }

// Dynamic LDS bytes of one k_rwmh workgroup (the layout at the top of k_rwmh): the
// ancestor search's buffer, which grows with N, lies over what the move uses after
// it. Beside it, a CU held 16 one-slice waves where it holds 20 at N = 262144 and 4
// for 6 from 2^21 on (k = 4, n = 1000, N = 2^20: 7054 us per ten steps, 5374 now).
constexpr size_t rwmh_dyn_lds_bytes(int slices, int nchunks, bool rows, int kd) {
    return larger(sizeof(double) * kWave * (kd + (kd <= 16 ? kd : 0) + 2 + slices) +
                      rows_lds_bytes(slices, rows),
                  sizeof(double) * ancestor_lds_doubles(nchunks));
}

// Dynamic LDS bytes of one k_rwmh_multi workgroup (the layout at its top).
constexpr size_t multi_dyn_lds_bytes(int slices, int nchunks, bool rows, int kd, int batch) {
    return larger(sizeof(double) * kWave * (kd + 1 + batch * (kd + 1) + slices) +
                      rows_lds_bytes(slices, rows),
                  sizeof(double) * ancestor_lds_doubles(nchunks));
}

// Moves whose random numbers a k_rwmh_multi workgroup holds at once: two with
// drawing waves, else as many as leave LDS for the 16 waves a CU that its registers
// admit, at most 13 KB of them (k*d = 4: five moves, two with one slice). Ten moves
// a step, k = 4, n = 100, N = 262144: 6945 us per 20 steps at five moves, 5356 at
// two.
constexpr int kMultiWavesPerCu = 16;
constexpr size_t kCuLds = 156 * 1024;
constexpr int multi_batch(int kd, int slices, bool rows, int n_moves, bool drawers) {
    if (drawers) return 2;
    const size_t fixed = multi_dyn_lds_bytes(slices, 0, rows, kd, 0);
    const size_t one = sizeof(double) * kWave * (kd + 1);
    int fit = 1;
    while (fit < n_moves && (fit + 1) * one <= size_t{13 * 1024} &&
           fixed + (fit + 1) * one <= kCuLds * slices / kMultiWavesPerCu)
        ++fit;
    return fit;
}

// Ancestors of the 64 particles of this workgroup after resampling
// (cooperative: every thread of the block must call it). Wave 0 forms the chunk
// offsets and ends in LDS (exclusive double-double scan of the chunk totals; buf
// holds ancestor_lds_doubles(ms.nchunks)), then each of its lanes takes the
// scheme's point U_i for particle i and finds idx = min{j : U < C_j} (or the
// first j with C_j = C_{N-1}), C_j = offset + within-chunk prefix rounded once.
__device__ __forceinline__ void fused_ancestors(const MoveStep& ms, int N, uint32_t step, int pc,
                                                int* anc, double* buf) {
    const int lane = lane_id();
    double* offh = buf;
    double* offl = offh + ms.nchunks;
    double* cend = offl + ms.nchunks;
    double* win = cend + ms.nchunks;
    if (wave_id() == 0) {
        // two passes over the lane's chunk totals (sum, then running offsets)
        // keep the register footprint of this prologue small
        const int per = wave_uniform((ms.nchunks + kWave - 1) / kWave);
        dd run = dd_zero();
        for (int q = 0; q < per; ++q) {
            const int c = lane * per + q;
            if (c < ms.nchunks) run = dd_add(run, dd{ms.chunk_tot[2 * c], ms.chunk_tot[2 * c + 1]});
        }
        const dd inc = wave_scan(run);
        dd excl{__shfl_up(inc.hi, 1, kWave), __shfl_up(inc.lo, 1, kWave)};
        if (lane == 0) excl = dd_zero();
        for (int q = 0; q < per; ++q) {
            const int c = lane * per + q;
            if (c < ms.nchunks) {
                offh[c] = excl.hi;
                offl[c] = excl.lo;
                excl = dd_add(excl, dd{ms.chunk_tot[2 * c], ms.chunk_tot[2 * c + 1]});
                cend[c] = excl.hi;
            }
        }
        wave_sync();
        const double u = ms.scheme == 0 ? u01_left_closed(draw(ms.seed, 0, 0, step, kResamp, 0).w0)
                                        : 0.0;
        // pc is clamped to N - 1 past the end, so the tile's points are sorted
        // for the systematic and stratified schemes
        const double U = resample_point(ms.scheme, ms.seed, step, pc, N, u);
        const CdfView cdf{N, ms.chunk, ms.nchunks, ms.cdf_hi, ms.cdf_lo, offh, offl, cend};
        anc[lane] = ms.scheme == SMC_RESAMPLE_MULTINOMIAL
                        ? cdf_search(U, cdf)
                        : cdf_search_sorted_wave(U, true, cdf, win);
    }
    __syncthreads();
}

// Metropolis-Hastings log acceptance ratio for particle p of a random-walk
// move: log alpha = beta (l' - l) + log p0(theta') - log p0(theta).
// cur_at(c) / pr_at(c) return coordinate c of the current state / proposal;
// the prior's squares are summed in index order.
template <int KD, class PropAt, class CurAt>
__device__ __forceinline__ double rwmh_log_alpha(int p, PropAt pr_at, CurAt cur_at, double l_cur,
                                                 double l_prop, const double* beta_vec,
                                                 const StepSrc& src, uint32_t step,
                                                 const GmmDev& g) {
    // log p0(theta') - log p0(theta): the normalising constants cancel
    double lp;
    if (g.prior == SMC_PRIOR_GAUSS) {
        double sq_cur = 0.0, sq_prop = 0.0;
#pragma unroll
        for (int c = 0; c < KD; ++c) {
            // theta - pa, scaled (exactly) so that no square leaves the FP64 range
            // where the ratio does not
            const double zc = __builtin_amdgcn_ldexp(cur_at(c) - g.pa, g.pexp);
            const double zp = __builtin_amdgcn_ldexp(pr_at(c) - g.pa, g.pexp);
            sq_cur = fma(zc, zc, sq_cur);
            sq_prop = fma(zp, zp, sq_prop);
        }
        lp = (sq_cur - sq_prop) * g.inv2pb2;
    } else {
        bool in_cur = true, in_prop = true;
#pragma unroll
        for (int c = 0; c < KD; ++c) {
            const double xc = cur_at(c);
            const double xp = pr_at(c);
            in_cur = in_cur && (xc >= g.pa) && (xc <= g.pb);
            in_prop = in_prop && (xp >= g.pa) && (xp <= g.pb);
        }
        lp = (in_prop ? 0.0 : -INFINITY) - (in_cur ? 0.0 : -INFINITY);
    }
    const double beta = beta_vec ? beta_vec[p]
                                 : (src.beta_dev ? src.beta_dev[step] : src.beta_host);
    return beta * (l_prop - l_cur) + lp;
}

// Metropolis-Hastings decision: accept iff log alpha >= 0 or log u < log alpha
// (log u drawn here, or already drawn at *log_u).
template <int KD, class PropAt, class CurAt>
__device__ __forceinline__ bool rwmh_decide(int p, PropAt pr_at, CurAt cur_at, double l_cur,
                                            double l_prop, const double* beta_vec,
                                            const StepSrc& src, uint32_t step, uint64_t seed,
                                            uint32_t move, const GmmDev& g,
                                            const double* log_u = nullptr) {
    const double la = rwmh_log_alpha<KD>(p, pr_at, cur_at, l_cur, l_prop, beta_vec, src, step, g);
    if (log_u != nullptr) return (la >= 0.0) || (*log_u < la);
    return (la >= 0.0) || (rwmh_log_u(static_cast<uint32_t>(p), step, seed, move) < la);
}

// The step duties of a move's first launch: publish W (1/N after resampling)
// and reset logw after resampling (in place, or into logw_out).
__device__ __forceinline__ void move_duties(int p, int N, const MoveStep& ms) {
    const bool rs = (ms.state != nullptr) && (ms.state->resampled != 0);
    if (ms.W_out) {
        ms.W_out[p] = rs ? 1.0 / static_cast<double>(N)
                         : exp_fp64(ms.logw[p] - ms.state->M) / ms.state->S;
    }
    if (ms.logw_out) ms.logw_out[p] = rs ? 0.0 : ms.logw[p];
    else if (rs && ms.reset_logw) ms.logw[p] = 0.0;
}

// Decision and write-back of particle p of a random-walk move, its current
// state given by cur_at(c) and l_cur; pr_at(c) returns coordinate c of the
// proposal. Rejected particles are copied when the move is out of place
// (write_always). l_new (optional) receives the particle's log-likelihood after
// the move.
template <int KD, class PropAt, class CurAt>
__device__ __forceinline__ bool rwmh_accept_state(int p, int N, PropAt pr_at, CurAt cur_at,
                                                  double l_cur, double l_prop, bool write_always,
                                                  double* theta, double* l,
                                                  const double* beta_vec, const StepSrc& src,
                                                  uint32_t step, uint64_t seed, uint32_t move,
                                                  const GmmDev& g, int* status,
                                                  const MoveStep& ms, double* l_new = nullptr,
                                                  const double* log_u = nullptr) {
    const bool acc = rwmh_decide<KD>(p, pr_at, cur_at, l_cur, l_prop, beta_vec, src, step, seed,
                                     move, g, log_u);
    if (acc) {
#pragma unroll
        for (int c = 0; c < KD; ++c) theta[static_cast<size_t>(c) * N + p] = pr_at(c);
        l[p] = l_prop;
    } else if (write_always) {
#pragma unroll
        for (int c = 0; c < KD; ++c) theta[static_cast<size_t>(c) * N + p] = cur_at(c);
        l[p] = l_cur;
    }
    if (l_prop != l_prop) atomicOr(status, kStatusNaN);
    move_duties(p, N, ms);
    if (l_new) *l_new = acc ? l_prop : l_cur;
    return acc;
}

// rwmh_accept_state with the current state read from column a of (th_src,
// l_src) (a = p, or p's ancestor after a fused resampling).
template <int KD, class PropAt>
__device__ __forceinline__ bool rwmh_accept(int p, int a, int N, PropAt pr_at, double l_prop,
                                            const MoveSource& srcs, double* theta, double* l,
                                            const double* beta_vec, const StepSrc& src,
                                            uint32_t step, uint64_t seed, uint32_t move,
                                            const GmmDev& g, int* status, const MoveStep& ms,
                                            double* l_new = nullptr,
                                            const double* log_u = nullptr) {
    const double* th_src = srcs.th;
    return rwmh_accept_state<KD>(
        p, N, pr_at, [&](int c) { return th_src[static_cast<size_t>(c) * N + a]; }, srcs.l[a],
        l_prop, srcs.write_always, theta, l, beta_vec, src, step, seed, move, g, status, ms,
        l_new, log_u);
}

}  // namespace smc
