// Search of the correctly rounded CDF kept as within-chunk prefixes
// (cdf_hi/cdf_lo, each rounded once from a double-double scan of its chunk)
// plus per-chunk double-double totals: the pieces of systematic, stratified and
// multinomial resampling shared by the tempering steps, the batched runs and
// the particle filter's fused propagation.
#pragma once
#include "internal.hpp"
#include "dd.hpp"
#include "philox.hpp"
#include "reduce.hpp"

namespace smc {

// A CDF kept as within-chunk prefixes: C_j = offset of j's chunk + prefix j,
// rounded once. The chunk offsets and ends are in LDS; a chunk's end is C at its
// last element, formed by the same operation (its total is the prefix stored
// there), so a search may pick the chunk from the ends alone.
struct CdfView {
    int N, chunk, nchunks;
    const double* hi;          // [N] prefixes, high and low parts (global)
    const double* lo;
    const double* offh;        // [nchunks] offsets (LDS)
    const double* offl;
    const double* cend;        // [nchunks] ends (LDS)
    __device__ __forceinline__ double at(int c, int j) const {
        return dd_add(dd{offh[c], offl[c]}, dd{hi[j], lo[j]}).hi;
    }
    __device__ __forceinline__ double last() const { return cend[nchunks - 1]; }
};

// Chunk offsets and ends into LDS offh, offl, cend [nchunks]: the exclusive
// double-double scan of the chunk totals [2 * nchunks] (hi, lo), formed by every
// thread of a kRedBlock-thread block (cooperative; ends with a barrier).
__device__ __forceinline__ void block_cdf_offsets(const double* chunk_tot, int nchunks,
                                                  double* offh, double* offl, double* cend) {
    constexpr int per = kMaxChunks / kRedBlock;
    const int c0 = threadIdx.x * per;
    dd tot[per], loc[per];
    dd run = dd_zero();
#pragma unroll
    for (int q = 0; q < per; ++q)
        tot[q] = c0 + q < nchunks ? dd{chunk_tot[2 * (c0 + q)], chunk_tot[2 * (c0 + q) + 1]}
                                  : dd_zero();
#pragma unroll
    for (int q = 0; q < per; ++q) {
        loc[q] = run;
        if (c0 + q < nchunks) run = dd_add(run, tot[q]);
    }
    dd total;
    const dd lead = block_dd_exclusive_scan(run, total);
#pragma unroll
    for (int q = 0; q < per; ++q) {
        if (c0 + q >= nchunks) break;
        const dd o = dd_add(lead, loc[q]);
        offh[c0 + q] = o.hi;
        offl[c0 + q] = o.lo;
        cend[c0 + q] = dd_add(o, tot[q]).hi;
    }
    __syncthreads();
}

// Whether C_j = c lies at or past the ancestor of point U: the ancestor is
// min{j : U < C_j}, or the first j with C_j = C_{N-1} when U is not below that.
// Monotone in j and true at N - 1.
__device__ __forceinline__ bool cdf_past(double U, double c, double clast) {
    return U < clast ? (U < c) : (c >= clast);
}

// First position in [lo, hi] where f holds (f is monotone and true at hi).
template <class F>
__device__ __forceinline__ int first_true(int lo, int hi, F f) {
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (f(mid)) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// The same by the 32 lanes of a half-wave together, each half its own search
// (lo, hi and f differ between the halves only): every level probes 32 positions
// at once. Every lane of the wave calls it.
template <class F>
__device__ __forceinline__ int first_true_half(int lo, int hi, F f) {
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5, hl = lane & 31;
    while (__any(hi > lo)) {
        const int len = hi - lo + 1;
        const int step = (len + 31) >> 5;
        int q = lo + (hl + 1) * step - 1;
        q = q < hi ? q : hi;
        const unsigned long long m = __ballot(f(q));
        const unsigned mh = static_cast<unsigned>(half ? (m >> 32) : (m & 0xffffffffull));
        const int k = mh != 0u ? __ffs(mh) - 1 : 31;       // 0 only for a CDF that is not finite
        const int nlo = lo + k * step;
        const int nhi = nlo + step - 1;
        hi = nhi < hi ? nhi : hi;
        lo = nlo < hi ? nlo : hi;
    }
    return lo;
}

// Ancestor of one point (unsorted points): the chunk by its end in LDS, then the
// element.
__device__ __forceinline__ int cdf_search(double U, const CdfView& v) {
    const double clast = v.last();
    const int c = first_true(0, v.nchunks - 1, [&](int q) { return cdf_past(U, v.cend[q], clast); });
    const int j0 = c * v.chunk;
    const int j1 = (v.N - j0 < v.chunk ? v.N : j0 + v.chunk) - 1;
    return first_true(j0, j1, [&](int j) { return cdf_past(U, v.at(c, j), clast); });
}

// Ancestors of the points of a whole wave whose valid lanes hold non-decreasing
// points in lane order (systematic and stratified resampling, one point per
// particle, particles consecutive along the lanes). Every lane of the wave must
// call it (invalid lanes get an unspecified result). The ancestor is
// non-decreasing in the point, so those of the wave's first and last points bound
// every lane's: the two half-waves find them together (the chunk from the ends in
// LDS, then 32 probes a level inside it), the window between them comes into the
// wave's LDS row `win` with independent loads, and each lane searches it there.
// Dependent loads from memory: three levels and the window for chunks of 2048,
// where a search over all of C and then of the window in memory took four levels
// at N = 2^17 and one load per halving of the window (about seven).
constexpr int kCdfWin = 256;
__device__ __forceinline__ int cdf_search_sorted_wave(double U, bool valid, const CdfView& v,
                                                      double* win) {
    const int lane = threadIdx.x & 63;
    const double clast = v.last();
    // the wave's first and last valid points (lane order = point order)
    const unsigned long long vm = __ballot(valid);
    if (vm == 0ull) return 0;
    const int first = __ffsll(static_cast<long long>(vm)) - 1;
    const int last = 63 - __clzll(static_cast<long long>(vm));
    const double u_first = __shfl(U, first, 64);
    const double u_last = __shfl(U, last, 64);
    const double us = (lane >> 5) ? u_last : u_first;
    const int c = first_true_half(0, v.nchunks - 1,
                                  [&](int q) { return cdf_past(us, v.cend[q], clast); });
    const int j0 = c * v.chunk;
    const int j1 = (v.N - j0 < v.chunk ? v.N : j0 + v.chunk) - 1;
    const int e = first_true_half(j0, j1, [&](int j) { return cdf_past(us, v.at(c, j), clast); });
    const int a = __shfl(e, 0, 64);
    const int b = __shfl(e, 32, 64);
    const int ca = __shfl(c, 0, 64);
    const int cb = __shfl(c, 32, 64);
    const int len = b - a + 1;
    if (len > kCdfWin || cb > ca + 1) {
        if (!valid) return a;
        return first_true(a, b, [&](int j) { return cdf_past(U, v.at(j / v.chunk, j), clast); });
    }
#pragma unroll
    for (int r = 0; r < kCdfWin; r += kWave)
        if (r + lane < len) win[r + lane] = v.at(a + r + lane < cb * v.chunk ? ca : cb, a + r + lane);
    wave_sync();
    const int j = a + first_true(0, len - 1, [&](int q) { return cdf_past(U, win[q], clast); });
    wave_sync();                          // read before the row is filled again
    return j;
}

}  // namespace smc
