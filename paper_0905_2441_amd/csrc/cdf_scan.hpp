// Double-double prefix sums of the resampling weights, one workgroup per chunk.
#pragma once
#include "internal.hpp"
#include "reduce.hpp"

namespace smc {

// Inclusive prefixes (double-double) of the piece [piece, piece + kRedBlock*PER)
// clipped to `end`, offset by `carry`, stored rounded in two halves to
// out_hi/out_lo; returns the prefix stored for the piece's last element. Each
// thread scans PER consecutive elements, but the weights are read and the prefixes
// written striped across the block (element e*256 + t by thread t: every wave
// access is 512 contiguous bytes) through LDS, whose rows are padded by one double
// per PER elements so that the per-thread runs do not fall on the same banks.
template <int PER, class WeightAt>
__device__ __forceinline__ dd scan_piece(int piece, int end, dd carry, double* out_hi,
                                         double* out_lo, WeightAt weight) {
    constexpr int kPiece = kRedBlock * PER;
    constexpr int kPadded = kPiece + kPiece / PER;
    __shared__ double sh_hi[kPadded], sh_lo[kPadded];
    auto at = [](int j) { return j + j / PER; };
    const int t = threadIdx.x;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = e * kRedBlock + t;
        sh_hi[at(j)] = piece + j < end ? weight(piece + j) : 0.0;
    }
    __syncthreads();
    const int base = t * PER;
    dd pre[PER];
    dd run = dd_zero();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        if (piece + base + e < end) run = dd_add(run, sh_hi[at(base + e)]);
        pre[e] = run;
    }
    dd total;
    const dd excl = block_dd_exclusive_scan(run, total);     // ends with a barrier
    const dd lead = dd_add(carry, excl);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const dd c = dd_add(lead, pre[e]);
        sh_hi[at(base + e)] = c.hi;
        sh_lo[at(base + e)] = c.lo;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = e * kRedBlock + t;
        if (piece + j < end) {
            out_hi[piece + j] = sh_hi[at(j)];
            out_lo[piece + j] = sh_lo[at(j)];
        }
    }
    const int tail = at((end - piece < kPiece ? end - piece : kPiece) - 1);
    const dd out{sh_hi[tail], sh_lo[tail]};
    __syncthreads();
    return out;
}

// Within-chunk inclusive prefixes of chunk b of the fused step's layout (up to
// kMaxChunks chunks of kScanChunk-element pieces) into cdf_hi/cdf_lo and the
// chunk's total (the prefix stored for its last element) into chunk_tot.
template <class WeightAt>
__device__ __forceinline__ void scan_chunk(int b, int N, int chunk, double* cdf_hi,
                                           double* cdf_lo, double* chunk_tot, WeightAt weight) {
    const int begin = b * chunk;
    const int end = min(N, begin + chunk);
    dd carry = dd_zero();
    for (int piece = begin; piece < end; piece += kScanChunk)
        carry = scan_piece<kScanPerThread>(piece, end, carry, cdf_hi, cdf_lo, weight);
    if (threadIdx.x == 0) {
        chunk_tot[2 * b] = carry.hi;
        chunk_tot[2 * b + 1] = carry.lo;
    }
}

}  // namespace smc
