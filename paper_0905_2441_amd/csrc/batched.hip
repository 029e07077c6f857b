// Many independent SMC runs with uneven sizes in one step (serving-style batch).
//
// Each run r owns a contiguous block of particles [p_off, p_off + N_r) in the
// concatenated state arrays (its theta block is the usual [kd][N_r] layout at
// theta + kd*p_off) and a contiguous block of observations [y_off, y_off + n_r).
// All runs share the model constants and the tempering schedule and advance in
// lockstep; each has its own Philox key (seed), so a run's random numbers are
// exactly those it would draw alone.
//
// A batched tempering step is four launches whatever the number of runs, the first
// three over every run's chunks of 2048 particles (cdf_layout), a workgroup each,
// so that one large run keeps no compute unit alone at work:
//   k_b_reweight  the chunk's reweight and log-sum-exp partial;
//   k_b_mid       combines the run's partials (every workgroup of the run, in the
//                 same order); the first one publishes the run's evidence
//                 increment, ESS and decision; a run that resamples has its
//                 chunk's CDF prefixes scanned;
//   k_b_gather    a resampling run's ancestor search and gather (others exit);
// One workgroup per run took 144 us for the reweight and 1.34 ms for the
// resampling of 64 runs of up to 65536 particles; 13, 14 and 42 us now.
//   k_b_move      a workgroup per work unit. A unit is 8 / S consecutive 64-particle tiles
//                 of one run, each moved by S of the workgroup's 8 waves
//                 (proposal + mixture likelihood over the run's n_r
//                 observations, the S waves splitting the data + accept). S is
//                 per run (launch table or built-in rule), so short-data runs
//                 fill the workgroup with several tiles instead of leaving waves
//                 idle. Units are listed, and so started, longest data first
//                 (LPT), so runs whose work differs by 10^3 balance.
// and a one-thread kernel that advances the step counter.
#include <algorithm>

#include "cdf_scan.hpp"
#include "gmm_common.hpp"
#include "reduce.hpp"

namespace smc {
namespace {

constexpr int kBatchBlock = kBatchWaves * kWave;
// Units per launch: a grid of workgroups of up to 1024 threads has below 2^32.
constexpr int kMaxUnitGrid = 1 << 21;

// One chunk's reweight and its log-sum-exp partial. A thread's elements are loaded
// together, then summed about their own maximum (one exp each for the old and the
// new weights, none waiting on another).
__global__ void __launch_bounds__(kRedBlock)
k_b_reweight(const BatchRun* __restrict__ runs, const BatchChunk* __restrict__ chunks,
             double* __restrict__ logw, const double* __restrict__ l, StepSrc src,
             RwPartial* __restrict__ part, int* status) {
    const BatchChunk ch = chunks[blockIdx.x];
    const BatchRun rd = runs[ch.run];
    const int t = step_index(src);
    const double dbeta = src.beta_dev[t] - src.beta_dev[t - 1];
    double* lw = logw + rd.p_off;
    const double* lr = l + rd.p_off;
    const int begin = ch.index * rd.chunk;
    const int end = min(rd.N, begin + rd.chunk);
    Lse3 o = lse3_empty(), nw = lse3_empty();
    bool bad = false;
    for (int piece = begin; piece < end; piece += kScanChunk) {
        double lo[kScanPerThread], ln[kScanPerThread];
#pragma unroll
        for (int e = 0; e < kScanPerThread; ++e) {
            const int p = piece + e * kRedBlock + static_cast<int>(threadIdx.x);
            lo[e] = p < end ? lw[p] : -INFINITY;
            ln[e] = p < end ? lr[p] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < kScanPerThread; ++e) {
            const int p = piece + e * kRedBlock + static_cast<int>(threadIdx.x);
            ln[e] = p < end ? lo[e] + dbeta * ln[e] : -INFINITY;
            if (p < end) lw[p] = ln[e];
            bad = bad || (ln[e] != ln[e]) || (ln[e] == INFINITY);
        }
        o = lse3_merge(o, lse3_of(lo));
        nw = lse3_merge(nw, lse3_of(ln));
    }
    if (bad) atomicOr(status, kStatusNaN);
    block_lse3_pair(o, nw);
    if (threadIdx.x == 0) part[blockIdx.x] = RwPartial{o.m, o.s1, nw.m, nw.s1, nw.s2, 0.0};
}

// Every chunk's workgroup combines its run's partials in the same order, so all
// reach the same decision; the run's first one publishes the step state and the
// statistics; if the run resamples, each scans its chunk of the weights.
__global__ void __launch_bounds__(kRedBlock)
k_b_mid(const BatchRun* __restrict__ runs, const BatchChunk* __restrict__ chunks,
        const double* __restrict__ logw, StepSrc src, const RwPartial* __restrict__ part,
        StepState* __restrict__ st, double* __restrict__ stats, double ess_frac,
        double* __restrict__ chunk_tot, double* __restrict__ cdf_hi, double* __restrict__ cdf_lo,
        int* status) {
    __shared__ double sh_M, sh_S;
    __shared__ int sh_fire;
    const BatchChunk ch = chunks[blockIdx.x];
    const BatchRun rd = runs[ch.run];
    Lse3 o = lse3_empty(), nw = lse3_empty();
    for (int q = threadIdx.x; q < rd.nchunks; q += blockDim.x) {
        const RwPartial v = part[rd.c_off + q];
        o = lse3_merge(o, Lse3{v.mo, v.so, 0.0});
        nw = lse3_merge(nw, Lse3{v.mn, v.s1, v.s2});
    }
    block_lse3_pair(o, nw);
    if (threadIdx.x == 0) {
        const double ess = (nw.s1 * nw.s1) / nw.s2;
        const int fire = (ess_frac > 0.0) && (ess < ess_frac * static_cast<double>(rd.N));
        sh_M = nw.m;
        sh_S = nw.s1;
        sh_fire = fire;
        if (ch.index == 0) {
            StepState s{};
            s.M = nw.m;
            s.S = nw.s1;
            s.S2 = nw.s2;
            s.lse_old = (o.m == -INFINITY) ? -INFINITY : o.m + log(o.s1);
            s.lse_new = (nw.m == -INFINITY) ? -INFINITY : nw.m + log(nw.s1);
            s.ess = ess;
            s.resampled = fire;
            s.t = step_index(src);
            if (nw.m == -INFINITY || !(ess == ess)) atomicOr(status, kStatusAllZeroWeight);
            st[ch.run] = s;
            double* sr = stats + 4 * static_cast<size_t>(ch.run);
            sr[0] += s.lse_new - s.lse_old;
            sr[1] = s.ess;
            if (fire) sr[2] += 1.0;
        }
    }
    __syncthreads();
    if (!sh_fire) return;
    const double M = sh_M, S = sh_S;
    const double* lw = logw + rd.p_off;
    scan_chunk(ch.index, rd.N, rd.chunk, cdf_hi + rd.p_off, cdf_lo + rd.p_off,
               chunk_tot + 2 * static_cast<size_t>(rd.c_off),
               [&](int j) { return exp_fp64(lw[j] - M) / S; });
}

// A resampling run's ancestors and gather, a chunk of offspring per workgroup;
// logw = 0.
__global__ void __launch_bounds__(kRedBlock)
k_b_gather(const BatchRun* __restrict__ runs, const BatchChunk* __restrict__ chunks,
           const StepState* __restrict__ st, double* __restrict__ logw,
           const double* __restrict__ theta, const double* __restrict__ l,
           const double* __restrict__ chunk_tot, const double* __restrict__ cdf_hi,
           const double* __restrict__ cdf_lo, double* __restrict__ theta_tmp,
           double* __restrict__ l_tmp, int kd, int scheme) {
    __shared__ double offh[kMaxChunks], offl[kMaxChunks], cend[kMaxChunks];
    __shared__ double win[kRedBlock / kWave][kCdfWin];
    const BatchChunk ch = chunks[blockIdx.x];
    if (!st[ch.run].resampled) return;
    const BatchRun rd = runs[ch.run];
    const int N = rd.N;
    block_cdf_offsets(chunk_tot + 2 * static_cast<size_t>(rd.c_off), rd.nchunks, offh, offl, cend);
    const CdfView cdf{N, rd.chunk, rd.nchunks, cdf_hi + rd.p_off, cdf_lo + rd.p_off, offh, offl,
                      cend};
    const uint32_t step = static_cast<uint32_t>(st[ch.run].t);
    const double u = scheme == 0 ? u01_left_closed(draw(rd.seed, 0, 0, step, kResamp, 0).w0) : 0.0;
    const double* th = theta + static_cast<size_t>(kd) * rd.p_off;
    double* tt = theta_tmp + static_cast<size_t>(kd) * rd.p_off;
    const int begin = ch.index * rd.chunk;
    const int end = min(N, begin + rd.chunk);
    for (int i0 = begin + wave_id() * kWave; i0 < end; i0 += kRedBlock) {
        const int i = i0 + lane_id();
        const double U = resample_point(scheme, rd.seed, step, i < N ? i : N - 1, N, u);
        const int j = scheme == SMC_RESAMPLE_MULTINOMIAL
                          ? cdf_search(U, cdf)
                          : cdf_search_sorted_wave(U, true, cdf, win[wave_id()]);
        if (i >= end) continue;
        for (int c = 0; c < kd; ++c)
            tt[static_cast<size_t>(c) * N + i] = th[static_cast<size_t>(c) * N + j];
        l_tmp[rd.p_off + i] = l[rd.p_off + j];
        logw[rd.p_off + i] = 0.0;
    }
}

// Every run's draw from the prior, by chunks.
template <int KD>
__global__ void __launch_bounds__(kRedBlock)
k_b_prior(const BatchRun* __restrict__ runs, const BatchChunk* __restrict__ chunks, GmmDev g,
          double* __restrict__ theta) {
    const BatchChunk ch = chunks[blockIdx.x];
    const BatchRun rd = runs[ch.run];
    const int begin = ch.index * rd.chunk;
    const int end = min(rd.N, begin + rd.chunk);
    for (int p = begin + static_cast<int>(threadIdx.x); p < end; p += kRedBlock)
        prior_draw<KD>(p, rd.N, rd.seed, g, theta + static_cast<size_t>(KD) * rd.p_off);
}

// The log-likelihood of every run's particles: a workgroup takes a unit's tiles,
// each over the unit's slices, with the same arithmetic as the single-run kernel
// at those slices. One launch per run was bound by its own few workgroups (64
// runs of up to 65536 particles and 100000 data, k = 4, FP32: 9.3 ms in 64
// launches, 6.0 ms in one; 7.4 without the bound on registers, at 86 of them,
// which leaves a CU one workgroup of the two).
template <int K, int PREC>
__global__ void __launch_bounds__(kMaxSlices * kWave, PREC == SMC_PREC_FP32 && K <= 4 ? 8 : 4)
k_b_loglik(const BatchRun* __restrict__ runs, const BatchUnit* __restrict__ units,
           const float* __restrict__ y, const double* __restrict__ theta, GmmDev g,
           double* __restrict__ l, int* status) {
    __shared__ double red[kMaxSlices][kWave];
    const BatchUnit un = units[blockIdx.x];
    const BatchRun rd = runs[un.run];
    const int lane = lane_id();
    const int w = wave_uniform(threadIdx.x / kWave);
    const int S = wave_uniform(un.slices);
    const int grp = w / S;                           // this wave's tile within the unit
    const int sl = w - grp * S;                      // and its data slice
    const bool active = grp < un.ntiles;
    const int N = rd.N, n = rd.n;
    const int p = (un.tile0 + (active ? grp : 0)) * kWave + lane;
    const int pc = p < N ? p : N - 1;
    if (active) {
        const double* th = theta + static_cast<size_t>(K) * rd.p_off;
        double pr[K];
#pragma unroll
        for (int c = 0; c < K; ++c) pr[c] = th[static_cast<size_t>(c) * N + pc];
        int j0, j1;
        slice_bounds(n, sl, S, j0, j1);
        red[w][lane] = slice_partial<K, 1, PREC>(y + rd.y_off, j0, j1, pr, g, true,
                                                 PivotStage{pivot_row<PREC, 1, kMaxSlices>()});
    }
    __syncthreads();
    if (active && sl == 0 && p < N) {
        const double v = finish_loglik<PREC>(sum_slices(red + w, S), n, g);
        l[rd.p_off + p] = v;
        if (v != v) atomicOr(status, kStatusNaN);
    }
}

// One move of a unit's tiles. Bound by the likelihood's arithmetic. FP32 up to
// k = 4 fits 64 registers with its spills outside the loop over the data, four
// workgroups to a CU; as a persistent loop over a work counter it took 127, since
// the loop's invariants were held through the likelihood (64 runs of up to 65536
// particles and 100000 data, k = 4: 5.02 ms so, 4.95 with a workgroup a unit at 91
// registers, 4.65 at 80, 4.51 at 64; three steps and the first likelihood at 64, 80
// and 96 registers, k = 1: 2.01, 2.07 and 2.28 ms, k = 2: 9.00, 9.19 and 9.64, k = 3:
// 14.5, 15.1 and 15.6).
template <int K, int PREC>
__global__ void __launch_bounds__(kBatchBlock, PREC == SMC_PREC_FP32 && K <= 4 ? 8 : 4)
k_b_move(const BatchRun* __restrict__ runs, const BatchUnit* __restrict__ units,
         const float* __restrict__ y, double* theta, double* l,
         const double* __restrict__ logw, double* __restrict__ W,
         const double* __restrict__ theta_tmp, const double* __restrict__ l_tmp,
         const StepState* __restrict__ st, StepSrc src, double sd, uint32_t move, int first,
         GmmDev g, unsigned long long* n_acc, int* status) {
    constexpr int KD = K;
    __shared__ double red[kBatchWaves][kWave];
    __shared__ double prs[kBatchWaves][KD][kWave];
    __shared__ double lus[kBatchWaves][kWave];
    const int lane = lane_id();
    const int w = wave_uniform(threadIdx.x / kWave);
    const BatchUnit un = units[blockIdx.x];
    const BatchRun rd = runs[un.run];
    const int S = wave_uniform(un.slices);
    const int grp = w / S;                       // this wave's tile within the unit
    const int sl = w - grp * S;                  // and its data slice
    const bool active = grp < un.ntiles;
    const int N = rd.N;
    const int n = rd.n;
    const int p = (un.tile0 + (active ? grp : 0)) * kWave + lane;
    const int pc = p < N ? p : N - 1;
    const StepState* sr = st + un.run;
    const uint32_t step = static_cast<uint32_t>(sr->t);
    const bool use_alt = first && sr->resampled;
    double* th_run = theta + static_cast<size_t>(KD) * rd.p_off;
    double* l_run = l + rd.p_off;
    const double* th_src = use_alt ? theta_tmp + static_cast<size_t>(KD) * rd.p_off : th_run;
    const double l_src = use_alt ? l_tmp[rd.p_off + pc] : l_run[pc];
    // the tile's Box-Muller pairs and its log u shared out over its S waves (an
    // idle wave of a short last unit draws none but meets the barrier)
    double pr[KD];
    block_proposals<KD>(rd.seed, static_cast<uint32_t>(pc), step, move, th_src, N, pc, sd,
                        active ? sl : (KD + 1) / 2 + 1, S, prs[grp], pr, nullptr, nullptr,
                        nullptr, lus[grp]);
    double part = 0.0;
    if (active) {
        int j0, j1;
        slice_bounds(n, sl, S, j0, j1);
        part = slice_partial<K, 1, PREC>(y + rd.y_off, j0, j1, pr, g, near_data(l_src, n, g),
                                         PivotStage{pivot_row<PREC, 1, kBatchWaves>()});
    }
    red[w][lane] = part;
    __syncthreads();
    if (active && sl == 0) {
        bool acc = false;
        if (p < N) {
            const double l_prop = finish_loglik<PREC>(sum_slices(red + w, S), n, g);
            MoveStep ms{};
            if (first) {
                ms.theta_alt = theta_tmp + static_cast<size_t>(KD) * rd.p_off;
                ms.l_alt = l_tmp + rd.p_off;
                ms.state = sr;
                ms.W_out = W + rd.p_off;
                ms.logw = const_cast<double*>(logw) + rd.p_off;
            }
            const MoveSource srcs = move_source(ms, th_run, l_run);
            acc = rwmh_accept<KD>(p, p, N, [&](int c) { return pr[c]; }, l_prop, srcs, th_run,
                                  l_run, nullptr, src, step, rd.seed, move, g, status, ms,
                                  nullptr, &lus[grp][lane]);
        }
        const unsigned long long mask = __ballot(acc);
        if (lane == 0 && n_acc != nullptr && mask != 0ull)
            atomicAdd(n_acc, static_cast<unsigned long long>(__popcll(mask)));
    }
}

__global__ void k_b_end(int* t_dev) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *t_dev += 1;
}

}  // namespace

hipError_t launch_batch_init(const BatchDev& b, const GmmDev& g, const float* y, double* theta,
                             double* l, int prec, int* status, hipStream_t s) {
    const int pi = prec == SMC_PREC_FP32 ? 1 : 0;
    const dim3 block(kMaxSlices * kWave);
#define SMC_BI(KK)                                                                              \
    if (g.k == KK) {                                                                            \
        hipLaunchKernelGGL((k_b_prior<KK>), dim3(b.n_chunks), dim3(kRedBlock), 0, s, b.runs,    \
                           b.chunks, g, theta);                                                 \
        for (int u = 0; u < b.n_init_units[pi]; u += kMaxUnitGrid) {                            \
            const dim3 grid(static_cast<unsigned>(std::min(kMaxUnitGrid, b.n_init_units[pi] - u))); \
            if (prec == SMC_PREC_FP32)                                                          \
                hipLaunchKernelGGL((k_b_loglik<KK, SMC_PREC_FP32>), grid, block, 0, s, b.runs,  \
                                   b.init_units[pi] + u, y, theta, g, l, status);               \
            else                                                                                \
                hipLaunchKernelGGL((k_b_loglik<KK, SMC_PREC_FP64>), grid, block, 0, s, b.runs,  \
                                   b.init_units[pi] + u, y, theta, g, l, status);               \
        }                                                                                       \
        return hipGetLastError();                                                               \
    }
    SMC_BI(1) SMC_BI(2) SMC_BI(3) SMC_BI(4) SMC_BI(5) SMC_BI(6) SMC_BI(7) SMC_BI(8)
#undef SMC_BI
    return hipErrorInvalidValue;
}

hipError_t launch_batch_step(const BatchDev& b, const GmmDev& g, const float* y, double* theta,
                             double* l, double* logw, double* W, const double* beta, int T,
                             int* t_dev, double sd, int n_moves, double ess_frac, int prec,
                             double* stats, unsigned long long* n_acc, int* status, int scheme,
                             hipStream_t s) {
    StepSrc src{};
    src.t_dev = t_dev;
    src.beta_dev = beta;
    src.t_max = T;
    hipLaunchKernelGGL(k_b_reweight, dim3(b.n_chunks), dim3(kRedBlock), 0, s, b.runs, b.chunks,
                       logw, l, src, b.part, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_mid, dim3(b.n_chunks), dim3(kRedBlock), 0, s, b.runs, b.chunks, logw,
                       src, b.part, b.state, stats, ess_frac, b.chunk_tot, b.cdf_hi, b.cdf_lo,
                       status);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_gather, dim3(b.n_chunks), dim3(kRedBlock), 0, s, b.runs, b.chunks,
                       b.state, logw, theta, l, b.chunk_tot, b.cdf_hi, b.cdf_lo, b.theta_tmp,
                       b.l_tmp, g.k * g.d, scheme);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int pi = prec == SMC_PREC_FP32 ? 1 : 0;
    for (int m = 0; m < n_moves; ++m) {
        for (int u = 0; u < b.n_units[pi]; u += kMaxUnitGrid) {
            const dim3 grid(static_cast<unsigned>(std::min(kMaxUnitGrid, b.n_units[pi] - u)));
            const BatchUnit* units = b.units[pi] + u;
#define SMC_BM(KK, P)                                                                           \
            hipLaunchKernelGGL((k_b_move<KK, P>), grid, dim3(kBatchBlock), 0, s, b.runs, units, \
                               y, theta, l, logw, W, b.theta_tmp, b.l_tmp, b.state, src, sd,    \
                               static_cast<uint32_t>(m), m == 0 ? 1 : 0, g, n_acc, status)
#define SMC_BK(KK)                                                                              \
            if (g.k == KK) {                                                                    \
                if (prec == SMC_PREC_FP32) SMC_BM(KK, SMC_PREC_FP32);                           \
                else SMC_BM(KK, SMC_PREC_FP64);                                                 \
            }
            SMC_BK(1) SMC_BK(2) SMC_BK(3) SMC_BK(4) SMC_BK(5) SMC_BK(6) SMC_BK(7) SMC_BK(8)
#undef SMC_BK
#undef SMC_BM
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    hipLaunchKernelGGL(k_b_end, dim3(1), dim3(64), 0, s, t_dev);
    return hipGetLastError();
}

}  // namespace smc
