// d-dimensional mixture log-likelihood on the matrix cores (gfx950 MFMA).
//
// For d-variate components with covariance sigma2*I the per-component term is
// a quadratic form; in base-2 units
//   a_{j,i} = log2 w_i - s2 ||y_j - mu_i||^2,        s2 = log2(e) / (2 sigma2)
//           = (2 s2 y_j) . mu_i  - s2 ||y_j||^2  + (log2 w_i - s2 ||mu_i||^2),
// which is one contraction over K = 64 between a data row and a component
// column. BF16 keeps 8 significant bits, so every FP32/FP64 value is split into
// three BF16 parts (hi + mid + lo, exact for FP32 data and 24-bit accurate for
// the FP64 means) and the cross term keeps the six products down to 2^-16 of
// the leading one (hi*hi, hi*mid, mid*hi, hi*lo, lo*hi, mid*mid); the two norm
// terms enter the same contraction as three BF16 parts against ones. Products
// of BF16 values are exact in the FP32 accumulator, so the result carries only
// FP32 accumulation error and the 2^-24 truncation of the dropped products.
// The quadratic forms are evaluated at the represented means (hi+mid+lo), so
// the norm and cross terms are consistent and no systematic bias is introduced.
//
// K layout (eight slots of eight coordinates; slots 0-3 feed the first
// 16x16x32 MFMA and slots 4-7 the second):
//   slot  A (data row j)                         B (particle p, component i)
//   0     u_hi                                   mu_hi
//   1     u_hi                                   mu_mid
//   2     u_mid                                  mu_hi
//   3     u_hi                                   mu_lo
//   4     u_lo                                   mu_hi
//   5     u_mid                                  mu_mid
//   6     [Y_hi, Y_mid, Y_lo, 1, 1, 1, 0, 0]     [1, 1, 1, C_hi, C_mid, C_lo, 0, 0]
//   7     0                                      0
// with u = 2 s2 y (FP32), Y = -s2 ||y||^2, C_i = log2 w_i - s2 ||mu_i||^2.
// In the 16x16x32 operand layout lane l holds row (l mod 16) of A and column
// (l mod 16) of B for K elements 8*(l/16)..+7, so every lane handles exactly one
// slot per MFMA, and the output lane holds four data rows 4*(l/16)..+3 of its
// column. One MFMA pair per mixture component puts all k component values of a
// (datum, particle) pair in the same lane: the epilogue (hardware exp2, sum,
// product accumulation; with the per-datum max shift only for waves holding a
// particle far from the data) needs no cross-lane traffic.
//
// Workgroup = 4 waves x 16 particles; the data rows of a slice are staged in LDS
// (16 KB stages, double-buffered, 16-byte slots XOR-swizzled by row to spread
// the banks) and shared by the 4 waves. Slices of the data go to different
// workgroups; their partial sums are combined in slice order by a second kernel.
//
// Bound by VALU issue (the matrix instructions run beside it): per 16 x 16 tile
// and k = 8, 32 exp2 at two issue slots, 28 adds and 16 issues of the matrix
// unit in the direct form, 0.85 ms at N = 16384, n = 65536 (1.26 ms in the
// shifted form with its maxima and differences). Measured 1.03 and 1.38 ms
// (1.28 and 1.61 before): the direct form consumes one component's results at a
// time with the next one's products in flight, so the results stay out of the
// accumulation registers (32 moves a tile), four exp2 go before their four adds
// (an exp2 result needs a slot before its use), a whole tile carries no per-row
// bounds test, and the stages are loaded from memory straight into LDS, which
// leaves room for 4 waves per SIMD. Recomputing the products in the shifted form
// instead of holding all k results was slower (1.78 ms), and so was a larger
// register budget at 3 waves (1.42 ms shifted).
#include "gmm_common.hpp"

namespace smc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowElems = 64;              // BF16 per staged data row
constexpr int kRowBytes = 2 * kRowElems;
constexpr int kTileRows = 16;
constexpr int kStageTiles = 8;
constexpr int kStageRows = kStageTiles * kTileRows;
constexpr int kStageBytes = kStageRows * kRowBytes;   // 16 KB
constexpr int kDdBlock = 256;                          // 4 waves, 64 particles
constexpr int kDdDim = 8;                              // coordinates per slot

__device__ __forceinline__ void split3(float x, __bf16& h, __bf16& m, __bf16& l) {
    h = static_cast<__bf16>(x);
    const float r1 = x - static_cast<float>(h);
    m = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(m);
    l = static_cast<__bf16>(r2);
}

// FP64 value -> three BF16 parts and the value they represent (exact sum).
__device__ __forceinline__ double split3d(double x, __bf16& h, __bf16& m, __bf16& l) {
    h = static_cast<__bf16>(static_cast<float>(x));
    const double r1 = x - static_cast<double>(static_cast<float>(h));
    m = static_cast<__bf16>(static_cast<float>(r1));
    const double r2 = r1 - static_cast<double>(static_cast<float>(m));
    l = static_cast<__bf16>(static_cast<float>(r2));
    return (static_cast<double>(static_cast<float>(h)) + static_cast<double>(static_cast<float>(m))) +
           static_cast<double>(static_cast<float>(l));
}

// One thread per (padded) data row: the 64-element A row of the K layout.
__global__ void __launch_bounds__(256)
k_dd_prep(const float* __restrict__ y, int n, int n_pad, double s2, __bf16* __restrict__ A) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_pad) return;
    bf16x8 slot[8];
    const __bf16 zero = static_cast<__bf16>(0.0f);
    const __bf16 one = static_cast<__bf16>(1.0f);
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) slot[s][c] = zero;
    if (j < n) {
        double yn = 0.0;
#pragma unroll
        for (int c = 0; c < kDdDim; ++c) {
            const float yc = y[static_cast<size_t>(j) * kDdDim + c];
            yn += static_cast<double>(yc) * static_cast<double>(yc);
            const float u = static_cast<float>(2.0 * s2 * static_cast<double>(yc));
            __bf16 h, m, l;
            split3(u, h, m, l);
            slot[0][c] = h;
            slot[1][c] = h;
            slot[2][c] = m;
            slot[3][c] = h;
            slot[4][c] = l;
            slot[5][c] = m;
        }
        __bf16 h, m, l;
        split3(static_cast<float>(-s2 * yn), h, m, l);
        slot[6][0] = h;
        slot[6][1] = m;
        slot[6][2] = l;
        slot[6][3] = one;
        slot[6][4] = one;
        slot[6][5] = one;
    }
    bf16x8* dst = reinterpret_cast<bf16x8*>(A + static_cast<size_t>(j) * kRowElems);
#pragma unroll
    for (int s = 0; s < 8; ++s) dst[s] = slot[s];
}

// One thread per (particle, component): the 64-element B column of the K
// layout, from the current means or (PROP) from the random-walk proposal of the
// move, which is also stored for the accept kernel.
template <bool PROP>
__global__ void __launch_bounds__(256)
k_dd_build(const double* __restrict__ theta, int N, int K, GmmDev g, double s2, MoveStep ms,
           double sd, uint64_t seed, StepSrc src, uint32_t move, __bf16* __restrict__ B,
           double* __restrict__ theta_prop) {
    int p, i;
    if (!dd_column(blockIdx.x * blockDim.x + threadIdx.x, N, K, p, i)) return;
    const double* th = theta;
    if constexpr (PROP) {
        const bool rs = ms.state != nullptr && ms.state->resampled != 0;
        th = (rs && ms.theta_alt) ? ms.theta_alt : (ms.theta_src ? ms.theta_src : theta);
    }
    double mu[kDdDim];
#pragma unroll
    for (int c = 0; c < kDdDim; ++c) mu[c] = th[static_cast<size_t>(i * kDdDim + c) * N + p];
    if constexpr (PROP) {
        const uint32_t step = static_cast<uint32_t>(step_index(src));
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const Words4 wd = draw(seed, static_cast<uint32_t>(p), 2 * i + b, step, kProp, move);
            double z0, z1, z2, z3;
            box_muller(wd.w0, wd.w1, z0, z1);
            box_muller(wd.w2, wd.w3, z2, z3);
            mu[4 * b + 0] = mu[4 * b + 0] + sd * z0;
            mu[4 * b + 1] = mu[4 * b + 1] + sd * z1;
            mu[4 * b + 2] = mu[4 * b + 2] + sd * z2;
            mu[4 * b + 3] = mu[4 * b + 3] + sd * z3;
        }
#pragma unroll
        for (int c = 0; c < kDdDim; ++c) theta_prop[static_cast<size_t>(i * kDdDim + c) * N + p] = mu[c];
    }
    if (B == nullptr) return;              // the FP64 form reads the proposals themselves
    const __bf16 zero = static_cast<__bf16>(0.0f);
    const __bf16 one = static_cast<__bf16>(1.0f);
    bf16x8 sh, sm, sl, s6, s7;
    double nrm = 0.0;
#pragma unroll
    for (int c = 0; c < kDdDim; ++c) {
        __bf16 h, m, l;
        const double rep = split3d(mu[c], h, m, l);
        nrm += rep * rep;
        sh[c] = h;
        sm[c] = m;
        sl[c] = l;
        s7[c] = zero;
    }
    __bf16 ch, cm, cl;
    split3(static_cast<float>(g.lw[i] * kLog2e - s2 * nrm), ch, cm, cl);
    s6[0] = one; s6[1] = one; s6[2] = one;
    s6[3] = ch; s6[4] = cm; s6[5] = cl;
    s6[6] = zero; s6[7] = zero;
    bf16x8* dst = reinterpret_cast<bf16x8*>(B + (static_cast<size_t>(p) * K + i) * kRowElems);
    dst[0] = sh;   // slot 0: mu_hi
    dst[1] = sm;   // slot 1: mu_mid
    dst[2] = sh;   // slot 2: mu_hi
    dst[3] = sl;   // slot 3: mu_lo
    dst[4] = sh;   // slot 4: mu_hi
    dst[5] = sm;   // slot 5: mu_mid
    dst[6] = s6;   // slot 6: ones against the data norm, the component constant
    dst[7] = s7;   // slot 7: padding
}

template <int K>
__global__ void __launch_bounds__(kDdBlock, 4)
k_dd_partial(const __bf16* __restrict__ A, int n, int n_pad, const __bf16* __restrict__ B, int N,
             int S, int unit_mass, double* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[2][kStageBytes];
    const int lane = lane_id();
    const int w = wave_uniform(wave_id());
    const int grp = lane >> 4;            // K group of this lane: slots grp and 4 + grp
    const int col = lane & 15;            // particle column within the wave's tile
    const int p = blockIdx.x * 64 + w * 16 + col;
    const int pc = p < N ? p : N - 1;
    const int slice = blockIdx.y;
    const int ntiles = n_pad / kTileRows;
    const int t0 = static_cast<int>((static_cast<int64_t>(ntiles) * slice) / S);
    const int t1 = static_cast<int>((static_cast<int64_t>(ntiles) * (slice + 1)) / S);

    // B operands of this lane: slot grp (first MFMA) and 4 + grp (second)
    bf16x8 b1[K], b2[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const bf16x8* colp = reinterpret_cast<const bf16x8*>(B + (static_cast<size_t>(pc) * K + i) * kRowElems);
        b1[i] = colp[grp];
        b2[i] = colp[4 + grp];
    }

    double msum = 0.0;
    float prod = 1.0f;
    int expo = 0;
    // direct form (no per-datum max shift) while every lane's tile product
    // stays >= 2^-100; the wave keeps the shifted form from the first tile
    // where one does not (the same rule as the VALU form's partial_fp32)
    bool direct = unit_mass != 0;
    constexpr float kFloor = 0x1p-100f;
    const int nst = (t1 - t0 + kStageTiles - 1) / kStageTiles;
    // a stage goes from memory straight into LDS, 16 bytes a lane: each load
    // fills 64 consecutive slots of LDS, so the swizzle is on the source (slot q
    // of row q / 8 holds the row's slot (q mod 8) ^ (row mod 8)); rows past the
    // slice repeat its last one and are not read
    auto load_stage = [&](int st, int buf) {
        const int row0 = (t0 + st * kStageTiles) * kTileRows;
        const int last = t1 * kTileRows - 1 - row0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q0 = (k * 4 + w) * kWave;
            const int row = (q0 + lane) >> 3;
            const int sl = (lane & 7) ^ (row & 7);
            const __bf16* src =
                A + static_cast<size_t>(row0 + min(row, last)) * kRowElems + sl * 8;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)src,
                (__attribute__((address_space(3))) void*)&lds[buf][q0 * 16], 16, 0, 0);
        }
    };
    if (nst > 0) load_stage(0, 0);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int buf = st & 1;
        if (st + 1 < nst) load_stage(st + 1, buf ^ 1);
        const int tile0 = t0 + st * kStageTiles;
        const int tiles_here = min(kStageTiles, t1 - tile0);
        for (int tt = 0; tt < tiles_here; ++tt) {
            const int row = tt * kTileRows + col;
            const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(
                &lds[buf][row * kRowBytes + ((grp ^ (row & 7)) << 4)]);
            const bf16x8 a2 = *reinterpret_cast<const bf16x8*>(
                &lds[buf][row * kRowBytes + (((4 + grp) ^ (row & 7)) << 4)]);
            const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
            auto exponents = [&](int i) {
                const f32x4 h = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1[i], z, 0, 0, 0);
                return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b2[i], h, 0, 0, 0);
            };
            const int grow = (tile0 + tt) * kTileRows + grp * 4;
            const bool whole = (tile0 + tt + 1) * kTileRows <= n;      // wave-uniform
            float e[4];
            bool done = false;
            if (direct) {
                f32x4 acc = exponents(0);
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    f32x4 next = acc;
                    if (i + 1 < K) next = exponents(i + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    float x[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = __builtin_amdgcn_exp2f(acc[r]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) e[r] = i == 0 ? x[r] : e[r] + x[r];
                    __builtin_amdgcn_sched_barrier(0);
                    acc = next;
                }
                if (!whole) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) e[r] = grow + r < n ? e[r] : 1.0f;
                }
                float pd = prod;
#pragma unroll
                for (int r = 0; r < 4; ++r) pd *= e[r];
                if (__all(pd >= kFloor)) {
                    prod = pd;
                    done = true;
                } else {
                    direct = false;
                }
            }
            if (!done) {
                f32x4 acc[K];
#pragma unroll
                for (int i = 0; i < K; ++i) acc[i] = exponents(i);
                float m[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    m[r] = acc[0][r];
#pragma unroll
                    for (int i = 1; i < K; ++i) m[r] = fmaxf(m[r], acc[i][r]);
                    e[r] = __builtin_amdgcn_exp2f(acc[0][r] - m[r]);
#pragma unroll
                    for (int i = 1; i < K; ++i) e[r] += __builtin_amdgcn_exp2f(acc[i][r] - m[r]);
                }
                if (!whole) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        m[r] = grow + r < n ? m[r] : 0.0f;
                        e[r] = grow + r < n ? e[r] : 1.0f;
                    }
                }
                float mblk = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    prod *= e[r];
                    mblk += m[r];
                }
                msum += static_cast<double>(mblk);
            }
            expo += __builtin_amdgcn_frexp_expf(prod);
            prod = __builtin_amdgcn_frexp_mantf(prod);
        }
        __syncthreads();                  // the next stage has arrived, this one is read
    }
    double v = msum + static_cast<double>(expo) + log2(static_cast<double>(prod));
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    if (grp == 0 && p < N) part[static_cast<size_t>(slice) * N + p] = v;
}

// ---------------------------------------------------------------- FP64 form
//
// The same contraction on the FP64 matrix instruction (v_mfma_f64_16x16x4_f64),
// for the d-dimensional FP64 likelihood: with a centre c of the data,
//   a_{j,i} = u_j . v_i + (C_i - Y_j),  u_j = y_j - c,  v_i = 2 s2 (mu_i - c),
//   C_i = log2 w_i - ||v_i||^2 / (4 s2),  Y_j = s2 ||u_j||^2,
// two instructions of K = 4 per component, started from C_i - Y_j. Lane l holds
// row (l mod 16) of A, column (l mod 16) of B at K element l / 16, and the four
// results of rows (l / 16) + 4 r of its column; A row a carries data row
// 4 (a mod 4) + a / 4 of the tile, so that a lane's results are data rows
// 4 (l / 16) + r. One component's results are consumed (exp2, add) before the
// next one's need a register, so a wave holds its particles' means (4 VGPRs per
// component) where the VALU form keeps all k*d of a particle per lane: at
// k = d = 8 those 128 VGPRs spilled, and the VALU form took 32.7 ms at
// N = 16384, n = 65536 against 6.2 ms here.
//
// Bound by FP64 issue: per (datum, particle) k = 8 components of 8 multiply-adds
// on the matrix unit and 16 instructions of exp2, its start and its sum (5.7 ms
// at the 5.8 cycles an FP64 instruction measured). Held to 3 waves per SIMD:
// 6.1 ms, against 6.6 at the 2 that the compiler's own choice of registers
// allows and 7.6 at 4 (spills).
//
// An exponent is a sum of terms of the size of Y_j and C_i. What its rounding does
// alike for every datum would not average out: the centre is an FP32 value (the
// mean of up to 64 data spread over the array, the same in every workgroup), so
// that u_j is exact; C_i is formed from the rounded v_i in two parts, so that the
// exponents are those of one mean within 2^-54 of mu_i, and the low part is a
// factor of the component's terms; s2, log2 w_i and ln 2 enter in two parts; and
// Y_j is summed as (s2 u) u, because a square of the few bits of a u ends in 0, 1
// or 4 of 8 and sums of them round one way. (With s2 in one part and Y_j = s2
// sum u^2 the relative error at n = 20000, near the modes, was 5.5e-16 at k = 8,
// sigma2 = 0.3 and 17.5e-16 at k = 2, 0.15, nearly all of it alike for every
// particle; it is 1.0e-16 and 1.5e-16, term by term 1.7e-16 and 2.8e-16.) What is
// left averages over the data: tiles holding a datum with Y_j above dd64_max_y(n), a
// datum that is not finite, or a particle with a mean that is not finite take the
// difference form (no expansion, plain FP64): 8 subtractions and 8 multiply-adds per
// component instead of the matrix unit's. A wave sets such tiles aside and works
// them off after every block of 64, when the expansion's operands are dead and their
// registers free, with the means from LDS: k = 8, N = 16384, n = 8192 1.34 ms (the
// expansion 0.81), where two passes of rolled loops over means and data in memory
// took 13.0 ms and the VALU form 4.1. Waves with a particle so far away that a
// datum's sum falls below 2^-1000 take each datum's largest exponent out first.
constexpr int kDd64StageTiles = 8;                     // data rows per LDS stage
constexpr int kDd64Rows = kDd64StageTiles * kTileRows;
constexpr int kDd64Block = 8;                          // stages per block: 64 tiles, a bit each
constexpr double kDd64MinC = -1.0e8;

constexpr double kLn2Tail = 2.3190468138462996e-17;    // ln 2 - kLn2
constexpr double kLog2eTail = 2.0355273740931033e-17;  // log2 e - kLog2e

typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int K>
__global__ void __launch_bounds__(kDdBlock, 3)
k_dd64_partial(const float* __restrict__ y, int n, const double* th, int N, GmmDev g, double s2,
               double s2_lo, double max_y, int S, double* part) {
    __shared__ double su[2][kDd64Rows * kDdDim];
    __shared__ __align__(16) double sy[2][kDd64Rows];
    __shared__ double cen[kDdDim];
    __shared__ double mean[K * kDdDim][64];          // the workgroup's particles' means
    const int lane = lane_id();
    const int w = wave_id();
    const int kg = lane >> 4;             // K element of the operands, row group of the results
    const int col = lane & 15;
    const int p = blockIdx.x * 64 + w * 16 + col;
    const int mp = w * 16 + col;          // this lane's column of `mean`
    for (int q = threadIdx.x; q < K * kDdDim * 64; q += kDdBlock) {
        const int pq = blockIdx.x * 64 + (q & 63);
        mean[q >> 6][q & 63] = th[static_cast<size_t>(q >> 6) * N + (pq < N ? pq : N - 1)];
    }
    const int slice = blockIdx.y;
    const int ntiles = (n + kTileRows - 1) / kTileRows;
    const int t0 = static_cast<int>((static_cast<int64_t>(ntiles) * slice) / S);
    const int t1 = static_cast<int>((static_cast<int64_t>(ntiles) * (slice + 1)) / S);

    // the centre
    {
        const float* yr = y + static_cast<size_t>((static_cast<int64_t>(lane) * n) / kWave) * kDdDim;
#pragma unroll
        for (int c = 0; c < kDdDim; ++c) {
            const float v = yr[c];
            const double sum = wave_sum(fabsf(v) < 1.0e18f ? static_cast<double>(v) : 0.0);
            if (threadIdx.x == 0) cen[c] = static_cast<double>(static_cast<float>(sum * (1.0 / kWave)));
        }
    }
    __syncthreads();

    // stages: thread t brings half a data row, (t / 2, 4 coordinates)
    const int half = threadIdx.x & 1;
    const int srow = threadIdx.x >> 1;
    double hc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) hc[q] = cen[half * 4 + q];
    float yv[4];
    auto load_stage = [&](int st) {
        const int row = (t0 * kTileRows) + st * kDd64Rows + srow;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            yv[q] = row < n ? y[static_cast<size_t>(row) * kDdDim + half * 4 + q] : 0.0f;
    };
    auto store_stage = [&](int buf) {
        double ys = 0.0;                             // (s2 d) d, not s2 (d d): see above
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double d = static_cast<double>(yv[q]) - hc[q];
            ys = fma(fma(s2, d, s2_lo * d), d, ys);
            su[buf][srow * kDdDim + half * 4 + q] = d;
        }
        ys += __shfl_xor(ys, 1, kWave);
        if (half == 0) sy[buf][srow] = ys;
    };
    const double quarter = 0.25 / s2;                // 1 / (4 s2) in two parts
    const double quarter_lo = fma(-quarter, 4.0 * s2_lo, fma(-quarter, 4.0 * s2, 1.0)) * quarter;
    const int nst = (t1 - t0 + kDd64StageTiles - 1) / kDd64StageTiles;
    if (nst > 0) {
        load_stage(0);
        store_stage(0);
    }
    __syncthreads();

    double prod = 1.0, msum = 0.0, nsum = 0.0;       // nsum: in natural units
    int expo = 0;
    bool direct = g.unit_mass != 0;
    const int arow = 4 * (col & 3) + (col >> 2);
    for (int s0 = 0; s0 < nst; s0 += kDd64Block) {
        const int s1 = min(nst, s0 + kDd64Block);
        // this lane's coordinates of its particle's means about the centre: formed for
        // every block of stages, so that they hold no registers in its difference form
        // (the empty asm keeps them from being read once for all blocks)
        double b1[K], b2[K], C[K];
        float cl[K];                                 // 2^(low part of C) - 1
        bool fine = true;
        {
            int mq = mp;
            asm volatile("" : "+v"(mq));
            const double c1 = cen[kg], c2 = cen[4 + kg];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const double m1 = mean[i * kDdDim + kg][mq] - c1;
                const double m2 = mean[i * kDdDim + 4 + kg][mq] - c2;
                b1[i] = fma(2.0 * s2, m1, 2.0 * s2_lo * m1);
                b2[i] = fma(2.0 * s2, m2, 2.0 * s2_lo * m2);
                // C_i in two parts from the rounded operands, so that the exponents are
                // those of one (slightly moved) mean whatever the datum
                const double p1 = b1[i] * b1[i], p2 = b2[i] * b2[i];
                dd q = two_sum(p1, p2);
                q.lo += fma(b1[i], b1[i], -p1) + fma(b2[i], b2[i], -p2);
                q = dd_add(q, dd{__shfl_xor(q.hi, 16, kWave), __shfl_xor(q.lo, 16, kWave)});
                q = dd_add(q, dd{__shfl_xor(q.hi, 32, kWave), __shfl_xor(q.lo, 32, kWave)});
                const double h = -q.hi * quarter;
                const double low = fma(-q.hi, quarter, -h) - q.hi * quarter_lo - q.lo * quarter;
                fine &= h >= kDd64MinC;                        // false for NaN
                const double lw = g.lw[i] * kLog2e;            // -inf: the component is skipped
                const double lw_lo = fma(g.lw[i], kLog2e, -lw) + g.lw[i] * kLog2eTail;
                const dd t = two_sum(h, lw);
                C[i] = t.hi;
                cl[i] = static_cast<float>((t.lo + low + lw_lo) * kLn2);
            }
        }
        fine = __all(fine);
        unsigned long long far = 0;                  // the block's tiles left to the differences
        for (int st = s0; st < s1; ++st) {
            const int buf = st & 1;
            const bool more = st + 1 < nst;
            if (more) load_stage(st + 1);
            const int tile0 = t0 + st * kDd64StageTiles;
            const int tiles = min(kDd64StageTiles, t1 - tile0);
            for (int tt = 0; tt < tiles; ++tt) {
                const double* ur = &su[buf][(tt * kTileRows + arow) * kDdDim];
                const double a1 = ur[kg], a2 = ur[4 + kg];
                double Y[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) Y[r] = sy[buf][tt * kTileRows + 4 * kg + r];
                const int grow = (tile0 + tt) * kTileRows + 4 * kg;
                const bool whole = (tile0 + tt + 1) * kTileRows <= n;
                const bool near =
                    __all(fmax(fmax(Y[0], Y[1]), fmax(Y[2], Y[3])) <= max_y && Y[0] == Y[0] &&
                          Y[1] == Y[1] && Y[2] == Y[2] && Y[3] == Y[3]);
                if (!(fine && near)) {
                    far |= 1ull << ((st - s0) * kDd64StageTiles + tt);
                    continue;
                }
                auto tile_exponents = [&](int i) {
                    f64x4 acc = {C[i] - Y[0], C[i] - Y[1], C[i] - Y[2], C[i] - Y[3]};
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1[i], acc, 0, 0, 0);
                    return __builtin_amdgcn_mfma_f64_16x16x4f64(a2, b2[i], acc, 0, 0, 0);
                };
                double e[4] = {0.0, 0.0, 0.0, 0.0};
                if (direct) {
                    // the next component's products are started before this one's
                    // exponentials; the fences keep the compiler from starting all K
                    f64x4 acc = tile_exponents(0);
#pragma unroll
                    for (int i = 0; i < K; ++i) {
                        f64x4 next = acc;
                        if (i + 1 < K) next = tile_exponents(i + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if (g.lw[i] != -INFINITY) {
                            const double wl = 1.0 + static_cast<double>(cl[i]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) e[r] = fma(exp2_fp64(acc[r]), wl, e[r]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        acc = next;
                    }
                    if (!whole) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) e[r] = grow + r < n ? e[r] : 1.0;
                    }
                    direct = __all(e[0] >= 0x1p-1000 && e[1] >= 0x1p-1000 && e[2] >= 0x1p-1000 &&
                                   e[3] >= 0x1p-1000);
                }
                if (!direct) {
                    // the empty asm keeps this path's K results, across its two passes,
                    // out of the direct path's registers
                    double m[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        m[r] = -INFINITY;
                        e[r] = 0.0;
                    }
#pragma unroll 1
                    for (int pass = 0; pass < 2; ++pass) {
                        asm volatile("" : "+v"(Y[0]), "+v"(Y[1]), "+v"(Y[2]), "+v"(Y[3]));
#pragma unroll
                        for (int i = 0; i < K; ++i) {
                            if (g.lw[i] == -INFINITY) continue;
                            const f64x4 acc = tile_exponents(i);
                            const double wl = 1.0 + static_cast<double>(cl[i]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                if (pass == 0) m[r] = fmax(m[r], acc[r]);
                                else e[r] = fma(exp2_fp64(fmax(acc[r] - m[r], -4000.0)), wl, e[r]);
                            }
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool in = grow + r < n;
                        msum += in ? m[r] : 0.0;
                        e[r] = in ? e[r] : 1.0;
                    }
                }
                // each factor may reach down to 2^-1000: renormalise after every one
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double q = prod * e[r];
                    expo += __builtin_amdgcn_frexp_exp(q);
                    prod = __builtin_amdgcn_frexp_mant(q);
                }
            }
            if (more) store_stage(buf ^ 1);
            __syncthreads();
        }
        // the tiles set aside: by differences, RB of a tile's rows of a lane at a time
        // (more spill beside their K exponents; k = 4: 694 us at 2, 708 at 4; k = 2:
        // 417 and 398), in natural units about each datum's largest exponent
        constexpr int RB = K > 2 ? 2 : 4;
        while (far != 0) {
            const int tile = t0 + s0 * kDd64StageTiles + __builtin_ctzll(far);
            far &= far - 1;
#pragma unroll 1
            for (int h = 0; h < 4; h += RB) {
                const int grow = tile * kTileRows + 4 * kg + h;
                int mq = mp;                         // as above: no means held between tiles
                asm volatile("" : "+v"(mq));
                double x[RB][kDdDim], a[RB][K], m[RB];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    m[r] = -INFINITY;
                    const float* yr = y + static_cast<size_t>(min(grow + r, n - 1)) * kDdDim;
#pragma unroll
                    for (int c = 0; c < kDdDim; ++c) x[r][c] = static_cast<double>(yr[c]);
                }
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    double q[RB];
#pragma unroll
                    for (int r = 0; r < RB; ++r) q[r] = 0.0;
#pragma unroll
                    for (int c = 0; c < kDdDim; ++c) {
                        const double mu = mean[i * kDdDim + c][mq];
#pragma unroll
                        for (int r = 0; r < RB; ++r) {
                            const double t = x[r][c] - mu;
                            q[r] = fma(t, t, q[r]);
                        }
                    }
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        a[r][i] = fma(-q[r], g.inv2s2, g.lw[i]);
                        m[r] = fmax(m[r], a[r][i]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    double e = 0.0;
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        e += exp2_fp64(fmax((a[r][i] - m[r]) * kLog2e, -4000.0));
                    const bool in = grow + r < n;
                    nsum += in ? m[r] : 0.0;
                    prod *= in ? e : 1.0;
                }
            }
            expo += __builtin_amdgcn_frexp_exp(prod);
            prod = __builtin_amdgcn_frexp_mant(prod);
        }
    }
    const double bits = msum + static_cast<double>(expo) + log2(prod);
    double v = nsum + fma(bits, kLn2, bits * kLn2Tail);
    // the differences' clamp passed over a NaN: a mean's, or that of a datum no
    // component has a finite exponent for
    bool nan = !(nsum > -INFINITY);
#pragma unroll 1
    for (int c = kg; c < K * kDdDim; c += 4) nan |= mean[c][mp] != mean[c][mp];
    if (nan) v = NAN;
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    if (kg == 0 && p < N) part[static_cast<size_t>(slice) * N + p] = v;
}

// Adds the slices' partial sums: bound by latency, so they are requested at once and
// a workgroup is one wave (k = 2, n = 1607, N = 4683: the whole call 22.1 -> 21.7 us).
template <int PREC>
__global__ void __launch_bounds__(kWave)
k_dd_finish(const double* part, int S, int N, int n, GmmDev g, double* out, int* status) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const double l = finish_loglik<PREC>(GroupSums(part, N, p, S).total(S), n, g);
    out[p] = l;
    if (l != l) atomicOr(status, kStatusNaN);
}

template <int K, int PREC>
__global__ void __launch_bounds__(256)
k_dd_accept(const double* part, int S, int N, int n, const double* theta_prop, double* theta,
            double* l,
            const double* __restrict__ beta_vec, StepSrc src, uint64_t seed, uint32_t move,
            GmmDev g, unsigned long long* n_acc, int* status, MoveStep ms) {
    constexpr int KD = K * kDdDim;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t step = static_cast<uint32_t>(step_index(src));
    if (ms.t_out != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        *ms.t_out = static_cast<int>(step);
    bool acc = false;
    if (p < N) {
        double tot = part[p];
        for (int s = 1; s < S; ++s) tot += part[static_cast<size_t>(s) * N + p];
        const double l_prop = finish_loglik<PREC>(tot, n, g);
        const MoveSource srcs = move_source(ms, theta, l);
        acc = rwmh_accept<KD>(
            p, p, N, [&](int c) { return theta_prop[static_cast<size_t>(c) * N + p]; }, l_prop,
            srcs, theta, l, beta_vec, src, step, seed, move, g, status, ms);
    }
    const unsigned long long mask = __ballot(acc);
    if (lane_id() == 0 && n_acc != nullptr && mask != 0ull)
        atomicAdd(n_acc, static_cast<unsigned long long>(__popcll(mask)));
}

double s2_of(const GmmDev& g) { return g.inv2s2 * kLog2e; }

}  // namespace

int64_t dd_padded_rows(int64_t n) { return ((n + kTileRows - 1) / kTileRows) * kTileRows; }

int dd_clamp_slices(int64_t n, int64_t S) {
    const int64_t tiles = dd_padded_rows(n) / kTileRows;
    if (S > 16) S = 16;
    if (S > tiles) S = tiles;
    if (S < 1) S = 1;
    return static_cast<int>(S);
}

int dd_slices(int64_t n, int64_t N) {
    const int64_t groups = (N + 63) / 64;
    return dd_clamp_slices(n, (2048 + groups - 1) / groups);
}

// Largest Y_j of a tile in the expansion over n data. A datum's exponent carries
// about ten roundings of 2^-53 Y; they average over the data, and the largest that
// leaves a log-likelihood's error at or below that of an exp per term and a log per
// datum was found against extended precision (k = 8, sigma2 = 1 and 0.3, means of
// spread 3, rms over particles, expansion and difference form against term by term,
// s2 in one part:
// n = 600 1.5 and 0.9 against 0.9e-16, n = 2000 1.2 and 0.9 against 1.6, sigma2 =
// 0.3 n = 2000 4.0 and 1.3 against 2.2, n = 20000 3.7 and 1.5 against 6.3).
double dd64_max_y(int64_t n) {
    const double m = std::min(static_cast<double>(n) / 16.0, 3.0 * std::sqrt(static_cast<double>(n)));
    return std::min(m, 4096.0);
}

bool dd64_takes(const GmmDev& g, int prec, int64_t n, int64_t N, bool move) {
    return prec == SMC_PREC_FP64 && dd_supported(g.k, g.d) && dd64_fits(g.k, N) &&
           dd64_pays(g.k, n, N, move);
}

int dd64_slices(int64_t n, int64_t N, int64_t want, int64_t part_cap) {
    const int64_t tiles = dd_padded_rows(n) / kTileRows;
    const int64_t groups = (N + 63) / 64;
    int64_t S = want > 0 ? want : (2048 + groups - 1) / groups;
    if (S > 16) S = 16;
    if (S > tiles) S = tiles;
    if (S * N > part_cap) S = part_cap / N;
    return static_cast<int>(S < 1 ? 1 : S);
}

bool dd_supported(int k, int d) { return d == kDdDim && (k == 1 || k == 2 || k == 4 || k == 8); }

hipError_t launch_dd_prep(const GmmDev& g, const float* y, int64_t n, __bf16* A, hipStream_t s) {
    const int64_t np = dd_padded_rows(n);
    hipLaunchKernelGGL(k_dd_prep, dim3(static_cast<unsigned>((np + 255) / 256)), dim3(256), 0, s, y,
                       static_cast<int>(n), static_cast<int>(np), s2_of(g), A);
    return hipGetLastError();
}

hipError_t launch_dd_loglik(const GmmDev& g, const __bf16* A, int64_t n, const double* theta,
                            int64_t N, __bf16* B, double* part, int S, double* out, int* status,
                            hipStream_t s) {
    const int64_t np = dd_padded_rows(n);
    const unsigned gb = static_cast<unsigned>((N * g.k + 255) / 256);
    hipLaunchKernelGGL((k_dd_build<false>), dim3(gb), dim3(256), 0, s, theta, static_cast<int>(N),
                       g.k, g, s2_of(g), MoveStep{}, 0.0, 0ull, StepSrc{}, 0u, B,
                       static_cast<double*>(nullptr));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>((N + 63) / 64), static_cast<unsigned>(S));
#define SMC_DD(KK)                                                                              \
    if (g.k == KK)                                                                              \
        hipLaunchKernelGGL((k_dd_partial<KK>), grid, dim3(kDdBlock), 0, s, A, static_cast<int>(n), \
                           static_cast<int>(np), B, static_cast<int>(N), S, g.unit_mass, part);
    SMC_DD(1) SMC_DD(2) SMC_DD(4) SMC_DD(8)
#undef SMC_DD
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dd_finish<SMC_PREC_FP32>,
                       dim3(static_cast<unsigned>((N + kWave - 1) / kWave)), dim3(kWave), 0, s,
                       part, S, static_cast<int>(N), static_cast<int>(n), g, out, status);
    return hipGetLastError();
}

hipError_t launch_dd_rwmh(const GmmDev& g, const __bf16* A, int64_t n, double* theta, double* l,
                          int64_t N, const double* beta_vec, StepSrc src, double sd,
                          uint64_t seed, uint32_t move, unsigned long long* n_accept,
                          __bf16* B, double* theta_prop, double* part, int S, int* status,
                          MoveStep ms, hipStream_t s) {
    const int64_t np = dd_padded_rows(n);
    const unsigned gb = static_cast<unsigned>((N * g.k + 255) / 256);
    hipLaunchKernelGGL((k_dd_build<true>), dim3(gb), dim3(256), 0, s, theta, static_cast<int>(N),
                       g.k, g, s2_of(g), ms, sd, seed, src, move, B, theta_prop);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>((N + 63) / 64), static_cast<unsigned>(S));
    const dim3 g1(static_cast<unsigned>((N + 255) / 256));
#define SMC_DD(KK)                                                                              \
    if (g.k == KK) {                                                                            \
        hipLaunchKernelGGL((k_dd_partial<KK>), grid, dim3(kDdBlock), 0, s, A, static_cast<int>(n), \
                           static_cast<int>(np), B, static_cast<int>(N), S, g.unit_mass, part);              \
        e = hipGetLastError();                                                                  \
        if (e != hipSuccess) return e;                                                          \
        hipLaunchKernelGGL((k_dd_accept<KK, SMC_PREC_FP32>), g1, dim3(256), 0, s, part, S,       \
                           static_cast<int>(N), static_cast<int>(n), theta_prop, theta, l,      \
                           beta_vec, src, seed, move, g, n_accept, status, ms);                 \
        return hipGetLastError();                                                               \
    }
    SMC_DD(1) SMC_DD(2) SMC_DD(4) SMC_DD(8)
#undef SMC_DD
    return hipErrorInvalidValue;
}

namespace {

hipError_t launch_dd64_partial(const GmmDev& g, const float* y, int64_t n, const double* theta,
                               int64_t N, double* part, int S, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>((N + 63) / 64), static_cast<unsigned>(S));
    const double s2 = s2_of(g);
    const double s2_lo = std::fma(g.inv2s2, kLog2e, -s2) + g.inv2s2 * kLog2eTail;
#define SMC_DD(KK)                                                                              \
    if (g.k == KK)                                                                              \
        hipLaunchKernelGGL((k_dd64_partial<KK>), grid, dim3(kDdBlock), 0, s, y,                  \
                           static_cast<int>(n), theta, static_cast<int>(N), g, s2, s2_lo,          \
                           dd64_max_y(n), S, part);
    SMC_DD(1) SMC_DD(2) SMC_DD(4) SMC_DD(8)
#undef SMC_DD
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dd64_loglik(const GmmDev& g, const float* y, int64_t n, const double* theta,
                              int64_t N, double* part, int S, double* out, int* status,
                              hipStream_t s) {
    const hipError_t e = launch_dd64_partial(g, y, n, theta, N, part, S, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dd_finish<SMC_PREC_FP64>,
                       dim3(static_cast<unsigned>((N + kWave - 1) / kWave)), dim3(kWave), 0, s,
                       static_cast<const double*>(part), S, static_cast<int>(N),
                       static_cast<int>(n), g, out, status);
    return hipGetLastError();
}

hipError_t launch_dd64_rwmh(const GmmDev& g, const float* y, int64_t n, double* theta, double* l,
                            int64_t N, const double* beta_vec, StepSrc src, double sd,
                            uint64_t seed, uint32_t move, unsigned long long* n_accept,
                            double* theta_prop, double* part, int S, int* status, MoveStep ms,
                            hipStream_t s) {
    const unsigned gb = static_cast<unsigned>((N * g.k + 255) / 256);
    hipLaunchKernelGGL((k_dd_build<true>), dim3(gb), dim3(256), 0, s, theta, static_cast<int>(N),
                       g.k, g, s2_of(g), ms, sd, seed, src, move, static_cast<__bf16*>(nullptr),
                       theta_prop);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_dd64_partial(g, y, n, theta_prop, N, part, S, s);
    if (e != hipSuccess) return e;
#define SMC_DD(KK)                                                                              \
    if (g.k == KK)                                                                              \
        hipLaunchKernelGGL((k_dd_accept<KK, SMC_PREC_FP64>),                                     \
                           dim3(static_cast<unsigned>((N + 255) / 256)), dim3(256), 0, s,        \
                           static_cast<const double*>(part), S,                                  \
                           static_cast<int>(N), static_cast<int>(n),                             \
                           static_cast<const double*>(theta_prop), theta, l, beta_vec, src,      \
                           seed, move, g, n_accept, status, ms);
    SMC_DD(1) SMC_DD(2) SMC_DD(4) SMC_DD(8)
#undef SMC_DD
    return hipGetLastError();
}

}  // namespace smc
