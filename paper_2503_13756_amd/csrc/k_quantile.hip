// Kernel and launcher of the stand-alone CDF/quantile stage (PMF tables ->
// quantile tables); the device routines are in quant_dev.h.
#include "quant_dev.h"

namespace sw {

template <int NT>
__global__ __launch_bounds__(NT) void k_quantile(const float *__restrict__ pmf, int64_t N,
                                                 QuantShape<NT> S,
                                                 const double2 *__restrict__ d64,
                                                 float *__restrict__ qt, double *__restrict__ aux) {
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) double ldsd[];  // 16-byte aligned: ds_read_b128 on strips
    const int64_t g = blockIdx.x;
    if (g >= N) return;
    const int L = S.L, n = S.n, Q = S.Q;
    double *colS = ldsd;
    float *Ut = (float *)(colS + 2 * n);
    const float *P = pmf + g * (int64_t)n * L;
    quantile_phase<NT>([&](int k, int b) { return P[(int64_t)k * L + b]; }, L, n, Q, S.levels, S.TC,
                       d64, Ut, colS, qt + g * (int64_t)Q * n, aux ? aux + 4 * g : nullptr);
}

// Ramp-filtered projections (signed) -> stacked quantile tables: rows 0..Q-1
// invert the positive part max(Pf, 0) of every column, rows Q..2Q-1 the
// negative part max(-Pf, 0), each normalised on its own (ramp-filtered SW of
// Sec. 2.3 and its appendix).  aux = { smallest part mass over the columns
// (NaN if a value is NaN), E of the stacked table, a of the stacked table =
// the mean of the two parts' moments }.
template <int NT, int QM>
__global__ __launch_bounds__(NT) void k_quantile_rf(const float *__restrict__ pf, int64_t N,
                                                    QuantShape<NT> S,
                                                    const double2 *__restrict__ d64,
                                                    float *__restrict__ qt,
                                                    double *__restrict__ aux) {
    extern __shared__ __align__(16) double ldsd[];
    const int64_t g = blockIdx.x;
    if (g >= N) return;
    const int L = S.L, n = S.n, Q = S.Q;
    double *colS = ldsd;
    float *Ut = (float *)(colS + 2 * n);
    const float *P = pf + g * (int64_t)n * L;
    quantile_phase_rf<NT, QM>([&](int k, int b) { return P[(int64_t)k * L + b]; }, L, n, Q, S.levels,
                          S.TC, d64, Ut, colS, qt + g * (int64_t)2 * Q * n,
                          aux ? aux + 4 * g : nullptr);
}

// Small batches: a block per (image, eight columns[, signed part]) instead of
// one per image, so that all columns are inverted at once: a column is a chain
// of FP64 scans and interpolations of about 4 us, and one block of 16 waves
// went through the columns of one image in turn.  The column sums (and the
// masses the image's aux needs) go to scratch, and the image's last block to
// finish reduces them in the order of quantile_phase: the same bits whichever
// block that is.  One image: 7.8 -> 5.7 us at L = n = Q = 64, 22 -> 7.6 at
// 128, 82 -> 9.0 at 256, the two signed parts at 128 55 -> 12.
//
// done[g] counts the finished blocks of image g; 0 before the launch (the
// projectors clear it).  The sums are stored and read as device-scope atomics,
// past the caches that the dies do not share, and a block counts once its
// stores are acknowledged.  That a store so acknowledged is seen by every die's
// later device-scope load is a property of this hardware (write-through at
// device scope, and a wait that covers stores), not of the memory model, which
// would ask for release and acquire.  (With plain stores and a device-scope fence a block,
// the fences' cache write-backs took 35 ns a block one after the other: 200
// images at L = n = 64 55 us, now 8.)
constexpr int kColsPerBlock = 8;

__device__ __forceinline__ void publish(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double published(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int NT, bool RF>
__global__ __launch_bounds__(NT) void k_quantile_cols(const float *__restrict__ pmf, int L, int n,
                                                      int Q, int levels,
                                                      const double2 *__restrict__ d64,
                                                      float *__restrict__ qt,
                                                      double *__restrict__ aux, double *colS,
                                                      double *colM, unsigned *done) {
    constexpr int TC = kColsPerBlock;
    extern __shared__ __align__(16) float Ut[];  // [Q][TC + 1]
    __shared__ double cs[2 * TC], cm[TC];
    __shared__ int last, nan;
    const int64_t g = blockIdx.x;
    const int k0 = TC * (int)blockIdx.y, part = RF ? (int)blockIdx.z : 0;
    constexpr int parts = RF ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float sign = part ? -1.f : 1.f;
    const float *P = pmf + g * (int64_t)n * L;
    if (RF) {
        if (threadIdx.x == 0) nan = 0;
        __syncthreads();
    }
    auto col = [&](int k, int b) {
        const float v = P[(int64_t)k * L + b];
        if (RF && v != v) nan = 1;  // every such lane writes the same
        return RF ? fmaxf(sign * v, 0.f) : v;
    };
    auto on_mass = [&](int k, double m) { cm[k - k0] = m; };  // the same on its lanes
    // cs holds the columns k0 .. k0 + TC - 1 of quantile_phase's colS
    if (L <= 128) invert_tile<NT, true>(col, L, Q, levels, TC, k0, Ut, cs - 2 * k0, on_mass);
    else invert_tile<NT, false>(col, L, Q, levels, TC, k0, Ut, cs - 2 * k0, on_mass);
    __syncthreads();
    // wave 0: the sums, and the masses of the columns (or of the parts).  A part's
    // mass is NaN for a NaN value, and infinite where the scan made a NaN of an
    // infinite one (an overflowed filter), which the smallest mass leaves out as
    // the fmin of quantile_phase_rf does.
    static_assert(2 * TC <= 64, "one wave publishes a block's sums");
    if (threadIdx.x < 2 * TC)
        publish(colS + ((g * parts + part) * n + k0) * 2 + threadIdx.x, cs[threadIdx.x]);
    if (threadIdx.x < TC)
        publish(colM + (g * parts + part) * n + k0 + threadIdx.x,
                !RF   ? cm[threadIdx.x]
                : nan ? __longlong_as_double(0x7ff8000000000000LL)
                      : fmin(cm[threadIdx.x], INFINITY));
    if (wave == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores have arrived
        if (lane == 0)
            last = __hip_atomic_fetch_add(done + g, 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) == gridDim.y * parts - 1;
    }
    write_tile<NT>(Ut, Q, TC, n, qt + (g * parts + part) * (int64_t)Q * n + k0);
    __syncthreads();
    if (!last || wave != 0 || !aux) return;
    // every block of the image has counted, its sums have arrived
    double sums[parts][3];
#pragma unroll
    for (int h = 0; h < parts; ++h)
        column_aux([&](int i) { return published(colS + (g * parts + h) * 2 * n + i); }, n, Q, d64,
                   lane, sums[h]);
    double *A = aux + 4 * g;
    if (!RF) {
        if (lane == 0) {
            A[0] = published(colM + g * n);
            A[1] = sums[0][0];
            A[2] = sums[0][1];
            A[3] = sums[0][2];
        }
        return;
    }
    double mn = INFINITY;
    int bad = 0;
    for (int k = lane; k < 2 * n; k += 64) {
        const double m = published(colM + g * 2 * n + k);
        if (m != m) bad = 1;
        else mn = fmin(mn, m);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mn = fmin(mn, __shfl_xor(mn, off, 64));
    bad = __any(bad);
    if (lane == 0) {
        A[0] = bad ? __longlong_as_double(0x7ff8000000000000LL) : mn;
        A[1] = sums[0][0] + sums[parts - 1][0];
        A[2] = 0.5 * (sums[0][1] + sums[parts - 1][1]);
        A[3] = 0.5 * (sums[0][2] + sums[parts - 1][2]);
    }
}

size_t quantile_cols_bytes(int64_t N, int n, int parts) {
    return sizeof(double) * (size_t)N * (n * 3 * parts + 1);
}

unsigned *quantile_cols_done(void *cols) { return (unsigned *)cols; }

template <bool RF>
static hipError_t launch_quantile_cols(const float *pmf, int64_t N, Geo g, const AngleTable &t,
                                       float *qt, double *aux, double *cols, hipStream_t s) {
    constexpr int parts = RF ? 2 : 1;
    // a double's room for each image's counter, then the sums, then the masses
    unsigned *done = quantile_cols_done(cols);
    double *colS = cols + N, *colM = colS + (size_t)N * g.n * 2 * parts;
    const dim3 grid((unsigned)N, (unsigned)(g.n / kColsPerBlock), parts);  // n: a multiple of 8
    const size_t lds = sizeof(float) * g.Q * (kColsPerBlock + 1);
    if (g.L <= 128)  // two columns per wave: four waves take a block's eight at once
        hipLaunchKernelGGL((k_quantile_cols<256, RF>), grid, dim3(256), lds, s, pmf, g.L, g.n, g.Q,
                           g.levels, t.d64, qt, aux, colS, colM, done);
    else
        hipLaunchKernelGGL((k_quantile_cols<512, RF>), grid, dim3(512), lds, s, pmf, g.L, g.n, g.Q,
                           g.levels, t.d64, qt, aux, colS, colM, done);
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_quantiles_t(const float *pmf, int64_t N, Geo g, const AngleTable &t,
                                     float *qt, double *aux, hipStream_t s) {
    QuantShape<NT> S{g.L, g.n, g.Q, g.levels, pick_tc(g.n, g.Q, 68 * 1024)};
    const size_t lds = sizeof(double) * 2 * g.n + sizeof(float) * g.Q * (S.TC + 1);
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_quantile<NT>, hipFuncAttributeMaxDynamicSharedMemorySize, 120 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_quantile<NT>), dim3((unsigned)N), dim3(NT), lds, s, pmf, N, S, t.d64, qt,
                       aux);
    return hipGetLastError();
}

// Small batches take many blocks per image where the caller has scratch for
// the column sums, else 16 waves per image; the results do not depend on it.
hipError_t launch_quantiles(const float *pmf, int64_t N, Geo g, const AngleTable &t, float *qt,
                            double *aux, hipStream_t s, bool small, double *cols) {
    if (N <= 0) return hipSuccess;
    if (small && cols) return launch_quantile_cols<false>(pmf, N, g, t, qt, aux, cols, s);
    if (small) return launch_quantiles_t<1024>(pmf, N, g, t, qt, aux, s);
    return launch_quantiles_t<256>(pmf, N, g, t, qt, aux, s);
}


template <int NT, int QM>
static hipError_t launch_quantiles_rf_t(const float *pf, int64_t N, Geo g, const AngleTable &t,
                                        float *qt, double *aux, hipStream_t s) {
    QuantShape<NT> S{g.L, g.n, g.Q, g.levels, pick_tc(g.n, g.Q, 68 * 1024)};
    const size_t lds = sizeof(double) * 2 * g.n + sizeof(float) * g.Q * (S.TC + 1);
    static const hipError_t attr = hipFuncSetAttribute((const void *)k_quantile_rf<NT, QM>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       120 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_quantile_rf<NT, QM>), dim3((unsigned)N), dim3(NT), lds, s, pf, N, S,
                       t.d64, qt, aux);
    return hipGetLastError();
}

hipError_t launch_quantiles_rf(const float *pf, int64_t N, Geo g, const AngleTable &t, float *qt,
                               double *aux, hipStream_t s, bool small, double *cols) {
    if (N <= 0) return hipSuccess;
    if (small && cols) return launch_quantile_cols<true>(pf, N, g, t, qt, aux, cols, s);
    const bool half = quant_mode_for(g.L) == kQuantHalf;
    if (small)
        return half ? launch_quantiles_rf_t<1024, kQuantHalf>(pf, N, g, t, qt, aux, s)
                    : launch_quantiles_rf_t<1024, kQuantWave>(pf, N, g, t, qt, aux, s);
    return half ? launch_quantiles_rf_t<256, kQuantHalf>(pf, N, g, t, qt, aux, s)
                : launch_quantiles_rf_t<256, kQuantWave>(pf, N, g, t, qt, aux, s);
}

}  // namespace sw
