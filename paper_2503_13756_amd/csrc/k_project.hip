// Kernel and launcher of the stand-alone line projection (images -> PMF
// tables); the device routines are in proj_dev.h.
#include "proj2_dev.h"
#include "proj_dev.h"

namespace sw {

__global__ __launch_bounds__(256) void k_plan_lanes(PlanLane *lanes, int count, int L) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const PlanLane p = lanes[i];
    float A3 = -100.f, A3n = -100.f;  // no item: clamps to the zero padding
    if (p.item >= 0) {
        const float c = p.A3, s = -p.A3n, r = s / c;
        const int b = p.item - p.slot * L;
        const double c0 = 0.5 * (double)(L - 1), ic = 1.0 / (double)c;
        const double a3 = ((double)b - c0 - 1.0) * ic + c0 + 3.0 - c0 * (double)r;
        A3 = (float)a3;
        A3n = (float)(a3 + (double)r);
    }
    lanes[i].A3 = A3;
    lanes[i].A3n = A3n;
}

hipError_t launch_plan_lanes(PlanLane *lanes, int count, int L, hipStream_t s) {
    hipLaunchKernelGGL(k_plan_lanes, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, lanes,
                       count, L);
    return hipGetLastError();
}

template <int NT, int TPW>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kProjMinWaves<NT, TPW>, NT <= 256 ? 2 : 4))) void k_project(const float *__restrict__ img, int64_t N,
                                                ProjShape P, const float2 *__restrict__ dtab,
                                                float *__restrict__ pmf) {
    extern __shared__ __align__(16) float lds[];
    const int64_t g = blockIdx.x;
    if (g >= N) return;
    const float *F = img + g * (int64_t)P.L * P.L;
    float *out = pmf + g * (int64_t)P.n * P.L;
    int bad = 0;
    // four-kind strips, the slot table after them (an opaque offset: a constant
    // one trips the compiler's LDS cast)
    int off = kStripFloats;
    asm volatile("" : "+s"(off));
    project_image4<NT, TPW>(F, P, dtab, lds, (float4 *)(lds + off), strip4_rows_max(P.L), bad,
                            [&](int k, int b, float v) { out[k * P.L + b] = v; });
    if (bad) {
        // an image with a non-finite value gets an all-NaN projection
        __syncthreads();
        for (int t = threadIdx.x; t < P.n * P.L; t += NT) out[t] = __int_as_float(0x7fc00000);
    }
}

// Two images per block (as the two-image tables kernel): both images'
// strips, IB bytes apart, share the weights and addresses of every (task,
// row); all tasks in one group.  With five or six tasks per wave the second
// image's accumulators wait in its own output (nL >= 4 TPW NT floats, which
// the launcher checks) while the first image's are written, so that the
// compiler keeps both sets in registers without spilling.  Bitwise the
// projections of k_project.
template <int NT, int TPW, int IB>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_project2(
    const float *__restrict__ img, int64_t N, ProjShape P, const float2 *__restrict__ dtab,
    float *__restrict__ pmf) {
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) float lds[];
    const int64_t g0 = 2 * (int64_t)blockIdx.x;
    if (g0 >= N) return;
    const int nimg = N - g0 >= 2 ? 2 : 1;
    const int L = P.L, n = P.n;
    const float *F[2] = {img + g0 * (int64_t)L * L, img + (g0 + nimg - 1) * (int64_t)L * L};
    // the slot table after both images' strips (an opaque offset, as above)
    int off = 2 * (IB / 4);
    asm volatile("" : "+s"(off));
    float acc[2][TPW][4];
    int bad[2];
    project_images2<NT, TPW, 2, 2, IB>(F, nimg, P, dtab, lds, (float4 *)(lds + off),
                                       s4_rows<NT>(L, IB), 0, acc, bad);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr bool kPark = TPW >= 5;
    float *park = pmf + (g0 + 1) * (int64_t)n * L + threadIdx.x;
    if (kPark && nimg == 2) {
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) park[(4 * t + v) * NT] = acc[1][t][v];
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if (g < nimg) {  // block-uniform
            if (kPark && g == 1) {
                asm volatile("" ::: "memory");
#pragma unroll
                for (int t = 0; t < TPW; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[1][t][v] = park[(4 * t + v) * NT];
                // every parked value is back in registers (the loads have
                // returned) before any thread's outputs overwrite the slots
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                __syncthreads();
            }
            float *out = pmf + (g0 + g) * (int64_t)n * L;
            if (!bad[g])
                emit_outputs<TPW>(P, 0, wave, NW, lane, acc[g],
                                  [&](int k, int b, float v) { out[k * L + b] = v; });
            else  // an image with a non-finite value gets an all-NaN projection
                for (int t = threadIdx.x; t < n * L; t += NT) out[t] = __int_as_float(0x7fc00000);
        }
    }
}

// Small batches: one block per (image, group of eight tasks, one task per
// wave), so that a single image spreads over several compute units.  Every
// block stages the whole image, in four-kind strips of R rows: what bounds a
// block is latency (the loads of a strip, its staging and the chain of a
// task's rows, with two waves per SIMD), so the block has as many threads to
// stage with as the strips allow, and few, tall strips.  One image (against
// 128-thread blocks of two tasks on 64 KiB of sliding windows): 18 -> 10 us at
// L = 64, 46 -> 19 at 128, 162 -> 43 at 256.  Bitwise the sums of the other
// kernels.
template <int NT, int KP>
__global__ __launch_bounds__(NT) void k_project_few(const float *__restrict__ img, int64_t N,
                                                    ProjShape P, const float2 *__restrict__ dtab,
                                                    float *__restrict__ pmf, int R,
                                                    int strip_floats, unsigned *clear) {
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) float lds[];
    const int64_t g = blockIdx.x;
    if (g >= N) return;
    const int L = P.L, n = P.n, tg0 = (int)blockIdx.y * NW;
    const float *const F[1] = {img + g * (int64_t)L * L};
    float *out = pmf + g * (int64_t)n * L;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (clear && blockIdx.y == 0 && threadIdx.x == 0) clear[g] = 0u;
    float acc[1][1][4];
    int bad[1];
    project_images2<NT, 1, 1, KP>(F, 1, P, dtab, lds, (float4 *)(lds + strip_floats), R, tg0, acc,
                                  bad);
    if (!bad[0])
        emit_outputs<1>(P, tg0, wave, NW, lane, acc[0],
                        [&](int k, int b, float v) { out[k * L + b] = v; });
    else if (blockIdx.y == 0)
        for (int t = threadIdx.x; t < n * L; t += NT) out[t] = __int_as_float(0x7fc00000);
}

// Geometries of more tasks than the kernels above hold at once (more than 72;
// L = n = 256 has 132): 1024 threads and 140 KiB of strips, one block per compute
// unit, in as many groups of tasks as it takes (each stages the images again).
// The accumulation is bound by the VALU: sharing the weights between two images
// takes it from 21.5 to 16.75 instructions per row and image, and the four-kind
// strips from four LDS reads per row to three.  1,500 images at L = n = 256 2.31
// -> 1.61 ms with two images of five tasks per wave against the one-image kernel
// on sliding windows (nine tasks per wave); all tasks in one group, with nine per
// wave, or eleven of 768 threads, spill: 1.64-1.87 ms.  One image per block, of
// nine tasks per wave, where every image has a compute unit of its own: 256
// images 498 us on sliding windows, 509 with two images on every second unit, 296
// so.  Bitwise the projections of k_project.
constexpr int kLargeStrips = 140 * 1024;

template <int NT, int TPW, int IMG>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_project_large(
    const float *__restrict__ img, int64_t N, ProjShape P, const float2 *__restrict__ dtab,
    float *__restrict__ pmf) {
    constexpr int IB = kLargeStrips / IMG, KP = 4 / IMG;
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) float lds[];
    const int64_t g0 = IMG * (int64_t)blockIdx.x;
    if (g0 >= N) return;
    const int nimg = N - g0 >= IMG ? IMG : 1;
    const int L = P.L, n = P.n;
    const float *F[IMG];
#pragma unroll
    for (int g = 0; g < IMG; ++g) F[g] = img + (g0 + min(g, nimg - 1)) * (int64_t)L * L;
    // the slot table after the strips (an opaque offset, as above)
    int off = kLargeStrips / 4;
    asm volatile("" : "+s"(off));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int tg0 = 0; tg0 < P.ntasks; tg0 += NW * TPW) {
        float acc[IMG][TPW][4];
        int bad[IMG];
        project_images2<NT, TPW, IMG, KP, IB>(F, nimg, P, dtab, lds, (float4 *)(lds + off),
                                              s4_rows<NT, KP>(L, IB), tg0, acc, bad);
#pragma unroll
        for (int g = 0; g < IMG; ++g) {
            if (g < nimg) {  // block-uniform
                float *out = pmf + (g0 + g) * (int64_t)n * L;
                if (!bad[g])
                    emit_outputs<TPW>(P, tg0, wave, NW, lane, acc[g],
                                      [&](int k, int b, float v) { out[k * L + b] = v; });
                else if (tg0 == 0)  // an image with a non-finite value: all NaN
                    for (int t = threadIdx.x; t < n * L; t += NT)
                        out[t] = __int_as_float(0x7fc00000);
            }
        }
    }
}

template <int NT, int TPW>
static hipError_t launch_project_t(const float *img, int64_t N, const ProjShape &P,
                                   const float2 *dtab, float *pmf, hipStream_t s) {
    const size_t lds = sizeof(float) * kStripFloats + sizeof(float4) * (P.slots + 1);
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_project<NT, TPW>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_project<NT, TPW>), dim3((unsigned)N), dim3(NT), lds, s, img, N, P, dtab,
                       pmf);
    return hipGetLastError();
}

template <int NT, int TPW>
static hipError_t launch_project2_t(const float *img, int64_t N, const ProjShape &P,
                                    const float2 *dtab, float *pmf, hipStream_t s) {
    constexpr int IB = kImg2BytesWide;
    const size_t lds = 2 * (size_t)IB + sizeof(float4) * (P.slots + 1);
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_project2<NT, TPW, IB>, hipFuncAttributeMaxDynamicSharedMemorySize,
        96 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_project2<NT, TPW, IB>), dim3((unsigned)((N + 1) / 2)), dim3(NT), lds, s,
                       img, N, P, dtab, pmf);
    return hipGetLastError();
}

// Strips of up to 140 KiB (one block per compute unit) while every block has
// a unit of its own, else of 64 KiB (two).  KP staging passes, the fewest that
// cover the strip's rows.
template <int NT, int KP>
static hipError_t launch_project_few_t(const float *img, int64_t N, const ProjShape &P, int R,
                                       const float2 *dtab, float *pmf, unsigned *clear,
                                       hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_project_few<NT, KP>, hipFuncAttributeMaxDynamicSharedMemorySize,
        152 * 1024);
    (void)attr;
    const int strip_floats = 4 * R * s4_positions(P.L);
    const size_t lds = sizeof(float) * strip_floats + sizeof(float4) * (P.slots + 1);
    const int groups = (P.ntasks + NT / 64 - 1) / (NT / 64);
    hipLaunchKernelGGL((k_project_few<NT, KP>), dim3((unsigned)N, (unsigned)groups), dim3(NT), lds,
                       s, img, N, P, dtab, pmf, R, strip_floats, clear);
    return hipGetLastError();
}

static int device_cus() {
    static const int cus = [] {
        int dev = 0, c = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
        return c > 0 ? c : 256;
    }();
    return cus;
}

static hipError_t launch_project_few(const float *img, int64_t N, const ProjShape &P,
                                     const float2 *dtab, float *pmf, unsigned *clear,
                                     hipStream_t s) {
    constexpr int NT = 512;
    const int groups = (P.ntasks + NT / 64 - 1) / (NT / 64);
    const int bytes = N * groups <= device_cus() ? 140 * 1024 : 64 * 1024;
    const int most = s4_rows<NT, 8>(P.L, bytes), strips = (P.L + most - 1) / most;
    const int R = (P.L + strips - 1) / strips;  // <= most: strips of nearly equal height
    if (s4_rows<NT, 2>(P.L, bytes) >= R)
        return launch_project_few_t<NT, 2>(img, N, P, R, dtab, pmf, clear, s);
    if (s4_rows<NT, 4>(P.L, bytes) >= R)
        return launch_project_few_t<NT, 4>(img, N, P, R, dtab, pmf, clear, s);
    return launch_project_few_t<NT, 8>(img, N, P, R, dtab, pmf, clear, s);
}

template <int NT, int TPW, int IMG>
static hipError_t launch_project_large(const float *img, int64_t N, const ProjShape &P,
                                       const float2 *dtab, float *pmf, hipStream_t s) {
    const size_t lds = (size_t)kLargeStrips + sizeof(float4) * (P.slots + 1);
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_project_large<NT, TPW, IMG>, hipFuncAttributeMaxDynamicSharedMemorySize,
        152 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_project_large<NT, TPW, IMG>), dim3((unsigned)((N + IMG - 1) / IMG)),
                       dim3(NT), lds, s, img, N, P, dtab, pmf);
    return hipGetLastError();
}

hipError_t launch_project(const float *img, int64_t N, Geo g, const AngleTable &t,
                          const ProjPlan &pp, float *pmf, hipStream_t s, bool split,
                          unsigned *clear) {
    if (N <= 0) return hipSuccess;
    ProjShape P = proj_shape(g.L, g.n);  // 64 KiB of strips: two blocks per CU
    if (pp.L != g.L || pp.n != g.n || pp.ntasks != P.ntasks) return hipErrorInvalidValue;
    P.perm = pp.perm;
    P.trow = pp.trow;
    if (split) return launch_project_few(img, N, P, t.d32, pmf, clear, s);
    const int w512 = tasks_per_wave(P.ntasks, 512);
    if (s4_supported(g.L)) {  // two images per block where all tasks fit one group of six
        const int64_t table = (int64_t)g.n * g.L;  // room to park the second image's sums
        if (w512 <= 2) return launch_project2_t<512, 2>(img, N, P, t.d32, pmf, s);
        if (w512 <= 4) return launch_project2_t<512, 4>(img, N, P, t.d32, pmf, s);
        if (w512 <= 5 && table >= 4 * 5 * 512)
            return launch_project2_t<512, 5>(img, N, P, t.d32, pmf, s);
        if (w512 <= 6 && table >= 4 * 6 * 512)
            return launch_project2_t<512, 6>(img, N, P, t.d32, pmf, s);
    }
    if (w512 <= 2) return launch_project_t<512, 2>(img, N, P, t.d32, pmf, s);
    if (w512 <= 4) return launch_project_t<512, 4>(img, N, P, t.d32, pmf, s);
    if (w512 <= 5) return launch_project_t<512, 5>(img, N, P, t.d32, pmf, s);
    if (w512 <= 6) return launch_project_t<512, 6>(img, N, P, t.d32, pmf, s);
    if (w512 <= 9) return launch_project_t<512, 9>(img, N, P, t.d32, pmf, s);
    if (N <= device_cus()) return launch_project_large<1024, 9, 1>(img, N, P, t.d32, pmf, s);
    return launch_project_large<1024, 5, 2>(img, N, P, t.d32, pmf, s);
}

}  // namespace sw
