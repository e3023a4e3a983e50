// Kernels and launchers of the angle spectra and the per-pair alignment;
// the device routines are in align_dev.h.
#include <algorithm>

#include "align_dev.h"
#include "wave_dev.h"

namespace sw {

// What the spectra of a table become: FP32 spectra (store_spectrum), packed
// bf16 complex spectra spec[w][j], or the coefficients of the register-FFT alignment of n = 128
// (gam, then gamx; see store_gamma128).
enum SpectrumOut { kSpecF32, kSpecBf16, kSpecGamma };

// Block (g, y) transforms the packed rows [y rows, (y + 1) rows) of table g,
// CH at a time.  The row split is what fills the device for few tables: one
// reference of n = Q = 128 went through one block in 40 us (149 us at 256,
// bound by the passes' latency, 255 compute units idle), and its coefficients
// through a second launch of 5 us; 1 vs 1,000 at L = 128 (bf16) 359 -> 325 us,
// 1 vs 1,500 at L = 256 3.56 -> 3.42 ms.
template <int NT, int OUT>
__global__ __launch_bounds__(NT) void k_spectrum(const float *__restrict__ qt, int64_t N, Geo g,
                                                 const float2 *__restrict__ tw32, void *out,
                                                 int rows, int CH, float2 *norms) {
    extern __shared__ __align__(16) float2 lds2[];
    const int64_t gi = blockIdx.x;
    if (gi >= N) return;
    const int P2 = g.Q / 2, Wn = g.n / 2 + 1, pbeg = (int)blockIdx.y * rows;
    const float *T = qt + gi * (int64_t)g.Q * g.n;
    const int pend = min(pbeg + rows, P2);
    if constexpr (OUT == kSpecGamma) {
        float2 *gam = (float2 *)out + gi * P2 * kA128Slots;
        float2 *gx = (float2 *)out + N * P2 * kA128Slots + gi * P2 * 2;
        spectrum_rows<NT, false>(T, g.n, pbeg, pend, CH, tw32, lds2,
                          [&](int p, int w, float2 xe, float2 xo) {
                              store_gamma128(gam, gx, p, w, xe, xo);
                          });
    } else if constexpr (OUT == kSpecBf16) {
        uint32_t *sp = (uint32_t *)out + gi * Wn * g.Q;
        float2 sq[kSpecNorms] = {};
        spectrum_rows<NT, true>(T, g.n, pbeg, pend, CH, tw32, lds2,
                          [&](int p, int w, float2 xe, float2 xo) {
                              const float2 e = bf16r2(xe), d = bf16r2(xo);
                              uint2 v;
                              v.x = (__float_as_uint(e.x) >> 16) |
                                    (__float_as_uint(e.y) & 0xffff0000u);
                              v.y = (__float_as_uint(d.x) >> 16) |
                                    (__float_as_uint(d.y) & 0xffff0000u);
                              *(uint2 *)(sp + (int64_t)w * g.Q + 2 * p) = v;
                              const float2 t = lds2[w];  // e^{-2 pi i w / n}
                              const float cw = w == 0 ? 0.f : w == Wn - 1 ? 1.f : 2.f;
                              const float ex = xe.x - e.x, ey = xe.y - e.y, dx = xo.x - d.x,
                                          dy = xo.y - d.y;
                              const float a =
                                  cw * (xe.x * xe.x + xe.y * xe.y + xo.x * xo.x + xo.y * xo.y);
                              const float b = cw * (ex * ex + ey * ey + dx * dx + dy * dy);
                              const float gw[kSpecNorms] = {
                                  2.f, __builtin_amdgcn_sqrtf(2.f - 2.f * t.x), 2.f * fabsf(t.y)};
#pragma unroll
                              for (int i = 0; i < kSpecNorms; ++i) {
                                  sq[i].x += gw[i] * a;
                                  sq[i].y += gw[i] * b;
                              }
                          });
        // this block's share of the squared norms (kSpecNorms)
        if (norms) {  // uniform
            __shared__ float2 ws[NT / 64][kSpecNorms];
#pragma unroll
            for (int i = 0; i < kSpecNorms; ++i) {
                const float2 sum = make_float2(wave_sum_f(sq[i].x), wave_sum_f(sq[i].y));
                if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6][i] = sum;
            }
            __syncthreads();
            if (threadIdx.x < kSpecNorms) {
                float2 v = ws[0][threadIdx.x];
                for (int w = 1; w < NT / 64; ++w) {
                    v.x += ws[w][threadIdx.x].x;
                    v.y += ws[w][threadIdx.x].y;
                }
                norms[(gi * gridDim.y + blockIdx.y) * kSpecNorms + threadIdx.x] = v;
            }
        }
    } else {
        float4 *sp = (float4 *)out + gi * Wn * P2;
        spectrum_rows<NT, false>(T, g.n, pbeg, pend, CH, tw32, lds2,
                          [&](int p, int w, float2 xe, float2 xo) {
                              store_spectrum(sp, Wn, p, w, xe, xo);
                          });
    }
}

// One block per image and run of `rg` references (all pairs), or per listed
// pair (rg = 1).
template <int NT, int RG>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(RG == 1 ? 6 : 5, 8))) void k_align_pairs(PairArgs a, Geo g, int rg,
                                                    const float2 *__restrict__ tw32,
                                                    const double2 *__restrict__ tw64) {
    extern __shared__ __align__(16) float2 lds2[];
    const int n = g.n, Q = g.Q, Wn = n / 2 + 1;
    const int64_t b = blockIdx.x;
    const int64_t r = a.pairs ? a.pairs[2 * b] : b / a.n_img * rg;
    const int64_t gi = a.pairs ? a.pairs[2 * b + 1] : b % a.n_img;
    const bool in_range = r >= 0 && r < a.n_ref && gi >= 0 && gi < a.n_img;
    const int64_t rr = in_range ? r : 0, gg = in_range ? gi : 0;
    const int64_t pi = a.pairs ? b : r * a.n_img + gi;
    PairsJob job;
    job.au = a.ref_aux + 4 * rr;
    job.av = a.img_aux + 4 * gg;
    job.U = a.ref_qt + rr * (int64_t)Q * n;
    job.V = a.img_qt + gg * (int64_t)Q * n;
    job.Uh = (const float4 *)a.ref_spec + rr * (int64_t)Wn * (Q / 2);
    job.res = a.out + pi;
    job.curve = a.curve ? a.curve + pi * n : nullptr;
    job.stride = a.n_img;
    job.nr = (int)min((int64_t)rg, a.n_ref - rr);
    job.status = in_range ? 0 : 3;
    align_pairs_block<NT, RG>(job, g, a.mode, a.bf16, a.top_k, tw32, tw64, lds2);
}

// Packed rows per block: one block per table, in chunks of kFftElems, when
// the tables alone fill the device twice over; fewer rows per block (down to
// one) for fewer tables, about kSpectrumBlocks blocks in all.
constexpr int kSpectrumBlocks = 512;

static int spectrum_rows_per_block(int64_t N, int P2) {
    const int64_t want = N < kSpectrumBlocks ? (kSpectrumBlocks + N - 1) / N : 1;
    return want >= P2 ? 1 : (int)((P2 + want - 1) / want);
}

int spectrum_blocks(int64_t N, Geo g) {
    const int rows = spectrum_rows_per_block(N, g.Q / 2);
    return (g.Q / 2 + rows - 1) / rows;
}

template <int OUT>
static hipError_t launch_spectrum_t(const float *qt, int64_t N, Geo g, const AngleTable &t,
                                    void *out, float2 *norms, hipStream_t s) {
    if (N <= 0) return hipSuccess;
    constexpr int NT = 256;
    const int rows = spectrum_rows_per_block(N, g.Q / 2);
    int CH = kFftElems / g.n;
    if (CH > rows) CH = rows;
    const size_t lds = sizeof(float2) * (size_t)(g.n + 2 * CH * g.n);
    hipLaunchKernelGGL((k_spectrum<NT, OUT>), dim3((unsigned)N, (unsigned)spectrum_blocks(N, g)),
                       dim3(NT), lds, s, qt, N, g, t.d32, out, rows, CH, norms);
    return hipGetLastError();
}

hipError_t launch_spectrum(const float *qt, int64_t N, Geo g, const AngleTable &t, void *spec,
                           int bf16, hipStream_t s, float2 *norms) {
    return bf16 ? launch_spectrum_t<kSpecBf16>(qt, N, g, t, spec, norms, s)
                : launch_spectrum_t<kSpecF32>(qt, N, g, t, spec, nullptr, s);
}

hipError_t launch_gamma128(const float *qt, int64_t N, Geo g, const AngleTable &t, float2 *gam,
                           hipStream_t s) {
    return launch_spectrum_t<kSpecGamma>(qt, N, g, t, gam, nullptr, s);
}

template <int RG>
static hipError_t launch_align_pairs_t(const PairArgs &a, Geo g, const AngleTable &t, int rg,
                                       int64_t blocks, hipStream_t s) {
    constexpr int NT = 256;
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)k_align_pairs<NT, RG>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
    (void)attr;
    hipLaunchKernelGGL((k_align_pairs<NT, RG>), dim3((unsigned)blocks), dim3(NT),
                       align_pairs_lds(g.n, RG), s, a, g, rg, t.d32, t.d64);
    return hipGetLastError();
}

// References per block: as many as eight, as long as that leaves kAlignBlocks
// blocks, four on every compute unit (fewer pairs are spread one by one).
// n = 512 has more spectral sums than a block of several references holds.
constexpr int64_t kAlignBlocks = 1024;

hipError_t launch_align_pairs(const PairArgs &a, Geo g, const AngleTable &t, hipStream_t s) {
    const int64_t P = a.pairs ? a.n_pairs : a.n_ref * a.n_img;
    if (P <= 0) return hipSuccess;
    int64_t rg = 1;
    if (!a.pairs && g.n < 512)
        rg = std::min({(int64_t)8, a.n_ref, std::max((int64_t)1, P / kAlignBlocks)});
    if (rg == 1) return launch_align_pairs_t<1>(a, g, t, 1, P, s);
    rg = (a.n_ref + (a.n_ref + rg - 1) / rg - 1) / ((a.n_ref + rg - 1) / rg);  // even runs
    return launch_align_pairs_t<8>(a, g, t, (int)rg, (a.n_ref + rg - 1) / rg * a.n_img, s);
}

}  // namespace sw
