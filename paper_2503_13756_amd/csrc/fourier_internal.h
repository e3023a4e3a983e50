// Declarations of the Fourier-slice projector (k_fourier.hip) shared with
// the host code.
#pragma once
#include "sw_internal.h"

namespace sw {

// Fourier-slice projector (k_fourier.hip): L even with factors 2 and 3
// (lgL, lgNf: log2 of L and Nf for powers of two, else -1), oversampled
// grid Nf = 2L with the spectrum columns 0 .. L stored.  Tables (device,
// context-owned): corr[j] = 1 / phihat((j - L/2) / Nf) for the interpolation
// kernel phi, twf[k] = exp(-2 pi i k / Nf) (k < Nf), twl[k] =
// exp(-2 pi i k / L) (k < L), shift[t] = (-1)^k exp(i pi k / L) with
// k = t for t < L/2 and t - L otherwise.
//
// The slice points (theta_m, k pi), m < nsl, k <= L/2, npts of them, are
// ordered by the step that completes their kernel's support (one per round of
// columns, and above L = 64 one for column L and its mirrors), and
// inside a round for the LDS banks (host code); `targets` holds five float4
// of each, the q-th of all points from targets + q npts (layout at
// slice_points in k_fourier.hip), and the points of step k are
// steps[k] .. steps[k + 1] - 1.
constexpr int kFourierW = 7;  // interpolation kernel width in fine-grid points
struct FourierShape {
    int L, n, Nf, lgNf, lgL;
    int mirror;  // 1: slices theta_m = 2 pi m / n, m < n/2, plus their theta + pi
                 // mirrors; 0: n slices at explicit angles (the targets table)
};
struct FourierTabs {
    const float *corr;
    const float2 *twf, *twl, *shift;
    const float4 *targets;
    const int *steps;
};
// Columns (and row pairs) transformed per round: one radix-4 butterfly per
// thread of a block of fourier_threads; all columns at once up to L = 36, where
// the rounds' latencies are most of an image's time.
__host__ __device__ inline int fourier_group(int L) {
    return L <= 16 ? 16 : L <= 32 ? 32 : L <= 36 ? 64 : L <= 64 ? 16 : 8;
}
// The LDS ring of columns: column v is in slot (v + fourier_first) mod
// (2 fourier_group).  A single round's slots are those of columns -3 .. L + 3.
// From 16 columns a round on, the ring takes the columns past L - 1 together
// with the last round.
__host__ __device__ inline int fourier_first(int L) { return L <= 36 ? 3 : 0; }
__host__ __device__ inline int fourier_ring(int L) { return L <= 36 ? L + 7 : 2 * fourier_group(L); }
__host__ __device__ inline bool fourier_tail(int L) { return L > 64; }  // a step of its own
inline int fourier_threads(int L) { return L <= 128 ? 512 : 1024; }
__host__ __device__ inline int fourier_rounds(int L) {
    const int G = fourier_group(L);  // a power of two
    return (L + G - 1) >> __builtin_ctz((unsigned)G);
}
__host__ __device__ inline int fourier_slices(const FourierShape &S) {
    return S.mirror ? S.n / 2 : S.n;
}
// Scratch of one image (float2): the row transforms R [rounds][L][group], two
// copies of column L, flags, the slice values Y [slices][L/2 + 1].
constexpr int kFourierFlags = 32;
__host__ __device__ inline size_t fourier_slot_elems(const FourierShape &S) {
    return (size_t)fourier_rounds(S.L) * S.L * fourier_group(S.L) + 2 * S.Nf + kFourierFlags +
           (size_t)fourier_slices(S) * (S.L / 2 + 1);
}
// Row stride of a column (or row) of the oversampled grid in LDS: the first
// entries again behind the last, so that a kernel's support never wraps.
__host__ __device__ inline int fourier_stride(int Nf) { return Nf + 8; }
size_t fourier_slot_bytes(const FourierShape &S);
int fourier_blocks_per_cu(const FourierShape &S);  // resident blocks of the projector per CU
// The scratch holds `slots` regions of fourier_slot_bytes.  clear (nullable):
// [N], set to 0.  few: the phases of an image split over blocks.
hipError_t launch_fourier(const float *img, int64_t N, const FourierShape &S, const FourierTabs &T,
                          void *scratch, int slots, bool few, float *pmf, hipStream_t s,
                          unsigned *clear = nullptr);

}  // namespace sw
