// Ramp filter of 16 projection columns on the matrix cores (Sec. 2.2,
// optional high-pass step), shared by the stand-alone filter kernel and the
// fused ramp-filtered tables kernel.
//
// With the filter |xi| sampled on the M = 2L point frequency grid of the
// detector (DC term zero) and each column zero-padded to M, the filtered
// column is the cyclic convolution Pf[b] = sum_{b'} h[(b - b') mod M] P[b'],
// b, b' < L: the product of the L x L Toeplitz matrix H[b][b'] = h[b - b']
// with the columns.  h is zero at even offsets other than 0, so the even bins
// come from the odd ones and the odd bins from the even ones, half of the
// products each, plus h[0] times the bin itself.
//
// A wave takes 16 columns and keeps their values as the B fragments of
// v_mfma_f32_16x16x4_f32, even and odd bins apart (bins 2 (4 s + lane / 16) and
// the next one, column lane % 16); every 16-row tile of the even (odd) outputs
// accumulates the LP/8 K-steps with A fragments read from the kernel table,
// LP = L rounded up to 16 with zero padding.
#pragma once
#include "sw_internal.h"

namespace sw {

typedef float f32x4r __attribute__((ext_vector_type(4)));

// hs[t] = h[t - (LP - 1)] for |t - (LP - 1)| < L, 0 otherwise (2 LP - 1
// entries, LDS).  ld(j, b) reads bin b of the tile's column j (j < 16, zero
// past the last column), st(j, b, v) writes it; the bins are all read before
// the first write, and each once more before it is written, so the filter may
// run in place.
template <int NS, typename Ld, typename St>
__device__ __forceinline__ void ramp_tile(const float *hs, int L, Ld ld, St st) {
    constexpr int LP = 4 * NS, LH = LP / 2, KS = LH / 4, NB = (LH + 15) / 16;
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    float in[2][KS];  // even, odd
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int b = 2 * (4 * s + lk) + p;
            in[p][s] = b < L ? ld(li, b) : 0.f;
        }
    const float h0 = hs[LP - 1];
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        f32x4r acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        // row c = 16 t + li of the even (odd) outputs, a last half tile's rows
        // past LH repeating row LH - 1: A[c][k] = h[2 (c - 4 s - k) -+ 1]
        const int c = min(16 * t + li, LH - 1);
        const float *ha = hs + 2 * (c - lk) + LP - 1;
        __builtin_amdgcn_sched_barrier(0);  // a tile's operands are loaded in its own time
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(ha[2 * p - 1 - 8 * s], in[1 - p][s],
                                                              acc[p], 0, 0, 0);
        // this lane holds rows 16 t + 4 (lane / 16) + r of its column
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int b = 2 * (16 * t + 4 * lk + r) + p;
                if (b < L) st(li, b, fmaf(h0, ld(li, b), acc[p][r]));
            }
    }
}

}  // namespace sw
