// Complex multiply and batched Stockham FFTs in LDS with radix 4, 3 and 2
// (lengths 2^a 3^b), shared by the per-pair alignment (angle FFTs) and the
// Fourier-slice projector (lengths that are not powers of two).
#pragma once
#include "sw_internal.h"

namespace sw {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

template <int R>
__device__ __forceinline__ void dft_small(float2 (&a)[R]) {
    if constexpr (R == 2) {
        const float2 x = a[0], y = a[1];
        a[0] = make_float2(x.x + y.x, x.y + y.y);
        a[1] = make_float2(x.x - y.x, x.y - y.y);
    } else if constexpr (R == 4) {
        const float2 t0 = make_float2(a[0].x + a[2].x, a[0].y + a[2].y);
        const float2 t1 = make_float2(a[0].x - a[2].x, a[0].y - a[2].y);
        const float2 t2 = make_float2(a[1].x + a[3].x, a[1].y + a[3].y);
        const float2 t3 = make_float2(a[1].x - a[3].x, a[1].y - a[3].y);
        a[0] = make_float2(t0.x + t2.x, t0.y + t2.y);
        a[2] = make_float2(t0.x - t2.x, t0.y - t2.y);
        a[1] = make_float2(t1.x + t3.y, t1.y - t3.x);  // t1 - i t3
        a[3] = make_float2(t1.x - t3.y, t1.y + t3.x);  // t1 + i t3
    } else {  // R == 3, w = e^{-2 pi i / 3}
        const float h3 = 0.86602540378443864676f;
        const float2 s = make_float2(a[1].x + a[2].x, a[1].y + a[2].y);
        const float2 d = make_float2(a[1].x - a[2].x, a[1].y - a[2].y);
        const float2 m = make_float2(a[0].x - 0.5f * s.x, a[0].y - 0.5f * s.y);
        a[0] = make_float2(a[0].x + s.x, a[0].y + s.y);
        a[1] = make_float2(m.x + h3 * d.y, m.y - h3 * d.x);
        a[2] = make_float2(m.x - h3 * d.y, m.y + h3 * d.x);
    }
}

// Quotient of small non-negative integers by d, given inv = 1 / d: the float
// product is within q 2^-22 of (x + 1/2) / d, which lies at least 1 / (2 d) from
// an integer, so the truncation is exact while x < 2^21.
__device__ __forceinline__ int div_small(int x, float inv) {
    return (int)(((float)x + 0.5f) * inv);
}
// The same of wave-uniform x and d, as a scalar: an integer division of two
// scalars is some twenty vector instructions.
__device__ __forceinline__ int div_uniform(int x, int d) {
    return __builtin_amdgcn_readfirstlane(div_small(x, __builtin_amdgcn_rcpf((float)d)));
}

// One Stockham pass of radix R over `rows` complex rows of length n, from X
// to Y (row stride rs).  p = product of the radices already applied, ts = n /
// (p R).  The indices are quotients by n / R and by p, which integer division
// would make most of the pass's instructions.
template <int NT, int R>
__device__ __forceinline__ void fft_pass(const float2 *X, float2 *Y, int rows, int n, int rs,
                                         int p, int ts, const float2 *tw) {
    const int nr = n / R;
    const int nb = rows * nr;
    const float inr = __builtin_amdgcn_rcpf((float)nr), ip = __builtin_amdgcn_rcpf((float)p);
    for (int idx = threadIdx.x; idx < nb; idx += NT) {
        const int row = div_small(idx, inr), i = idx - __mul24(row, nr);
        const int k = i - __mul24(div_small(i, ip), p);
        const float2 *x = X + __mul24(row, rs) + i;
        float2 v[R];
        int m = 0;  // q k ts
        const int dm = __mul24(k, ts);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            v[q] = x[q * nr];
            if (q > 0) v[q] = cmul(v[q], tw[m]);
            m += dm;
        }
        dft_small<R>(v);
        float2 *y = Y + __mul24(row, rs) + __mul24(i - k, R) + k;
#pragma unroll
        for (int q = 0; q < R; ++q) y[q * p] = v[q];
    }
    __syncthreads();
}

// Forward FFT of `rows` rows (row stride rs) held in A; B is a buffer of the
// same size.  The radices of product p have been applied already.  Returns the
// buffer holding the result.
template <int NT>
__device__ float2 *fft_rows(float2 *A, float2 *B, int rows, int n, int rs, int p,
                            const float2 *tw) {
    int m = n / p;  // p is 1 or 4 where it is called
    float2 *x = A, *y = B;
    while (m % 4 == 0) {
        m /= 4;
        fft_pass<NT, 4>(x, y, rows, n, rs, p, m, tw);
        p *= 4;
        float2 *t = x; x = y; y = t;
    }
    while (m % 3 == 0) {
        m /= 3;
        fft_pass<NT, 3>(x, y, rows, n, rs, p, m, tw);
        p *= 3;
        float2 *t = x; x = y; y = t;
    }
    while (m % 2 == 0) {
        m /= 2;
        fft_pass<NT, 2>(x, y, rows, n, rs, p, m, tw);
        p *= 2;
        float2 *t = x; x = y; y = t;
    }
    return x;
}
template <int NT>
__device__ float2 *fft_rows(float2 *A, float2 *B, int rows, int n, const float2 *tw) {
    return fft_rows<NT>(A, B, rows, n, n, 1, tw);
}

// Passes that fft_rows takes for length n, the radices of product p left out
// (n / p here).
__host__ __device__ inline int fft_passes(int n) {
    int c = 0;
    for (; n % 4 == 0; n /= 4) ++c;
    for (; n % 3 == 0; n /= 3) ++c;
    for (; n % 2 == 0; n /= 2) ++c;
    return c;
}

}  // namespace sw
