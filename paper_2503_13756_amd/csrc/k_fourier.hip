// Fourier-slice projector (Sec. 2.2: the 1-D Fourier transform of the line
// projection at angle theta is the central slice of the image's 2-D Fourier
// transform; Sec. 2.3 computes the slices with a NUFFT and returns to the
// detector with a 1-D inverse DFT).  The discretisation is that of the
// appendix's fixed-angle error theorem with NUFFT precision: slice
// frequencies k pi, k = -M .. M-1 (L = 2M), and the trigonometric polynomial
// with coefficients yhat_k / 2 sampled at the detector bin centres.
//
// One block per image slot of a persistent grid (as many slots as fit on the
// CUs at once); per image:
//  1. rows: the pixel masses (positive part inside the disk, exactly as for
//     the line sum) divided by the kernel's Fourier transform at their
//     centred index, zero-padded to Nf = 2L and transformed along x; two
//     real rows share one complex FFT.  The half spectrum v <= L goes to the
//     slot's scratch (R), in the order the next phase reads it; columns 0 and
//     L are real and share one complex column.
//  2. columns, G at a time: the same transform along y into the LDS, where
//     the last 2 G columns of the oversampled spectrum stay; every slice
//     point k pi d_theta (theta in [0, pi), k = 0..M, or every given angle)
//     whose kW columns are then complete is interpolated from them with a
//     separable exponential-of-semicircle kernel of width kW, phase-shifted
//     to the pixel centres and multiplied by the transform of one pixel cell.
//  3. slices: the coefficients of two slices are packed into one complex
//     L-point inverse FFT (both results are real), scaled by h/2, clipped at
//     zero and written with their theta + pi mirror.
// The spectrum itself (258 KiB at L = 128) never leaves the LDS: written out
// and gathered from memory, one line an access and 49 a point, it took
// 1,775 us for 4,000 images at L = n = 128 (now 836).  What bounds it now is
// the transforms' steps, LDS access and index arithmetic in turn, at six waves
// per SIMD (two blocks of 512 threads instead of three: 920 us).
//
// The FFTs are Stockham transforms in LDS over a batch of sequences: for L a
// power of two radix 4 with one radix-2 step for odd powers, with shift and
// mask indexing; for other L (factors 2 and 3) the mixed-radix transforms of
// fft_dev.h, the inverse as conj(FFT(conj x)).  The first radix-4 step of the
// zero-padded transforms has two zero inputs of four and no twiddles: it is
// taken on the two loaded values, in registers.
#include <algorithm>

#include "fft_dev.h"
#include "fourier_internal.h"

namespace sw {

namespace {

int lg_exact(int x) {  // log2 of a power of two, else -1
    return x > 0 && (x & (x - 1)) == 0 ? __builtin_ctz((unsigned)x) : -1;
}

__device__ __forceinline__ bool in_disk_f(int L, int i, int j) {
    const int a = 2 * j - L + 1, b = 2 * i - L + 1, r = L - 2;
    return a * a + b * b <= r * r;
}

// One Stockham step of radix R over cnt transforms of length 2^lg (row stride
// rs): element j + r 2^lg / R of each transform, twiddled by
// exp(-+2 pi i r (j mod Ns) / (Ns R)), goes through an R-point DFT to position
// (j / Ns) Ns R + (j mod Ns) + r Ns of the output.  tw[k << lgt] is
// exp(-2 pi i k / 2^lg).
template <int NT, int R>
__device__ __forceinline__ void fft_step(const float2 *a, float2 *b, int lg, int rs, int lgNs,
                                         int cnt, const float2 *tw, int lgt, bool inv) {
    constexpr int lgR = R == 4 ? 2 : 1;
    const int nq = 1 << (lg - lgR), Ns = 1 << lgNs;
    for (int idx = threadIdx.x; idx < cnt * nq; idx += NT) {
        const int f = idx >> (lg - lgR), j = idx & (nq - 1);
        const float2 *src = a + __mul24(f, rs);
        float2 *dst = b + __mul24(f, rs);
        const int jm = j & (Ns - 1);
        const int o = ((j - jm) << lgR) + jm;
        // twiddle index of r = 1: jm N / (Ns R)
        const int t1 = jm << (lg - lgNs - lgR + lgt);
        float2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[r] = src[j + r * nq];
            if (r > 0) {
                float2 w = tw[r * t1];
                if (inv) w.y = -w.y;
                v[r] = cmul(v[r], w);
            }
        }
        if (R == 2) {
            dst[o] = make_float2(v[0].x + v[1].x, v[0].y + v[1].y);
            dst[o + Ns] = make_float2(v[0].x - v[1].x, v[0].y - v[1].y);
        } else {
            const float2 a0 = make_float2(v[0].x + v[2].x, v[0].y + v[2].y);
            const float2 a1 = make_float2(v[0].x - v[2].x, v[0].y - v[2].y);
            const float2 a2 = make_float2(v[1].x + v[3].x, v[1].y + v[3].y);
            // (v1 - v3) times -i (forward) or +i (inverse)
            const float2 d = make_float2(v[1].x - v[3].x, v[1].y - v[3].y);
            const float2 a3 = inv ? make_float2(-d.y, d.x) : make_float2(d.y, -d.x);
            dst[o] = make_float2(a0.x + a2.x, a0.y + a2.y);
            dst[o + Ns] = make_float2(a1.x + a3.x, a1.y + a3.y);
            dst[o + 2 * Ns] = make_float2(a0.x - a2.x, a0.y - a2.y);
            dst[o + 3 * Ns] = make_float2(a1.x - a3.x, a1.y - a3.y);
        }
    }
}

// cnt transforms of length 2^lg held at a + f rs; b is a work buffer of the
// same size.  The steps of the first 2^lgNs points have been taken already;
// the rest are of radix 4, one of radix 2 last when their number is odd.
// inv selects the conjugate twiddles (exp(+2 pi i ...)).  The input need not
// be visible to the block on entry; returns the buffer holding the (naturally
// ordered) result, visible to the whole block.
template <int NT>
__device__ float2 *fft_batch(float2 *a, float2 *b, int lg, int rs, int lgNs, int cnt,
                             const float2 *tw, int lgt, bool inv) {
    for (; lgNs + 2 <= lg; lgNs += 2) {
        __syncthreads();
        fft_step<NT, 4>(a, b, lg, rs, lgNs, cnt, tw, lgt, inv);
        float2 *x = a;
        a = b;
        b = x;
    }
    if (lgNs < lg) {
        __syncthreads();
        fft_step<NT, 2>(a, b, lg, rs, lgNs, cnt, tw, lgt, inv);
        float2 *x = a;
        a = b;
        b = x;
    }
    __syncthreads();
    return a;
}

// The first radix-4 step of a forward transform whose middle half is zero, on
// the inputs x (element j) and y (element j + 3 Nf / 4): outputs 4 j .. 4 j + 3.
__device__ __forceinline__ void first_step(float2 *dst, int j, float2 x, float2 y) {
    float4 *d = (float4 *)(dst + 4 * j);
    d[0] = make_float4(x.x + y.x, x.y + y.y, x.x - y.y, x.y + y.x);
    d[1] = make_float4(x.x - y.x, x.y - y.y, x.x + y.y, x.y - y.x);
}

// Slice value yhat at a point of the table whose columns are in the ring (column
// v in slot v mod RC, row stride CS).  A point's entry
// (host-built per geometry, float4 x 5): (first row u0, slot of its first
// column | conj << 16) as ints and the complex factor (pixel-centre phase times
// the cell transform); the kW x-weights and the point's index in Y; the kW
// y-weights.  With conj the kernel was evaluated at the mirrored point and the
// sum is conjugated.
struct Point {
    float4 e[5];
};
__device__ __forceinline__ Point load_point(const float4 *__restrict__ T, int npts, int i) {
    return Point{{T[i], T[npts + i], T[2 * npts + i], T[3 * npts + i], T[4 * npts + i]}};
}
__device__ __forceinline__ void slice_point(const float2 *ring, int CS, int RC, const Point &p,
                                            float2 *__restrict__ Y) {
    const float4 e0 = p.e[0], e1 = p.e[1], e2 = p.e[2], e3 = p.e[3], e4 = p.e[4];
    const int vw = __float_as_int(e0.y);
    const float wx[kFourierW] = {e1.x, e1.y, e1.z, e1.w, e2.x, e2.y, e2.z};
    const float wy[kFourierW] = {e3.x, e3.y, e3.z, e3.w, e4.x, e4.y, e4.z};
    int s = vw & 0xffff;
    const float2 *row = ring + __float_as_int(e0.x);
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int c = 0; c < kFourierW; ++c) {
        const float2 *col = row + __mul24(s, CS);
        float2 ra = make_float2(0.f, 0.f);
#pragma unroll
        for (int a = 0; a < kFourierW; ++a) {
            const float2 bv = col[a];
            ra.x = fmaf(wy[a], bv.x, ra.x);
            ra.y = fmaf(wy[a], bv.y, ra.y);
        }
        acc.x = fmaf(wx[c], ra.x, acc.x);
        acc.y = fmaf(wx[c], ra.y, acc.y);
        s = (s + 1) & (RC - 1);
    }
    if (vw >> 16) acc.y = -acc.y;
    Y[__float_as_int(e2.w)] = cmul(acc, make_float2(e0.z, e0.w));
}

// Multiples and quotients by a transform length: shifts for powers of two,
// else float products with inv = 1 / n (div_small) where the registers allow it
// (FLOAT): at six waves per SIMD they add to the spills, 80 images at L = 96 54 ->
// 59 us.
template <bool POW2, bool FLOAT>
struct Len {
    int n, lg;
    float inv;
    __device__ __forceinline__ int mul(int x) const {
        if constexpr (POW2) return x << lg;
        else return x * n;
    }
    __device__ __forceinline__ int div(int x) const {
        if constexpr (POW2) return x >> lg;
        else if constexpr (FLOAT) return div_small(x, inv);
        else return x / n;
    }
};

// phases: bit 0 rows, 1 columns and points, 2 slices.  blockIdx.y of gridDim.y
// takes its share of the phase's rounds; all three phases at once go with
// gridDim.y = 1.  row_parts: gridDim.y of the launch that took the rows.
constexpr int kRows = 1, kColumns = 2, kSlices = 4;

//
// OWN: the slot is in LDS.
template <int NT, bool POW2, bool OWN>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 512 && !OWN ? 6 : 4, 6))) void k_fourier(
    const float *__restrict__ img, int64_t N, FourierShape S, FourierTabs T, int phases,
    int row_parts, float2 *__restrict__ scratch, float *__restrict__ pmf, unsigned *clear) {
    extern __shared__ __align__(16) float2 lds2[];
    const int L = S.L, M = L >> 1, n = S.n, Nf = S.Nf, lgNf = S.lgNf, lgL = S.lgL;
    const int G = fourier_group(L), lgG = 31 - __builtin_clz(G), RC = 2 * G, CS = fourier_stride(Nf);
    // with an own slot all phases come at once, in a single round
    if constexpr (OWN) phases = kRows | kColumns | kSlices, row_parts = 1;
    const int rounds = OWN ? 1 : fourier_rounds(L), nsl = fourier_slices(S), npts = nsl * (M + 1);
    const float h = 2.f / (float)L;
    const int tid = threadIdx.x, part = OWN ? 0 : blockIdx.y, parts = OWN ? 1 : gridDim.y;
    float2 *ring = lds2, *temp = ring + fourier_ring(L) * CS;  // [slots][CS], [G or L][CS]
    float2 *twf = temp + min(G, L) * CS;                       // [Nf]
    float2 *cols = ring + fourier_first(L) * CS;               // column 0, the first round's output
    float2 *twl = twf + Nf;                       // [L], L not a power of two
    for (int t = tid; t < Nf; t += NT) twf[t] = T.twf[t];
    if constexpr (!POW2)
        for (int t = tid; t < L; t += NT) twl[t] = T.twl[t];
    float2 *R;  // [rounds][L][G]
    const float2 *shift = T.shift;  // [L], in LDS before an own slot
    if constexpr (OWN) {
        float2 *sh = POW2 ? twl : twl + L;
        for (int t = tid; t < L; t += NT) sh[t] = T.shift[t];
        shift = sh;
        R = sh + L;
    } else {
        R = scratch + (size_t)blockIdx.x * fourier_slot_elems(S);
    }
    float2 *CL = R + (size_t)rounds * L * G;  // [2][Nf] column L
    int *flags = (int *)(CL + 2 * Nf);
    float2 *Y = CL + 2 * Nf + kFourierFlags;  // [nsl][M + 1]
    const Len<POW2, OWN> LM{M, lgL - 1, __builtin_amdgcn_rcpf((float)M)};
    const Len<POW2, OWN> LL{L, lgL, __builtin_amdgcn_rcpf((float)L)};
    // this block's share of `count` rounds or pairs
    auto share = [&](int count, int &from, int &to) {
        from = count * part / parts;
        to = count * (part + 1) / parts;
    };
    // the transforms of length Nf of cnt rows after their first step; that
    // step's output goes to fft_in(target), the result is in target
    const int later = POW2 ? (lgNf - 1) >> 1 : fft_passes(Nf / 4);
    auto fft_in = [&](float2 *target) { return later & 1 ? temp : target; };
    auto fft = [&](float2 *target, int cnt) {
        float2 *a = later & 1 ? temp : target, *b = later & 1 ? target : temp;
        if constexpr (POW2) {
            fft_batch<NT>(a, b, lgNf, CS, 2, cnt, twf, 0, false);
        } else {
            __syncthreads();
            fft_rows<NT>(a, b, cnt, Nf, CS, 4, twf);
        }
    };
    for (int64_t g = blockIdx.x; g < N; g += gridDim.x) {
        __syncthreads();  // previous image done with the buffers and the scratch
        if (phases & kRows) {
            const float *F = img + g * (int64_t)L * L;
            if (clear && tid == 0 && part == 0) clear[g] = 0u;
            // row pair rp0 + f, columns j and j + M
            const int f = LM.div(tid), j = tid - LM.mul(f);
            const int rr = OWN ? 1 : (M + G - 1) >> lgG;
            int k0, k1;
            share(rr, k0, k1);
            const float cl = f < G ? T.corr[j] : 0.f, cr = f < G ? T.corr[j + M] : 0.f;
            int bad = 0;
            float x[4];
            auto fetch = [&](int k) {
                const int i = 2 * (k * G + f);
                if (f < G && i < L) {
                    const float *p = F + (int64_t)i * L + j;
                    x[0] = p[0];
                    x[1] = p[M];
                    x[2] = p[L];
                    x[3] = p[L + M];
                }
            };
            auto mass = [&](float v, int i, int jj, float c) {
                if (!isfinite(v)) bad = 1;
                return (in_disk_f(L, i, jj) && v > 0.f) ? v * c : 0.f;
            };
            fetch(k0);
            for (int k = k0; k < k1; ++k) {
                const int i = 2 * (k * G + f);
                if (f < G && i < L) {
                    const float c0 = T.corr[i], c1 = T.corr[i + 1];
                    const float2 lo = make_float2(mass(x[0], i, j, c0 * cl), mass(x[2], i + 1, j, c1 * cl));
                    const float2 hi = make_float2(mass(x[1], i, j + M, c0 * cr),
                                                  mass(x[3], i + 1, j + M, c1 * cr));
                    // element q of the padded row is column (q + M) mod Nf
                    first_step(fft_in(cols) + __mul24(f, CS), j, hi, lo);
                }
                if (k + 1 < k1) fetch(k + 1);
                const int cnt = min(G, M - k * G);
                fft(cols, cnt);
                // Z = X_i + i X_{i+1}: X_i[v] = (Z[v] + conj Z[-v]) / 2,
                // X_{i+1}[v] = (Z[v] - conj Z[-v]) / (2 i)
                for (int idx = tid; idx < LL.mul(cnt); idx += NT) {
                    const int ff = LL.div(idx), v = idx - LL.mul(ff);
                    const float2 *Z = cols + __mul24(ff, CS);
                    const float2 zv = Z[v], zc = Z[v == 0 ? L : Nf - v];
                    float2 *r = R + (((v >> lgG) * L + 2 * (k * G + ff)) << lgG) + (v & (G - 1));
                    // v = 0: the real X[0] and X[L] as one complex value
                    r[0] = v == 0 ? make_float2(zv.x, zc.x)
                                  : make_float2(0.5f * (zv.x + zc.x), 0.5f * (zv.y - zc.y));
                    r[G] = v == 0 ? make_float2(zv.y, zc.y)
                                  : make_float2(0.5f * (zv.y + zc.y), -0.5f * (zv.x - zc.x));
                }
                __syncthreads();
            }
            const int any = __syncthreads_or(bad);
            if (tid == 0) flags[part] = any;
            __syncthreads();
        }
        if (phases & kColumns) {
            int k0, k1;
            share(rounds, k0, k1);
            const bool tail = k1 == rounds;  // this block also takes the points at column L
            // column f of the round, rows j and j + M
            const int f = tid & (G - 1), j = tid >> lgG;
            float2 lo, hi;
            auto fetch = [&](int k) {
                const float2 *p = R + (size_t)k * L * G + tid;
                if (j < M) {
                    lo = p[0];
                    hi = p[M << lgG];
                }
            };
            // entry u of a column mirrored from entry `from(u)` of another
            auto from = [&](int u) { return u == 0 || u == Nf ? 0 : u < Nf ? Nf - u : 2 * Nf - u; };
            auto slot = [&](int v) {
                return ring + __mul24((v + fourier_first(L)) & (RC - 1), CS);
            };
            const bool after = !OWN && fourier_tail(L);
            const int ka = max(k0 - 1, 0), end = k1 + (tail && after ? 1 : 0);
            // round 0 first where the copy of column L is needed and it is not
            // one of this block's (which then keeps a copy of its own)
            bool pre = tail && ka > 0;
            float2 *kept = pre ? CL + Nf : CL;
            int k = pre ? 0 : ka;
            fetch(k);
            Point first{};
            if constexpr (OWN)
                if (tid < npts) first = load_point(T.targets, npts, tid);
            while (k < end) {
                const int next = pre ? ka : k + 1;
                if (k < rounds) {  // columns k G .. of the spectrum into the ring
                    float2 *dst = cols + (k & 1) * G * CS;
                    const int cnt = min(G, L - k * G);
                    if (j < M && f < cnt) first_step(fft_in(dst) + __mul24(f, CS), j, hi, lo);
                    // (fewer threads than the round's butterflies: L = 36, own slots)
                    for (int jj = j + (NT >> lgG); jj < M; jj += NT >> lgG)
                        if (f < cnt) {
                            const float2 *p = R + (size_t)k * L * G + (jj << lgG) + f;
                            first_step(fft_in(dst) + __mul24(f, CS), jj, p[M << lgG], p[0]);
                        }
                    if (next < k1) fetch(next);
                    fft(dst, cnt);
                    for (int idx = tid; idx < cnt * 8; idx += NT) {
                        const int ff = idx >> 3, u = idx & 7;
                        if (k > 0 || ff > 0) dst[__mul24(ff, CS) + Nf + u] = dst[__mul24(ff, CS) + u];
                    }
                    if (k == 0) {
                        const bool only = rounds == 1;  // column L straight into the ring
                        float2 *sl = slot(L);
                        // Z = B[.][0] + i B[.][L], both Hermitian
                        for (int u = tid; u <= L; u += NT) {
                            const int um = u == 0 ? 0 : Nf - u;
                            const float2 z = dst[u], zc = dst[um];
                            const float2 b0 = make_float2(0.5f * (z.x + zc.x), 0.5f * (z.y - zc.y));
                            const float2 bl = make_float2(0.5f * (z.y + zc.y), -0.5f * (z.x - zc.x));
                            const float2 b0c = make_float2(b0.x, -b0.y), blc = make_float2(bl.x, -bl.y);
                            dst[um] = b0c;
                            dst[u] = b0;
                            if (u < 8) dst[Nf + u] = b0;
                            if (only) {
                                sl[um] = blc;
                                sl[u] = bl;
                                if (u < 8) sl[Nf + u] = bl;
                            } else {
                                kept[um] = blc;
                                kept[u] = bl;
                            }
                        }
                        // columns -1 .. -3: B[u][-v] = conj B[-u][v]
                        for (int v = 1; v <= 3; ++v)
                            for (int u = tid; u < Nf + 8; u += NT) {
                                const float2 z = slot(v)[from(u)];
                                slot(-v)[u] = make_float2(z.x, -z.y);
                            }
                    }
                }
                if (k == (after ? rounds : rounds - 1)) {
                    // column L, and L + 1 .. L + 3: B[u][L + v] = conj B[-u][L - v]
                    if (k > 0)
                        for (int u = tid; u < Nf + 8; u += NT) slot(L)[u] = kept[u < Nf ? u : u - Nf];
                    for (int v = 1; v <= 3; ++v)
                        for (int u = tid; u < Nf + 8; u += NT) {
                            const float2 z = slot(L - v)[from(u)];
                            slot(L + v)[u] = make_float2(z.x, -z.y);
                        }
                }
                __syncthreads();
                if constexpr (OWN) {  // one round: every point
                    if (tid < npts) slice_point(ring, CS, RC, first, Y);
                    for (int i = tid + NT; i < npts; i += NT)
                        slice_point(ring, CS, RC, load_point(T.targets, npts, i), Y);
                } else if (k >= k0 && !pre) {
                    const int i1 = T.steps[k + 1];
                    for (int i = T.steps[k] + tid; i < i1; i += NT)
                        slice_point(ring, CS, RC, load_point(T.targets, npts, i), Y);
                }
                __syncthreads();
                pre = false;
                k = next;
            }
        }
        if (phases & kSlices) {
            int isbad = 0;
            for (int i = 0; i < row_parts; ++i) isbad |= flags[i];
            float *out = pmf + g * (int64_t)n * L;
            // slices m < nsl, two per inverse transform: nsl = n/2 with their
            // theta + pi mirrors, or all n (slices at explicit angles)
            const int pairs = nsl >> 1;  // n is a multiple of 8
            int p0, p1;
            share(pairs, p0, p1);
            // two work buffers of `most` transforms of length L = Nf / 2
            const int most = 2 * min(G, L);
            float2 *fa = ring, *fb = ring + most * L;
            for (int pb = p0; pb < p1; pb += most) {
                const int cnt = min(most, p1 - pb);
                for (int idx = tid; idx < LL.mul(cnt); idx += NT) {
                    const int f = LL.div(idx), t = idx - LL.mul(f);
                    const int k = t < M ? t : t - L;
                    const float2 *Y1 = Y + (2 * (pb + f)) * (M + 1), *Y2 = Y1 + (M + 1);
                    float2 c1 = k >= 0 ? Y1[k] : Y1[-k], c2 = k >= 0 ? Y2[k] : Y2[-k];
                    if (k < 0) {  // the coefficients of a real projection are Hermitian
                        c1.y = -c1.y;
                        c2.y = -c2.y;
                    }
                    const float2 sh = shift[t];
                    float2 z1 = cmul(c1, sh), z2 = cmul(c2, sh);
                    if (k == 0 || k == -M) {  // self-paired frequencies: real part
                        z1.y = 0.f;
                        z2.y = 0.f;
                    }
                    float2 zz = make_float2(z1.x - z2.y, z1.y + z2.x);  // z1 + i z2
                    if constexpr (!POW2) zz.y = -zz.y;  // inverse as conj(FFT(conj))
                    fa[idx] = zz;
                }
                const float2 *X;
                if constexpr (POW2) {
                    X = fft_batch<NT>(fa, fb, lgL, L, 0, cnt, twf, 1, true);
                } else {
                    __syncthreads();
                    X = fft_rows<NT>(fa, fb, cnt, L, twl);
                }
                for (int idx = tid; idx < LL.mul(cnt); idx += NT) {
                    const int f = LL.div(idx), b = idx - LL.mul(f);
                    float2 z = X[idx];
                    if constexpr (!POW2) z.y = -z.y;
                    const int m1 = 2 * (pb + f), m2 = m1 + 1;
                    const float qnan = __int_as_float(0x7fc00000);
                    const float q1 = isbad ? qnan : fmaxf(0.5f * h * z.x, 0.f);
                    const float q2 = isbad ? qnan : fmaxf(0.5f * h * z.y, 0.f);
                    out[(int64_t)m1 * L + b] = q1;
                    out[(int64_t)m2 * L + b] = q2;
                    if (S.mirror) {
                        out[(int64_t)(m1 + (n >> 1)) * L + (L - 1 - b)] = q1;
                        out[(int64_t)(m2 + (n >> 1)) * L + (L - 1 - b)] = q2;
                    }
                }
                __syncthreads();  // the work buffers are rewritten next round
            }
        }
    }
}

}  // namespace

static size_t fourier_work_bytes(int L) {
    const int Nf = 2 * L;
    return sizeof(float2) *
           (size_t)((fourier_ring(L) + std::min(fourier_group(L), L)) * fourier_stride(Nf) + Nf +
                    (lg_exact(L) < 0 ? L : 0));
}

size_t fourier_slot_bytes(const FourierShape &S) { return sizeof(float2) * fourier_slot_elems(S); }

// Images of a single round (L <= 36) keep their slot in LDS as well, as long as
// two blocks fit a compute unit: their time is the phases' round trips.
static bool fourier_own(const FourierShape &S) {
    return fourier_rounds(S.L) == 1 &&
           fourier_work_bytes(S.L) + fourier_slot_bytes(S) <= 79 * 1024;
}

static size_t fourier_lds_bytes(const FourierShape &S) {
    return fourier_work_bytes(S.L) +
           (fourier_own(S) ? sizeof(float2) * S.L + fourier_slot_bytes(S) : 0);
}

using FourierKernel = decltype(&k_fourier<512, true, false>);

// Threads of a block.  With an own slot as few as take the rows' first butterflies
// (M^2) at once and the points in two turns: the rest only wait at the barriers,
// and with fewer waves a block more images are in flight.  5,000 images at L = 8
// 53 us with the spectrum in scratch and 512 threads, 63 with it in LDS, 20 with
// 128 threads; at L = 16 68, 70 and 25.
static int fourier_nt(const FourierShape &S) {
    if (!fourier_own(S)) return fourier_threads(S.L);
    const int M = S.L / 2, npts = fourier_slices(S) * (M + 1);
    int nt = 128;
    while (nt < 512 && (nt < M * M || 2 * nt < npts)) nt *= 2;
    return nt;
}

static FourierKernel fourier_kernel(const FourierShape &S) {
    static const FourierKernel ks[10] = {
        k_fourier<512, false, false>, k_fourier<512, true, false>, k_fourier<1024, false, false>,
        k_fourier<1024, true, false>, k_fourier<128, false, true>, k_fourier<128, true, true>,
        k_fourier<256, false, true>,  k_fourier<256, true, true>,  k_fourier<512, false, true>,
        k_fourier<512, true, true>};
    static const hipError_t attr = [] {
        for (FourierKernel k : ks)
            (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      128 * 1024);
        return hipSuccess;
    }();
    (void)attr;
    const int p2 = lg_exact(S.L) >= 0 ? 1 : 0;
    const int nt = fourier_nt(S);
    return ks[p2 + (fourier_own(S) ? nt == 128 ? 4 : nt == 256 ? 6 : 8 : nt == 1024 ? 2 : 0)];
}

int fourier_blocks_per_cu(const FourierShape &S) {
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &nb, (const void *)fourier_kernel(S), fourier_nt(S), fourier_lds_bytes(S));
    return e == hipSuccess && nb > 0 ? nb : 1;
}

hipError_t launch_fourier(const float *img, int64_t N, const FourierShape &S, const FourierTabs &T,
                          void *scratch, int slots, bool few, float *pmf, hipStream_t s,
                          unsigned *clear) {
    if (N <= 0) return hipSuccess;
    const int L = S.L, NT = fourier_nt(S);
    const size_t lds = fourier_lds_bytes(S);
    const FourierKernel k = fourier_kernel(S);
    float2 *scr = (float2 *)scratch;
    if (!few || fourier_own(S)) {
        const int grid = (int)(N < slots ? N : slots);
        hipLaunchKernelGGL(k, dim3(grid), dim3(NT), lds, s, img, N, S, T,
                           kRows | kColumns | kSlices, 1, scr, pmf, clear);
        return hipGetLastError();
    }
    // one launch per phase: a block per round of rows, of columns and (about
    // four butterflies a thread) of slices
    const int rows = (L / 2 + fourier_group(L) - 1) / fourier_group(L);
    const int pairs = fourier_slices(S) / 2;
    const int sl = std::max(1, std::min(pairs, pairs * L / (4 * NT)));
    for (int64_t i0 = 0; i0 < N; i0 += slots) {
        const int64_t m = std::min<int64_t>(N - i0, slots);
        const float *im = img + i0 * (int64_t)L * L;
        float *out = pmf + i0 * (int64_t)S.n * L;
        unsigned *cl = clear ? clear + i0 : nullptr;
        hipLaunchKernelGGL(k, dim3((unsigned)m, rows), dim3(NT), lds, s, im, m, S, T, kRows, rows,
                           scr, out, cl);
        hipLaunchKernelGGL(k, dim3((unsigned)m, fourier_rounds(L)), dim3(NT), lds, s, im, m, S, T,
                           kColumns, rows, scr, out, cl);
        hipLaunchKernelGGL(k, dim3((unsigned)m, sl), dim3(NT), lds, s, im, m, S, T, kSlices, rows,
                           scr, out, cl);
    }
    return hipGetLastError();
}

}  // namespace sw
