// Angle spectra and pairwise alignment of quantile tables.
//
// Sec. 2.3 (fast computation over rotations): a rotation of the image is a
// cyclic shift of the columns of its quantile table, and the cross term
// sum_{j,k} U[j][k] V[j][k+l] of the squared distance is, for every lag l at
// once, a cross-correlation along the angle axis, done by FFT row by row and
// summed over rows.  Summing over rows before the inverse transform leaves one
// length-n inverse transform per pair:
//   S(w) = sum_j conj(U^_j(w)) V^_j(w),
//   C(l) = (1/n) sum_w S(w) e^{2 pi i w l / n}.
// The translation at every lag is the least-squares shift of the quantile
// functions, which by the translation equivariance of SW2 (Thm 3.2 and its
// proof) reduces to the first angular moment of the column means:
//   b(l) = a_U - e^{i theta_l} a_V,  s*(l) = 2 b(l),  D*(l) = D0(l) - 2|b(l)|^2.
//
// FFTs: two real table rows are packed into one complex row and transformed
// by a Stockham FFT in LDS (radix 4, 3, 2, ping-pong between two buffers;
// twiddles from the angle table, which equals e^{-2 pi i m / n}); the two
// real spectra are separated from the packed one by conjugate symmetry.
#pragma once
#include <type_traits>
#include "fft_dev.h"
#include "wave_dev.h"

namespace sw {

// Complex elements of one LDS FFT chunk (8 KiB, two buffers).  The per-pair
// alignment is latency bound: small chunks keep its LDS near 22 KiB at
// n = 256, so that seven blocks fit on a compute unit instead of two.
constexpr int kFftElems = 1024;

// bfloat16 round-to-nearest-even of two floats, returned as floats: one
// v_cvt_pk_bf16_f32 for the pair (round to nearest even; equal to the bit
// formula u + 0x7fff + ((u >> 16) & 1), truncated, on every non-NaN float),
// then the halves shifted back
__device__ __forceinline__ float2 bf16r2(float2 v) {
    const __bf16 a = (__bf16)v.x, b = (__bf16)v.y;
    return make_float2((float)a, (float)b);
}

// Load complex rows p0 .. p0+rows-1 of a [Q][n] real table: row p packs table
// rows 2p (real part) and 2p+1 (imaginary part).
template <int NT>
__device__ __forceinline__ void load_packed(float2 *Z, const float *__restrict__ T, int n, int p0,
                                            int rows) {
    const float inv = __builtin_amdgcn_rcpf((float)n);
    const float *T0 = T + (int64_t)(2 * p0) * n;
    for (int idx = threadIdx.x; idx < rows * n; idx += NT) {
        const float *t = T0 + idx + __mul24(div_small(idx, inv), n);
        Z[idx] = make_float2(t[0], t[n]);
    }
}

// Separate the spectra of the two real rows packed in Z row pl at frequency w.
__device__ __forceinline__ void unpack(const float2 *Z, int pl, int n, int w, float2 &xe,
                                       float2 &xo) {
    const float2 zw = Z[pl * n + w];
    const float2 zc = Z[pl * n + (w == 0 ? 0 : n - w)];
    // xe = (zw + conj(zc)) / 2 ; xo = (zw - conj(zc)) / (2i)
    xe = make_float2(0.5f * (zw.x + zc.x), 0.5f * (zw.y - zc.y));
    const float dx = zw.x - zc.x, dy = zw.y + zc.y;
    xo = make_float2(0.5f * dy, -0.5f * dx);
}

__device__ __forceinline__ int fft_chunk_rows(int n, int Q) {
    const int c = div_uniform(kFftElems, n);
    return c < Q / 2 ? c : Q / 2;
}

// -------------------------------------------------------------- alignment
// b(l) = a_U - e^{i theta_l} a_V
__device__ __forceinline__ double2 trans_moment(const double *au, const double *av, double2 d) {
    const double c = d.x, s = -d.y;
    return make_double2(au[2] - (c * av[2] - s * av[3]), au[3] - (s * av[2] + c * av[3]));
}

// Angle spectra of the packed rows [pbeg, pend) of one [Q][n] table, at most
// CH of them at a time: emit(p, w, xe, xo) gets the spectra of table rows 2p
// and 2p + 1 at every w in [0, n/2], neighbouring threads neighbouring w (or,
// with ROWS, neighbouring p).  Each packed row is transformed on its own, so
// its spectra do not depend on the split.  lds: n + 2 CH n float2.
template <int NT, bool ROWS, typename Emit>
__device__ void spectrum_rows(const float *__restrict__ T, int n, int pbeg, int pend, int CH,
                              const float2 *__restrict__ tw32, float2 *lds2, Emit emit) {
    const int Wn = n / 2 + 1;
    float2 *tw = lds2;
    float2 *Z0 = lds2 + n;
    float2 *Z1 = Z0 + CH * n;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += NT) tw[i] = tw32[i];
    for (int p0 = pbeg; p0 < pend; p0 += CH) {
        const int rows = min(CH, pend - p0);
        __syncthreads();
        load_packed<NT>(Z0, T, n, p0, rows);
        __syncthreads();
        const float2 *Z = fft_rows<NT>(Z0, Z1, rows, n, tw);
        const int len = ROWS ? rows : Wn;
        const float inv = __builtin_amdgcn_rcpf((float)len);
        for (int idx = threadIdx.x; idx < rows * Wn; idx += NT) {
            const int q = div_small(idx, inv), o = idx - __mul24(q, len);
            const int w = ROWS ? q : o, pl = ROWS ? o : q;
            float2 xe, xo;
            unpack(Z, pl, n, w, xe, xo);
            emit(p0 + pl, w, xe, xo);
        }
    }
    __syncthreads();
}

// FP32 spectra of a table as the alignment reads them: spec[p][w], w <= n/2,
// the spectra of rows 2p and 2p + 1 side by side (a float4), so that
// neighbouring frequencies are neighbours in memory.
__device__ __forceinline__ void store_spectrum(float4 *spec, int Wn, int p, int w, float2 xe,
                                               float2 xo) {
    spec[(int64_t)p * Wn + w] = make_float4(xe.x, xe.y, xo.x, xo.y);
}

// The register-FFT alignment's coefficients (align128_dev.h) of packed row p
// at frequency w of an n = 128 table: alpha(w) = (conj xe - i conj xo) / 2 and
// beta(w) = (conj xe + i conj xo) / 2, laid out in that kernel's lane order.
// Frequency f (alpha at f < 64, beta of 128 - f from 64 on) sits in slot
// 16 lp + 8 tau + s with f = 2 lp + tau + 16 s; beta(0) and alpha(64) in gx.
constexpr int kA128Slots = 128;  // coefficients per packed row (8 lanes x 16)
__device__ __forceinline__ void store_gamma128(float2 *gam, float2 *gx, int p, int w, float2 xe,
                                               float2 xo) {
    const float2 alpha = make_float2(0.5f * (xe.x - xo.y), -0.5f * (xe.y + xo.x));
    const float2 beta = make_float2(0.5f * (xe.x + xo.y), 0.5f * (xo.x - xe.y));
    float2 *row = gam + p * kA128Slots;
    auto slot = [](int f) { return ((f & 14) << 3) | ((f & 1) << 3) | (f >> 4); };
    if (w < 64) row[slot(w)] = alpha;
    else gx[2 * p + 1] = alpha;
    if (w > 0) row[slot(128 - w)] = beta;
    else gx[2 * p] = beta;
}

// Alignment of one image table V with `nr` <= RG reference tables by one
// block: spectra of V (once for all references), spectral dots with the
// references' spectra, inverse transform over the lags, translation
// correction, top-k, FP32 rescore; writes the result of every pair (and its
// curve).  A pair's arithmetic does not depend on RG or nr.
//
// What bounds it is the issue of vector instructions: index arithmetic (no
// integer divisions here), the transforms and the rescore.  Sharing the image's
// transforms between references takes the transforms, two thirds of a pair's
// work at n = 64, out of all but one of them.  16 x 2,000 pairs at L = n = Q = 64
// 517 -> 128 us; one reference against 1,500 images at 256 508 -> 300 us, against
// 1,031 at L = 39 22 -> 15 us.
struct PairsJob {
    const float *U, *V;    // [nr][Q][n] and [Q][n] tables
    const double *au, *av; // aux of both, [nr][4] and [4]
    const float4 *Uh;      // [nr][Q/2][Wn] FP32 spectra of U (store_spectrum)
    Result *res;           // the pair of reference r: res[r stride], curve + r stride n
    float *curve;          // nullable
    int64_t stride;
    int nr;
    int status;            // 3: bad pair index (nr is 1; nothing is read)
};

constexpr int kAlignSlots = 4;  // candidates rescored at a time (eight spill registers)

// LDS of align_pairs_block: the angle table, then the two FFT buffers, the
// spectral sums and D* of every reference; the rescore has rows of the image
// table in all of it behind the angle table, at least 20 rows up to n = 256.
__host__ __device__ inline int align_work_floats(int n, int RG) {
    const int work = 4 * kFftElems + 2 * RG * (n / 2 + 2) + 2 * RG * n;
    const int rows = n <= 64 ? 4352 : n <= 256 ? 20 * n : 12 * n;
    return work > rows ? work : rows;
}
__host__ __device__ inline size_t align_pairs_lds(int n, int RG) {
    return sizeof(float2) * (size_t)n + sizeof(float) * (size_t)align_work_floats(n, RG);
}

template <int NT, int RG>
__device__ void align_pairs_block(const PairsJob &job, Geo g, int mode, int bf16, int top_k,
                                  const float2 *__restrict__ tw32,
                                  const double2 *__restrict__ tw64, float2 *lds2) {
    constexpr int NW = NT / 64;
    constexpr int IT = RG == 1 ? 2 : 1;  // spectral sums per thread (n = 512: 257 of them)
    __shared__ int lagS[RG * kMaxTopK];
    __shared__ float2 shiftS[RG * kMaxTopK];
    __shared__ float valS[RG * kMaxTopK];
    // the waves' sums of a batch of candidates, batches taking turns: a batch's
    // one barrier lies between its writes and wave 0's reads, and the next
    // batch's barrier between those reads and the next writes to the same set
    __shared__ float red[2][NW][kAlignSlots];
    const int n = g.n, Q = g.Q, Wn = n / 2 + 1, half = n / 2, K = top_k;
    // an opaque copy of the thread index: in a persistent caller, what is
    // derived from it is formed per job instead of being kept live across jobs
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nr = RG == 1 ? 1 : job.nr;
    float2 *tw = lds2;
    float2 *Z0 = tw + n;
    float2 *Z1 = Z0 + kFftElems;
    float2 *S = Z1 + kFftElems;                      // [RG][Wn + 1]
    double *D = (double *)(S + RG * (n / 2 + 2));    // [RG][n]
    auto fail = [&](int r, int status) {
        Result *res = job.res + r * job.stride;
        if (tid == 0) {
            res->rot_index = 0;
            res->theta_rad = 0.f;
            res->shift_px[0] = res->shift_px[1] = 0.f;
            res->sw2sq = __int_as_float(0x7fc00000);
            res->status = status;
        }
        if (job.curve)
            for (int l = tid; l < n; l += NT)
                job.curve[r * job.stride * n + l] = __int_as_float(0x7fc00000);
    };
    __syncthreads();  // the previous job of this block may still read LDS
    if (job.status) {
        fail(0, job.status);
        return;
    }
    const double *av = job.av;
    auto status_of = [&](int r) {  // uniform
        const double *au = job.au + 4 * r;
        if (isnan(au[0]) || isnan(av[0])) return 2;
        return !(au[0] > 0.0) || !(av[0] > 0.0) ? 1 : 0;
    };
    int live = 0;  // references whose pair is computed
    for (int r = 0; r < nr; ++r) {
        const int st = status_of(r);
        if (st) fail(r, st);
        else live |= 1 << r;
    }
    if (!live) return;

    for (int i = tid; i < n; i += NT) tw[i] = tw32[i];

    // --- spectra of V and the spectral dots with conj(U^).  Thread (gg, w),
    // w fastest, sums the packed rows gg, gg + G, .. of every chunk.
    const float iW = __builtin_amdgcn_rcpf((float)Wn);
    const int G = Wn >= NT ? 1 : div_uniform(NT, Wn), items = Wn * G;
    float2 s[IT][RG];
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int r = 0; r < RG; ++r) s[i][r] = make_float2(0.f, 0.f);
    const int gg0 = div_small(tid, iW);
    const int CH = fft_chunk_rows(n, Q);
    const int64_t specs = (int64_t)(Q / 2) * Wn;  // of one reference
    for (int p0 = 0; p0 < Q / 2; p0 += CH) {
        const int rows = min(CH, Q / 2 - p0);
        __syncthreads();
        load_packed<NT>(Z0, job.V, n, p0, rows);
        __syncthreads();
        const float2 *Z = fft_rows<NT>(Z0, Z1, rows, n, tw);
        // the rounding to bf16 as a compile-time choice: as a run-time flag
        // the compiler rounds on both paths and selects
        auto dot = [&](auto round) {
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int it = tid + i * NT;
                if (i > 0 && items <= NT) break;  // uniform
                const int gg = i ? 0 : gg0, w = i ? it : it - __mul24(gg0, Wn);
                if (it >= items) continue;
                for (int pl = gg; pl < rows; pl += G) {
                    float2 xe, xo;
                    unpack(Z, pl, n, w, xe, xo);
                    const float4 *uh = job.Uh + (int64_t)(p0 + pl) * Wn + w;
                    if constexpr (decltype(round)::value) {
                        xe = bf16r2(xe);
                        xo = bf16r2(xo);
                    }
#pragma unroll
                    for (int r = 0; r < RG; ++r) {
                        if (r >= nr) break;  // uniform
                        const float4 uu = uh[r * specs];
                        float2 ue = make_float2(uu.x, uu.y), uo = make_float2(uu.z, uu.w);
                        if constexpr (decltype(round)::value) {
                            ue = bf16r2(ue);
                            uo = bf16r2(uo);
                        }
                        // conj(ue) * xe + conj(uo) * xo
                        s[i][r].x += ue.x * xe.x + ue.y * xe.y + uo.x * xo.x + uo.y * xo.y;
                        s[i][r].y += ue.x * xe.y - ue.y * xe.x + uo.x * xo.y - uo.y * xo.x;
                    }
                }
            }
        };
        if (bf16)
            dot(std::true_type{});
        else
            dot(std::false_type{});
    }
    __syncthreads();
    // the threads' sums through the FFT buffers: [r][gg][w]
    float2 *Sacc = Z0;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int it = tid + i * NT;
#pragma unroll
        for (int r = 0; r < RG; ++r)
            if (r < nr && it < items) Sacc[r * items + it] = s[i][r];
    }
    __syncthreads();
    for (int x = tid; x < nr * Wn; x += NT) {
        const int r = div_small(x, iW), w = x - __mul24(r, Wn);
        float2 t = make_float2(0.f, 0.f);
        for (int gg = 0; gg < min(G, CH); ++gg) {  // further groups had no rows
            const float2 v = Sacc[r * items + __mul24(gg, Wn) + w];
            t.x += v.x;
            t.y += v.y;
        }
        S[r * (Wn + 1) + w] = t;
    }
    __syncthreads();

    // --- inverse transform over w.  Lags l and l + n/2 share every twiddle up
    // to the sign (-1)^w, so one sum over even w and one over odd w gives both;
    // the w range is cut in `parts` so that every thread has a share.
    const float ih = __builtin_amdgcn_rcpf((float)half);
    const int parts = min(8, max(1, div_uniform(NT, half)));
    const int len = div_uniform(half - 2 + parts, parts);
    float2 *ps = Z0;  // [parts][nr][half] (even, odd)
    const float ir = __builtin_amdgcn_rcpf((float)nr);
    for (int x = tid; x < parts * nr * half; x += NT) {
        const int pr = div_small(x, ih), l = x - __mul24(pr, half);
        const int part = div_small(pr, ir), r = pr - __mul24(part, nr);
        const float2 *Sr = S + r * (Wn + 1);
        const int w0 = 1 + part * len, w1 = min(w0 + len, half);
        float ev = 0.f, od = 0.f;
        int m = __mul24(w0, l);
        m -= __mul24(div_small(m, 0.5f * ih), n);
        for (int w = w0; w < w1; ++w) {
            const float2 t = tw[m], v = Sr[w];
            const float re = v.x * t.x + v.y * t.y;  // Re(S e^{+2 pi i w l / n})
            if (w & 1) od += re;
            else ev += re;
            m += l;
            if (m >= n) m -= n;
        }
        ps[x] = make_float2(ev, od);
    }
    __syncthreads();

    // --- translation correction, objective per lag
    const double nq = (double)n * (double)Q;
    for (int x = tid; x < nr * half; x += NT) {
        const int r = div_small(x, ih), l = x - __mul24(r, half);
        const double *au = job.au + 4 * r;
        float ev = 0.f, od = 0.f;
        for (int part = 0; part < parts; ++part) {
            const float2 v = ps[part * nr * half + x];
            ev += v.x;
            od += v.y;
        }
        const float2 *Sr = S + r * (Wn + 1);
        const float ends = Sr[0].x + ((l & 1) ? -Sr[half].x : Sr[half].x);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int lag = l + h * half;
            const double Cl = ((double)ends + 2.0 * (double)(h ? ev - od : ev + od)) / (double)n;
            double d = (au[1] + av[1] - 2.0 * Cl) / nq;
            if (mode == 0) {
                const double2 b = trans_moment(au, av, tw64[lag]);
                d -= 2.0 * (b.x * b.x + b.y * b.y);
            }
            D[r * n + lag] = d;
            if (job.curve && (live >> r & 1)) job.curve[r * job.stride * n + lag] = (float)d;
        }
    }
    __syncthreads();

    // --- top-K lags of each reference, one wave per reference
    for (int r = wave; r < nr; r += NW) {
        double *Dr = D + r * n;
        for (int c = 0; c < K; ++c) {
            double v = __builtin_inf();
            int i = 0x7fffffff;
            for (int l = lane; l < n; l += 64) argmin_merge(v, i, Dr[l], l);
            wave_argmin(v, i);
            if (i >= n) i = 0;  // every D* is NaN
            if (lane == 0) {
                Dr[i] = __builtin_inf();
                double2 b = make_double2(0.0, 0.0);
                if (mode == 0) b = trans_moment(job.au + 4 * r, av, tw64[i]);
                lagS[r * K + c] = i;
                shiftS[r * K + c] = make_float2((float)(2.0 * b.x), (float)(2.0 * b.y));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
    __syncthreads();

    // --- FP32 rescore of the candidates: direct residual sums, kAlignSlots of
    // the nr K candidates at a time.  RS rows of V at a time lie in LDS column
    // by column, RP / 4 an odd number of 16-byte groups per column, so that a
    // candidate's four rows at the lag's column are one conflict-free b128 read
    // from an address that only advances with the rows; a thread keeps its
    // column, with the translation's term and the column's offset of every
    // candidate, and takes every G2-th group of four rows.  (One element a step
    // took ten instructions a candidate, most of them indices; now four and a
    // quarter of a read: the pairs above took 199, 452 and 18 us with that.)
    float *Vs = (float *)Z0;
    const int slots = nr * K;
    const float in = __builtin_amdgcn_rcpf((float)n), iK = __builtin_amdgcn_rcpf((float)K);
    const int jg = div_small(tid, in), k_0 = tid - __mul24(jg, n);
    const int G2 = n < NT ? div_uniform(NT, n) : 1;
    int RS, RP;  // uniform; Q is a multiple of 4
    {
        int most = div_uniform(align_work_floats(n, RG), n) & ~3;
        if (!(most & 4)) most -= 4;
        const int chunks = div_uniform(Q + most - 1, most);
        RS = (div_uniform(Q + chunks - 1, chunks) + 3) & ~3;
        RP = RS & 4 ? RS : RS + 4;
    }
    auto rescore = [&](auto count, int c0, int nb) {
        constexpr int NB = decltype(count)::value;
        float(*sums)[kAlignSlots] = red[c0 / kAlignSlots & 1];
        float part[NB];
        int lag[NB], ref[NB];
        float2 sh[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const int q = c0 + min(c, nb - 1);  // slots past the last repeat it
            part[c] = 0.f;
            lag[c] = __builtin_amdgcn_readfirstlane(lagS[q]);
            ref[c] = __builtin_amdgcn_readfirstlane(div_small(q, iK));
            sh[c] = shiftS[q];
        }
        for (int j0 = 0; j0 < Q; j0 += RS) {
            const int quads = min(RS, Q - j0) >> 2;
            if (RS < Q || c0 == 0) {  // else V is there already
                const float *Vg = job.V + (int64_t)j0 * n;
                __syncthreads();
                if (jg < G2)
                    for (int k = k_0; k < n; k += NT)
                        for (int q = jg; q < quads; q += G2) {
                            const float *v = Vg + __mul24(4 * q, n) + k;
                            *(float4 *)(Vs + __mul24(k, RP) + 4 * q) =
                                make_float4(v[0], v[n], v[2 * n], v[3 * n]);
                        }
                __syncthreads();
            }
            if (jg >= G2) continue;  // no barrier but those every thread meets
            const float *Ug = job.U + (int64_t)j0 * n;
            for (int k = k_0; k < n; k += NT) {
                const float2 d = tw[k];
                float t[NB];
                const float *vc[NB];
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    int kk = k + lag[c];
                    if (kk >= n) kk -= n;
                    vc[c] = Vs + __mul24(kk, RP);
                    t[c] = sh[c].x * d.x + sh[c].y * d.y;
                }
                auto quad = [&](int q) {
                    float u[4];
                    const unsigned o = __mul24(4 * q, n) + k;
#pragma unroll
                    for (int c = 0; c < NB; ++c) {
                        if (c == 0 || ref[c] != ref[c - 1]) {  // uniform
                            const float *p = Ug + (int64_t)ref[c] * Q * n;
#pragma unroll
                            for (int i = 0; i < 4; ++i) u[i] = p[o + i * n];
                        }
                        const float4 v = *(const float4 *)(vc[c] + 4 * q);
                        const float e0 = u[0] - v.x - t[c], e1 = u[1] - v.y - t[c];
                        const float e2 = u[2] - v.z - t[c], e3 = u[3] - v.w - t[c];
                        // in pairs: a quarter of the roundings in the long sum
                        part[c] += fmaf(e1, e1, e0 * e0) + fmaf(e3, e3, e2 * e2);
                    }
                };
#pragma unroll 1
                for (int q = jg; q < quads; q += G2) quad(q);
            }
        }
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const float v = wave_butterfly_sum(part[c]);
            if (lane == 0) sums[wave][c] = v;
        }
        __syncthreads();
        if (tid < nb) {
            float t = 0.f;
            for (int w = 0; w < NW; ++w) t += sums[w][tid];
            valS[c0 + tid] = t / (float)nq;
        }
    };
    for (int c0 = 0; c0 < slots; c0 += kAlignSlots) {
        const int nb = min(kAlignSlots, slots - c0);
        if (nb == 1) rescore(std::integral_constant<int, 1>{}, c0, nb);
        else rescore(std::integral_constant<int, kAlignSlots>{}, c0, nb);
    }
    __syncthreads();
    if (tid < nr && (live >> tid & 1)) {
        const int r = tid;
        int bc = r * K;
        for (int c = bc + 1; c < r * K + K; ++c)
            if (valS[c] < valS[bc] || (valS[c] == valS[bc] && lagS[c] < lagS[bc])) bc = c;
        const float L = (float)g.L;
        Result *res = job.res + r * job.stride;
        res->rot_index = lagS[bc];
        res->theta_rad = (float)(6.283185307179586 * (double)lagS[bc] / (double)n);
        res->shift_px[0] = shiftS[bc].x * 0.5f * L;
        res->shift_px[1] = shiftS[bc].y * 0.5f * L;
        res->sw2sq = valS[bc];
        res->status = 0;
    }
}

}  // namespace sw
