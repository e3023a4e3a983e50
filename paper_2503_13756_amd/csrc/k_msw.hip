// Max-sliced alignment (extended alignment results: the max-sliced W2 over
// the equispaced slices, the norm of U - V taken over columns), rotation only:
//   M(l) = max_k (1/Q) sum_j (U[j][k] - V[j][(k+l) mod n])^2,  l* = argmin M.
// The column pairing of every lag at once is the n x n product
// C[k][k'] = sum_j U[j][k] V[j][k'] = (U^T V)[k][k'], run on the matrix cores
// in FP32 (v_mfma_f32_16x16x4f32): the lag-l residual of column k is
// |u_k|^2 + |v_{k+l}|^2 - 2 C[k][k+l], and the max over k per lag is an LDS
// atomic max over the diagonals of C.  The top_k lags of that FP32 estimate
// are then rescored as direct residual sums (no cancellation), and the
// smallest rescored value wins (ties to the smaller lag).
//
// One block per pair, n a multiple of 16 up to 128: W waves own RA row blocks
// each of the 16 x 16 tiles of C (W RA = n / 16, so that no wave multiplies
// padding) and all column blocks; V streams through LDS in chunks of 32 rows
// (row stride n + 16 floats, so the four rows of a B fragment fall in distinct
// banks), U comes straight from global memory (the reference tables are
// L2-resident).  The next chunk's rows of both are loaded into registers while
// the current one is multiplied, and the column energies come out of the same
// fragments.  The matrix products are 34 us of 3,001 pairs at n = Q = 96; the
// rest is latency: 238 -> 98 us against four waves with a quarter of
// their products padding and a serial energy loop on n threads (chunks of 64
// rows, not prefetched).
#include "sw_internal.h"

namespace sw {

typedef float f32x4m __attribute__((ext_vector_type(4)));

template <int NN>
struct MswShape {
    static constexpr int NB = NN / 16, RA = NB > 4 ? 2 : 1, W = NB / RA, NT = 64 * W;
};

template <int NN>
__global__ __launch_bounds__(MswShape<NN>::NT) void k_align_msw(PairArgs a, Geo g) {
    static_assert(NN % 16 == 0 && NN <= 128, "n a multiple of 16 up to 128");
    constexpr int NB = MswShape<NN>::NB, RA = MswShape<NN>::RA, W = MswShape<NN>::W,
                  NT = MswShape<NN>::NT;
    constexpr int KC = 32, KS = KC / 4, VS = NN + 16, VL = KC * (NN / 4) / NT;
    static_assert(W * RA == NB && VL * NT == KC * (NN / 4), "msw layout");
    __shared__ float vs[KC * VS];
    __shared__ float uu[NN], vv[NN];
    __shared__ unsigned Dbits[NN];
    __shared__ float colred[NT];
    __shared__ int cand[kMaxTopK];
    __shared__ float cval[kMaxTopK];
    const int Q = g.Q;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int64_t pi = blockIdx.x;
    const int64_t P = a.pairs ? a.n_pairs : a.n_ref * a.n_img;
    if (pi >= P) return;
    const int64_t r = a.pairs ? a.pairs[2 * pi] : pi / a.n_img;
    const int64_t gi = a.pairs ? a.pairs[2 * pi + 1] : pi % a.n_img;
    const bool in_range = r >= 0 && r < a.n_ref && gi >= 0 && gi < a.n_img;
    Result *res = a.out + pi;
    float *curve = a.curve ? a.curve + pi * NN : nullptr;
    int status = 0;
    const double *au = a.ref_aux + 4 * (in_range ? r : 0), *av = a.img_aux + 4 * (in_range ? gi : 0);
    if (!in_range) status = 3;  // bad pair index
    else if (isnan(au[0]) || isnan(av[0])) status = 2;
    else if (!(au[0] > 0.0) || !(av[0] > 0.0)) status = 1;
    if (status) {
        if (t == 0) {
            res->rot_index = 0;
            res->theta_rad = 0.f;
            res->shift_px[0] = res->shift_px[1] = 0.f;
            res->sw2sq = __int_as_float(0x7fc00000);
            res->status = status;
        }
        if (curve)
            for (int l = t; l < NN; l += NT) curve[l] = __int_as_float(0x7fc00000);
        return;
    }
    const float *U = a.ref_qt + r * (int64_t)Q * NN;
    const float *V = a.img_qt + gi * (int64_t)Q * NN;
    for (int i = t; i < NN; i += NT) Dbits[i] = 0u;
    f32x4m acc[RA][NB];
#pragma unroll
    for (int ra = 0; ra < RA; ++ra)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[ra][b] = f32x4m{0.f, 0.f, 0.f, 0.f};
    // column energies: U's in this wave's row blocks (lane: column li, rows lk
    // mod 4), V's in the column blocks b = wave, wave + W, ..
    float ue[RA], ve[(NB + W - 1) / W];
#pragma unroll
    for (int ra = 0; ra < RA; ++ra) ue[ra] = 0.f;
#pragma unroll
    for (int i = 0; i < (NB + W - 1) / W; ++i) ve[i] = 0.f;
    // A fragments A[i][kk] = U[j0 + 4 s + kk][16 (wave + W ra) + i] and the
    // thread's float4s of V's rows, of the chunk at j0; 0 past row Q
    float afr[2][RA][KS];
    float4 vld[VL];
    auto fetch = [&](int j0, float(&A)[RA][KS]) {
#pragma unroll
        for (int i = 0; i < VL; ++i) {
            const int q = t + NT * i, jr = q / (NN / 4), c4 = q - jr * (NN / 4);
            vld[i] = j0 + jr < Q ? *(const float4 *)(V + (int64_t)(j0 + jr) * NN + 4 * c4)
                                 : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int ra = 0; ra < RA; ++ra)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int j = j0 + 4 * s + lk;
                A[ra][s] = j < Q ? U[(int64_t)j * NN + 16 * (wave + W * ra) + li] : 0.f;
            }
    };
    fetch(0, afr[0]);
    auto chunk = [&](int j0, float(&A)[RA][KS], float(&An)[RA][KS]) {
        __syncthreads();  // the previous chunk is no longer read
#pragma unroll
        for (int i = 0; i < VL; ++i) {
            const int q = t + NT * i, jr = q / (NN / 4), c4 = q - jr * (NN / 4);
            *(float4 *)(vs + jr * VS + 4 * c4) = vld[i];
        }
        __syncthreads();
        if (j0 + KC < Q) fetch(j0 + KC, An);
#pragma unroll
        for (int ra = 0; ra < RA; ++ra)
#pragma unroll
            for (int s = 0; s < KS; ++s) ue[ra] = fmaf(A[ra][s], A[ra][s], ue[ra]);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (j0 + 4 * s >= Q) break;  // uniform: Q is a multiple of 4
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                // B[kk][jj] = V[j0 + 4 s + kk][16 b + jj]
                const float bfr = vs[(4 * s + lk) * VS + 16 * b + li];
                if (b % W == wave) ve[b / W] = fmaf(bfr, bfr, ve[b / W]);  // wave-uniform
#pragma unroll
                for (int ra = 0; ra < RA; ++ra)
                    acc[ra][b] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(A[ra][s], bfr, acc[ra][b], 0, 0, 0);
            }
        }
    };
    for (int j0 = 0; j0 < Q; j0 += 2 * KC) {
        chunk(j0, afr[0], afr[1]);
        if (j0 + KC < Q) chunk(j0 + KC, afr[1], afr[0]);
    }
    // sum the four row classes of every column
    auto rows4 = [&](float x) {
        x += __shfl_xor(x, 16, 64);
        return x + __shfl_xor(x, 32, 64);
    };
#pragma unroll
    for (int ra = 0; ra < RA; ++ra) {
        const float x = rows4(ue[ra]);
        if (lk == 0) uu[16 * (wave + W * ra) + li] = x;
    }
#pragma unroll
    for (int i = 0; i < (NB + W - 1) / W; ++i) {
        const float x = rows4(ve[i]);
        if (lk == 0 && wave + W * i < NB) vv[16 * (wave + W * i) + li] = x;
    }
    __syncthreads();
    // residual of column k at lag (k' - k) mod n, max over k by atomics
    const float invQ = 1.f / (float)Q;
#pragma unroll
    for (int ra = 0; ra < RA; ++ra) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 16 * (wave + W * ra) + 4 * lk + e, kp = 16 * b + li;
                const float v = fmaxf((uu[k] + vv[kp] - 2.f * acc[ra][b][e]) * invQ, 0.f);
                const int lag = kp >= k ? kp - k : kp - k + NN;
                atomicMax(&Dbits[lag], __float_as_uint(v));
            }
        }
    }
    __syncthreads();
    if (curve)
        for (int l = t; l < NN; l += NT) curve[l] = __uint_as_float(Dbits[l]);
    // top_k lags of the estimate (wave 0; ties to the smaller lag)
    const int K = a.top_k;
    if (wave == 0) {
        float v0 = lane < NN ? __uint_as_float(Dbits[lane]) : __builtin_inff();
        float v1 = lane + 64 < NN ? __uint_as_float(Dbits[lane + 64]) : __builtin_inff();
        for (int c = 0; c < K; ++c) {
            float v = v0;
            int i = lane;
            if (v1 < v) {
                v = v1;
                i = lane + 64;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const float v2 = __shfl_xor(v, off, 64);
                const int i2 = __shfl_xor(i, off, 64);
                if (v2 < v || (v2 == v && i2 < i)) {
                    v = v2;
                    i = i2;
                }
            }
            if (lane == 0) cand[c] = i;
            if (i == lane) v0 = __builtin_inff();
            if (i == lane + 64) v1 = __builtin_inff();
        }
    }
    __syncthreads();
    // rescore: direct FP32 column residuals at every candidate, max over k
    // (threads past TPC n idle)
    constexpr int TPC = NT / NN;  // threads per column
    const int k = t % NN, part = t / NN;
    for (int c = 0; c < K; ++c) {
        const int l = cand[c];
        const float *Vc = V + (k + l < NN ? k + l : k + l - NN);
        float s = 0.f;
        if (part < TPC)
            for (int j0 = part; j0 < Q; j0 += 8 * TPC) {  // eight rows' loads in flight
                float d[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int64_t o = (int64_t)min(j0 + i * TPC, Q - 1) * NN;
                    d[i] = U[o + k] - Vc[o];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (j0 + i * TPC < Q) s = fmaf(d[i], d[i], s);
            }
        colred[t] = s;
        __syncthreads();
        if (t < NN) {
            float col = 0.f;
            for (int p2 = 0; p2 < TPC; ++p2) col += colred[p2 * NN + t];
            colred[t] = col;
        }
        __syncthreads();
        if (wave == 0) {
            float m = fmaxf(lane < NN ? colred[lane] : 0.f, lane + 64 < NN ? colred[lane + 64] : 0.f);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
            if (lane == 0) cval[c] = m * invQ;
        }
        __syncthreads();
    }
    if (t == 0) {
        int bl = cand[0];
        float bv = cval[0];
        for (int c = 1; c < K; ++c)
            if (cval[c] < bv || (cval[c] == bv && cand[c] < bl)) {
                bv = cval[c];
                bl = cand[c];
            }
        res->rot_index = bl;
        res->theta_rad = (float)(6.283185307179586 * (double)bl / (double)NN);
        res->shift_px[0] = res->shift_px[1] = 0.f;
        res->sw2sq = bv;
        res->status = 0;
    }
}

bool msw_supported(Geo g) { return g.n % 16 == 0 && g.n <= 128; }

template <int NN>
static void launch_msw_t(const PairArgs &a, Geo g, int64_t P, hipStream_t s) {
    hipLaunchKernelGGL((k_align_msw<NN>), dim3((unsigned)P), dim3(MswShape<NN>::NT), 0, s, a, g);
}

hipError_t launch_align_msw(const PairArgs &a, Geo g, hipStream_t s) {
    const int64_t P = a.pairs ? a.n_pairs : a.n_ref * a.n_img;
    if (P <= 0) return hipSuccess;
    switch (g.n) {  // the admissible n (factors 2 and 3) that are multiples of 16 up to 128
    case 16: launch_msw_t<16>(a, g, P, s); break;
    case 32: launch_msw_t<32>(a, g, P, s); break;
    case 48: launch_msw_t<48>(a, g, P, s); break;
    case 64: launch_msw_t<64>(a, g, P, s); break;
    case 96: launch_msw_t<96>(a, g, P, s); break;
    case 128: launch_msw_t<128>(a, g, P, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sw
