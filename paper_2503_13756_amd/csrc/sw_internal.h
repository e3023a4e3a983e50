// Internal declarations shared by the kernels and the host runtime of
// libswalign.  Not part of the public ABI (include/swalign.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sw {

constexpr int kMaxL = 256;
constexpr int kMaxN = 512;
constexpr int kMaxQ = 512;
constexpr int kMaxTopK = 8;

// LDS region of the projection's image strips (proj2_dev.h) in a 512-thread
// block, two of which share a compute unit: 64 KiB.
constexpr int kStripFloats = 16384;
// Rows of the four-kind strips of one image (the persistent mixed tables
// kernel): (L + 5) | 1 positions of 16 bytes per row in the 64 KiB region,
// staged in at most four passes of 512 threads both over the strip's rows of
// ceil(L / 2) column pairs (R <= 4 (512 / H)) and over the H image rows of
// its column runs (R <= 512 / ceil(H / 4)).
__host__ __device__ inline int strip4_rows_max(int L) {
    const int P = (L + 5) | 1, H = (L + 1) >> 1;
    int r = 65536 / (16 * P);
    if (r > L) r = L;
    const int cap = 4 * (512 / H), cap1 = 512 / ((H + 3) / 4);
    if (r > cap) r = cap;
    return r < cap1 ? r : cap1;
}

// Projection work order of one geometry (L, n).  The projection's work
// items are (slot angle, bin) pairs, item = slot * L + bin, in units of 8
// consecutive bins of one slot (the last unit of a slot padded); a task is
// eight units, one item per lane, so that each 8-lane group of a wave reads
// evenly spaced LDS windows.  perm lists the items of task t at
// [64 t, 64 t + 64) (-1 for padding), units grouped so that the lines of a
// task cross nearly the same image rows inside the disk, and trow[t] =
// (first, last) is the range of rows where any of them has a pixel of
// non-zero weight (first > last: none).  Device memory, owned by the context.
__host__ __device__ inline int proj_ntasks(int L, int n) {
    return ((n / 8 + 1) * ((L + 7) / 8) + 7) / 8;
}
// One lane of a task: its item, the item's slot angle (slots for none) and
// the line's offsets: the line of bin b crosses image row i (c0 = (L-1)/2,
// c = cos theta, r = tan theta) at column u(i) = (b - c0)/c + c0 + r (i - c0),
// and A3 = u(0) - 1/c + 3, A3n = A3 + r, each rounded once from FP64
// (launch_plan_lanes; every projection kernel reads these, so that all form
// the same positions).
struct PlanLane {
    float A3, A3n;
    int slot, item;
};
struct ProjPlan {
    int L = 0, n = 0, ntasks = 0;
    PlanLane *perm = nullptr;  // [ntasks * 64]
    int2 *trow = nullptr;  // [ntasks]
};

struct Geo {
    int L, n, Q, levels;
};

// Device copy of the angle table of one n: d[m] = (cos theta_m, -sin theta_m),
// theta_m = 2 pi m / n, which is also the forward DFT twiddle e^{-2 pi i m/n}.
struct AngleTable {
    int n = 0;
    float2 *d32 = nullptr;   // [n]
    double2 *d64 = nullptr;  // [n]
};

// Result record, identical in layout to sw_result.
struct Result {
    int32_t rot_index;
    float theta_rad;
    float shift_px[2];
    float sw2sq;
    int32_t status;
};
static_assert(sizeof(Result) == 24, "sw_result is 24 bytes");

// Fills A3 and A3n of the lanes [0, count) of a plan, which hold (cos theta,
// -sin theta) of their slots (in FP32, from the angle table) on entry.
hipError_t launch_plan_lanes(PlanLane *lanes, int count, int L, hipStream_t s);

// ---- launchers (each returns hipGetLastError() after its launches) ----
// split: one block per (image, task group), for batches too small to fill the
// device with one block per image; clear (with split; nullable): [N], set to 0
hipError_t launch_project(const float *img, int64_t N, Geo g, const AngleTable &t,
                          const ProjPlan &pp, float *pmf, hipStream_t s, bool split = false,
                          unsigned *clear = nullptr);
// small: for batches too small to fill the device with one block per image;
// cols: scratch of quantile_cols_bytes() (one part, or two for the signed
// parts) for the launches that take many blocks per image, or null.  Its
// quantile_cols_done(), N counters, must be 0: the projectors clear them.
size_t quantile_cols_bytes(int64_t N, int n, int parts);
unsigned *quantile_cols_done(void *cols);
hipError_t launch_quantiles(const float *pmf, int64_t N, Geo g, const AngleTable &t, float *qt,
                            double *aux, hipStream_t s, bool small = false,
                            double *cols = nullptr);
// Ramp-filtered projections: the stacked [2Q][n] tables of the positive and
// negative parts (per image) from signed [n][L] columns.
hipError_t launch_quantiles_rf(const float *pf, int64_t N, Geo g, const AngleTable &t, float *qt,
                               double *aux, hipStream_t s, bool small = false,
                               double *cols = nullptr);
// Ramp filter of C columns of L bins (src may equal dst).  hx: the filter's
// cyclic kernel as a table of 2 LP - 1 floats, hx[t] = h[t - (LP - 1)] for
// |t - (LP - 1)| < L and 0 otherwise, LP = ramp_padded_length(L).
int ramp_padded_length(int L);
hipError_t launch_ramp(const float *src, float *dst, int64_t C, int L, const float *hx,
                       hipStream_t s);
// Fused image -> stacked ramp-filtered tables, for geometries where
// tables_rf_fused_fits() holds; hx as for launch_ramp; per_block as for
// launch_tables.
bool tables_rf_fused_fits(Geo g);
hipError_t launch_tables_rf(const float *img, int64_t N, Geo g, const AngleTable &t,
                            const ProjPlan &pp, const float *hx, float *qt, double *aux,
                            hipStream_t s, int per_block = 2);
// sw2sq of the valid results, and the curve, times f.
hipError_t launch_scale_results(Result *out, int64_t P, float *curve, int n, float f,
                                hipStream_t s);
// Fused image -> quantile table; only for geometries where
// tables_fused_fits() holds (the PMF table must fit in LDS).
bool tables_fused_fits(Geo g);
// per_block: images per block, 2 (weights shared by two images, where the
// geometry allows it) or 1; the results are the same.
hipError_t launch_tables(const float *img, int64_t N, Geo g, const AngleTable &t,
                         const ProjPlan &pp, float *qt, double *aux, hipStream_t s,
                         int per_block = 2);
// Angle spectra of quantile tables, w in [0, n/2]: bf16 != 0 stores spec[g][w][j],
// j in [0, Q), as bfloat16 pairs; bf16 == 0 stores [g][j/2][w][j%2] float pairs.
// norms (bf16 only, nullable): [N][spectrum_blocks()][kSpecNorms] partial sums
// over the frequencies 1 .. n/2 of g c_w |U^|^2 and g c_w |U^ - bf16(U^)|^2,
// c_w = 2, 1 at n/2, with g = 2, 2 sin(pi w / n) and 2 |sin(2 pi w / n)|: the
// largest |e^{i a} - e^{i b}| for any two lags, for neighbours and for lags two
// apart.
constexpr int kSpecNorms = 3;
int spectrum_blocks(int64_t N, Geo g);
hipError_t launch_spectrum(const float *qt, int64_t N, Geo g, const AngleTable &t, void *spec,
                           int bf16, hipStream_t s, float2 *norms = nullptr);
struct PairArgs {
    const float *ref_qt;
    const double *ref_aux;
    const float2 *ref_spec;  // FP32 spectra of the references
    int64_t n_ref;
    const float *img_qt;
    const double *img_aux;
    int64_t n_img;
    const int64_t *pairs;  // nullable
    int64_t n_pairs;
    int mode, bf16, top_k;
    Result *out;
    float *curve;  // nullable
};
hipError_t launch_align_pairs(const PairArgs &a, Geo g, const AngleTable &t, hipStream_t s);
// Max-sliced alignment (rotation only) of every pair: n a multiple of 16 up to 128.
bool msw_supported(Geo g);
hipError_t launch_align_msw(const PairArgs &a, Geo g, hipStream_t s);
// The same for n = 128 with register-resident angle FFTs, from the references'
// coefficients (align128_scratch_bytes() of them, written by launch_gamma128
// from the reference tables; a.ref_spec is not read).  per_wave: one pair per
// wave (k_align128w) instead of one pair per block (k_align128).
bool align128_supported(Geo g);
size_t align128_scratch_bytes(Geo g, int64_t n_ref);
hipError_t launch_gamma128(const float *qt, int64_t N, Geo g, const AngleTable &t, float2 *gam,
                           hipStream_t s);
hipError_t launch_align128(const PairArgs &a, Geo g, const AngleTable &t, const float2 *gam,
                           hipStream_t s, bool per_wave = true);

// All reference x image pairs on MFMA (bfloat16 spectra, FP32 accumulate),
// top-k lags per pair, then an FP32 rescore of those lags.
struct MfmaArgs {
    const uint32_t *spec_ref;  // [n_ref][n/2+1][Q] packed bf16 complex
    const uint32_t *spec_img;  // [n_img][n/2+1][Q]
    const float *ref_qt;
    const double *ref_aux;
    int64_t n_ref;
    const float *img_qt;
    const double *img_aux;
    int64_t n_img;
    int mode, top_k;
    const float2 *norm_ref, *norm_img;  // partial norms of the spectra, or null: no pruning
    int nb_ref, nb_img;                 // partial sums per table (spectrum_blocks)
    int16_t *cand;  // [n_ref * n_img][top_k] scratch
    Result *out;
};
bool mfma_path_supported(Geo g);
hipError_t launch_mfma_all_pairs(const MfmaArgs &a, Geo g, const AngleTable &t, hipStream_t s);

hipError_t launch_fill_synthetic(float *x, int64_t n, hipStream_t s);

}  // namespace sw
