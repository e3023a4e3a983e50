// Line projection of images (the Radon transform of Sec. 2.2, discretised
// as a hat-weighted line sum, i.e. pixel-driven linear interpolation onto the
// detector bins).
//
// Formulation on the GPU: gather, atomic-free.  A lane owns one output bin b
// of one "slot" angle theta in [0, pi/4] and walks the image rows.  In row i
// the line of bin b crosses the row at column u = (b - c0 + s (i - c0))/c + c0
// (c = cos theta >= s = sin theta), and the pixels with non-zero weight are
// at most three consecutive columns (the hat has half-width 1/c <= sqrt 2
// columns, because the pixel spacing along the detector is c >= 1/sqrt 2
// bins).  The three hat weights are shared by four angles of the same orbit
// under the symmetries of the square pixel grid:
//   theta        : F[i][j]            -> bin b
//   pi/2 - theta : F[j][i]            -> bin L-1-b
//   pi - theta   : F[i][L-1-j]        -> bin b
//   pi/2 + theta : F[L-1-j][i]        -> bin b
// and theta + pi is the reversed projection of theta.  So one set of weights
// per (slot, bin, row) feeds up to eight output columns; the angle table is
// built with these symmetries exact.
//
// The image is staged through LDS in strips of R rows together with the same
// R columns transposed (the four-kind strips of proj2_dev.h), so that all four
// variants read along LDS rows.  Accumulators live in registers across strips.
// This header holds the task plan's access and the emit step.
#pragma once
#include "sw_internal.h"

namespace sw {

struct ProjShape {
    int L, n, slots;
    int ntasks;            // tasks of 64 lanes (proj_ntasks)
    const PlanLane *perm;  // work order (ProjPlan)
    const int2 *trow;
};

__host__ inline ProjShape proj_shape(int L, int n) {
    ProjShape p;
    p.L = L;
    p.n = n;
    p.slots = n / 8 + 1;
    p.ntasks = proj_ntasks(L, n);
    p.perm = nullptr;
    p.trow = nullptr;
    return p;
}

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) f32x4v LdsF4;

// Item of lane `lane` of task `task` in the work order, or -1.
__device__ __forceinline__ int task_item(const ProjShape &P, int task, int lane) {
    return task < P.ntasks ? P.perm[task * 64 + lane].item : -1;
}

// Walk one output value per (task, variant) to its columns, including the
// theta + pi mirror.  Emit(k, b, value) is called for each produced column.
// Tasks of this wave are tg0 + wave + t * nwaves.
template <int TPW, typename Emit>
__device__ __forceinline__ void emit_outputs(const ProjShape &P, int tg0, int wave, int nwaves,
                                             int lane, const float (&acc)[TPW][4], Emit emit) {
    const int L = P.L, n = P.n, q = n / 4, h = n / 2, o = n / 8;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int item = task_item(P, tg0 + wave + t * nwaves, lane);
        if (item < 0) continue;
        const int k = item / L, b = item - k * L;
        // variant 0: angle k, bin b
        emit(k, b, acc[t][0]);
        emit(k + h, L - 1 - b, acc[t][0]);
        if (k != o) {  // variant 1: angle n/4 - k, bin L-1-b
            emit(q - k, L - 1 - b, acc[t][1]);
            emit(q - k + h, b, acc[t][1]);
        }
        if (k != 0) {  // variant 2: angle n/2 - k, bin b
            emit(h - k, b, acc[t][2]);
            emit(n - k, L - 1 - b, acc[t][2]);
        }
        if (k != 0 && k != o) {  // variant 3: angle n/4 + k, bin b
            emit(q + k, b, acc[t][3]);
            emit(q + k + h, L - 1 - b, acc[t][3]);
        }
    }
}

// Waves per SIMD that a projection kernel of NT threads and TPW tasks per
// wave is compiled for: two 512-thread blocks per compute unit (128 VGPRs)
// while the accumulators and task constants of TPW <= 6 fit.
template <int NT, int TPW>
constexpr int kProjMinWaves = (NT == 512 && TPW <= 6) ? 4 : 1;

// Tasks per wave for a block of nt threads.
inline int tasks_per_wave(int ntasks, int nt) {
    const int nw = nt / 64;
    return (ntasks + nw - 1) / nw;
}

}  // namespace sw
