// The far field of the obstacles: a table of local polynomials, built from
// the obstacle set alone, that replaces the walk over far obstacles in the
// fused barrier.
//
// Away from an obstacle 1/(|q - c|^2 - r^2) is smooth in q, so over a cell the
// sum over all obstacles beyond a few cell widths is a polynomial of low
// degree to within FP32 rounding.  The plane around the obstacles is covered
// by three grids of square cells, each finer inside the next; a cell's record
// holds the polynomial of its far obstacles (total degree 8, coefficients in
// FP32, fitted in FP64) and the list of its near obstacles, which are summed
// exactly as before.  A query outside the grids, or in a cell whose near list
// is full, walks all obstacles.
//
// The polynomials are of 1/h itself, and the barrier is 1/max(h, h_eps): an
// obstacle with an h below h_eps anywhere in a cell is near there, however far
// it lies.
//
// Near and far are told apart by an estimate of the polynomial's error: an
// obstacle of radius r whose edge lies kappa half-widths W beyond the cell
// leaves, in units of its term at the centre, an error of 8 (kappa + 1)^-9.25
// times 1.5 for r -> 0, 1.1 at r = 0.2 W, 0.8 at 0.5 W, 0.3 to 0.5 at W and 0.05
// to 0.08 at 5 W (the largest over the cell and the obstacle's direction, for
// the kappas below).  A cell takes the smallest kappa of {3.25, 4, 4.75} at which
// 8 (kappa + 1)^-9.25, each times its obstacle's term, adds up to at most 1.5e-7
// of the far sum, else 6, where no sum is formed and 1.8e-7 is the most.  So the
// far sum is off by at most 2.3e-7, and its macro cell's part by as much again,
// were all errors of one sign at the cell's worst corner; over random worlds
// the sum's error measured 2e-9 to 6e-9 of the whole barrier (rms), at most
// 1e-7, below the FP32 rounding of the walk it replaces.
#pragma once

#include "mppi_internal.hpp"

namespace dbas {

constexpr int kFieldDeg = 8;
constexpr int kFieldCoefs = (kFieldDeg + 1) * (kFieldDeg + 2) / 2;      // 45
constexpr int kFieldWords = 64;                     // 32-bit words per cell record
constexpr int kFieldNear = 2 * (kFieldWords - kFieldCoefs - 1);         // most near obstacles listed: 36
constexpr int kFieldFull = 0xFFFF;                  // the count of a cell whose list is full
constexpr int kFieldLevels = 3;
constexpr int kMacro = 4;                           // cells per macro cell and axis

// Most macro cells of each level (16 cells each): no more than 512 in all, two
// workgroups of the build on each of 256 CUs.  The outermost grid is asked from
// half a box width off the obstacles on: few, large cells.
constexpr int kFieldMacros0 = 276, kFieldMacros1 = 156, kFieldMacros2 = 20;
constexpr int kFieldMacros = kFieldMacros0 + kFieldMacros1 + kFieldMacros2;
constexpr size_t kFieldCellBytes = (size_t)kFieldMacros * kMacro * kMacro * kFieldWords * 4;    // 1.85 MB

// One grid: lower corner, cell side, cells per axis, first record.
struct FieldLevel {
    double x0, y0, side;
    int32_t nx, ny, base, pad;
};

struct FieldHeader {
    FieldLevel level[kFieldLevels];
    float margin;               // how far from the query the evaluated points may lie
    int32_t J;                  // the obstacles it was built for; 0: no field (too far apart for FP32, or
                                //   the obstacles have changed).  A captured iteration holds its own count,
                                //   and walks where this is another.
};
constexpr size_t kFieldBytes = 256 + kFieldCellBytes;       // header, then the records
static_assert(sizeof(FieldHeader) <= 256, "field header");

// Which controllers use a field: those whose step saves at least what a caller
// pays who sets the obstacles before every step (the build kernel, measured 32
// us longer than mppi_set_obstacles alone at J = 64, 40 at 200, 66 at 400;
// mppi_step_noalloc builds in every call).  A step walks every obstacle at
// every pose; by the field a pose costs as much as the walk of j0 obstacles,
// whatever their number.  Measured rollouts, walk against field, at K = 4096
// (T = 50 unless said): quadrotor J = 100 35.4 / 26.9 us, T = 64 J = 64 35.3 /
// 27.6, K = 16384 T = 100 J = 400 with a costmap 455 / 112; vehicle J = 100 37.1 / 42.7, J =
// 160 45.5 / 42.6, J = 400 84.9 / 37.4; its indicator J = 100 38.2 / 25.0,
// J = 200 55.3 / 25.5; a ten-point body J = 160 100.9 / 44.0.  Hence us saved
// = per_pair K T (J - j0).
inline bool field_wanted(int model, int K, int T, int J, int P, int32_t shape_kind, int32_t cost_mode)
{
    if (J < 64) return false;
    double per_pair = 1.9e-7 * P;                       // the general form
    int j0 = 25;
    if (cost_mode != MPPI_COST_DBAS) {
        per_pair = 1.0e-7 * P;
        j0 = 30;
    } else if (P == fixed_points(model) && shape_kind != kShapeGeneral) {
        per_pair = model == MPPI_CAR ? 8.3e-7 : 5.8e-7;
        j0 = model == MPPI_CAR ? 115 : 50;
    }
    return per_pair * (double)K * T * (J - j0) >= 26.0 + 0.1 * J;
}

// How far from the query the points lie whose barriers are summed: the whole
// body for the quadrotors' axis layout (one query per pose), a point at a
// time (0) for every other form.
inline float field_margin(int model, int P, int32_t shape_kind, int32_t cost_mode, const float (*sh)[2])
{
    if (model == MPPI_CAR || cost_mode != MPPI_COST_DBAS || P != fixed_points(model) || shape_kind == kShapeGeneral)
        return 0.0f;
    float m = 0.0f;
    for (int i = 0; i < P; ++i) {
        const float a = sh[i][0] < 0.0f ? -sh[i][0] : sh[i][0];
        m = a > m ? a : m;
    }
    return m;
}

// Device memory of a field, and its build on a stream (one kernel).
hipError_t launch_field(const float* d_obs, int J, float margin, float h_eps, void* d_field, hipStream_t s);

}  // namespace dbas
