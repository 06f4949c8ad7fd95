// The planes a ray crosses, without the voxels: which planes of each axis,
// in what order, and between which columns.
//
// Plain C++ (no HIP), so that a host program can check every index against
// an enumeration of the planes.
#pragma once

#include <math.h>

#ifdef __HIPCC__
#define DRR_HOST_DEVICE __host__ __device__
#else
#define DRR_HOST_DEVICE
#endif

namespace drr {

// One axis of a ray.  Planes 0..n are numbered in the order the ray meets
// them; plane k lies at alpha = fma(k, da, a0), and fma(alpha, c1, c0) is the
// ray's coordinate in planes.  An axis the ray runs parallel to has
// a0 = -inf, da = c1 = 0 and c0 = its voxel's index: one plane, always passed.
struct RunAxis {
    double a0, da, c1, c0;
    bool neg;   // the ray runs towards lower indices
};

// Planes of the axis at or before alpha (strictly before it with STRICT).
// Every decision about a plane compares the same value, fma(k, da, a0), so
// the order of two crossings is the same from whichever it is asked; the
// coordinate only finds the one plane that is in doubt.
template <bool STRICT>
DRR_HOST_DEVICE inline int planes_passed(const RunAxis& x, double alpha)
{
    const double m = rint(fma(alpha, x.c1, x.c0));
    const double am = fma(m, x.da, x.a0);
    return (int)m + ((STRICT ? am < alpha : am <= alpha) ? 1 : 0);
}

// A direction this small crosses no plane within the ray's [0, 1]: its axis
// counts as parallel (and 1 / d stays finite for the others).
constexpr double kParallel = 1e-200;

// Axis of a grid of n voxels of size sp from o, for the ray s + alpha d;
// *exit is the parameter of the last plane (+inf if parallel), *miss is set
// where a parallel ray lies outside the half-open slab.
DRR_HOST_DEVICE inline RunAxis run_axis(double s, double d, double o, double sp, double inv_sp,
                                        int n, double* exit, bool* miss)
{
#ifdef __clang__
#pragma clang fp contract(off)
#endif
    RunAxis x;
    const double hi = o + (double)n * sp;
    x.neg = d < 0.0;
    const double first = x.neg ? hi : o;
    const double inv = 1.0 / fabs(d);
    x.a0 = (x.neg ? s - first : first - s) * inv;
    x.da = sp * inv;
    x.c1 = fabs(d) * inv_sp;
    x.c0 = (x.neg ? first - s : s - first) * inv_sp;
    *exit = fma((double)n, x.da, x.a0);
    if (!(fabs(d) > kParallel)) {
        if (!(s >= o && s < hi)) *miss = true;
        x.neg = false;
        x.a0 = -HUGE_VAL;
        x.da = x.c1 = 0.0;
        x.c0 = fmin(floor((s - o) / sp), (double)(n - 1));
        *exit = HUGE_VAL;
    }
    return x;
}

// A source or pixel 2^44 voxels away leaves too few bits for the position
// inside the grid; such a ray reads nothing.
DRR_HOST_DEVICE inline bool run_too_far(const RunAxis& x)
{
    return !(fmax(fabs(x.c0), x.c1) < 0x1p44);
}

// Axis along which the ray's runs go.  Best is the axis whose planes it
// crosses most often; `pose` (that axis for the pose's central ray) is taken
// while the ray crosses its planes at least a third as often, so that the rays
// of a wave agree (half as often left more waves with two directions, whose
// passes follow one another: the gradient of two poses of 301 x 301 pixels on
// 88 x 247 x 149 voxels 43.6 us, a third 39.7 us, a quarter 40.0 us).  Per ray and pose, so that results do not depend on which
// rays share a wave.
DRR_HOST_DEVICE inline int run_direction(const double d[3], const double inv_sp[3], int pose)
{
    const double e0 = fabs(d[0]) * inv_sp[0], e1 = fabs(d[1]) * inv_sp[1],
                 e2 = fabs(d[2]) * inv_sp[2];
    const int most = (e0 >= e1 && e0 >= e2) ? 0 : (e1 >= e2 ? 1 : 2);
    const double e = pose == 0 ? e0 : (pose == 1 ? e1 : e2);
    const double m = most == 0 ? e0 : (most == 1 ? e1 : e2);
    return pose >= 0 && 3.0 * e >= m ? pose : most;
}

}  // namespace drr
