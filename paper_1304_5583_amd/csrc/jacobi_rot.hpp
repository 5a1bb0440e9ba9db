// The plane rotation shared by the Jacobi eigensolvers.
#pragma once

#include <hip/hip_runtime.h>

namespace lrr {

// Rotation [c s; -s c] with [c s; -s c]^T [app apq; apq aqq] [c s; -s c] nearly
// diagonal.  t = tan of the angle comes from the hardware's approximate square
// root and reciprocal (about 2^-23): an inexact angle only leaves about 1e-7 of
// the rotated coupling behind, which the following sweep removes unless it is below the
// absolute floor, like couplings that were never rotated (one Newton step on t changed no
// error of Z measured at orders of 130, 1e-6 on replaced columns).  What has to
// hold to full precision is c^2 + s^2 = 1: c = 1 / sqrt(1 + t^2) takes one
// third-order step from the approximate value.  d and f are scaled by a power of
// two first, so that their squares neither overflow nor vanish.  The chain of a
// division, two square roots and another division it replaces took about 600 of
// the 2000 cycles of an inner step.
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double& c, double& s) {
    double d = aqq - app, f = 2.0 * apq;
    const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(f)));
    d = __builtin_amdgcn_ldexp(d, e);
    f = __builtin_amdgcn_ldexp(f, e);
    const double h = __builtin_amdgcn_sqrt(fma(d, d, f * f));
    const double t = (d < 0.0 ? -f : f) * __builtin_amdgcn_rcp(fabs(d) + h);
    const double x = fma(t, t, 1.0);
    const double y = __builtin_amdgcn_rsq(x);
    const double r = fma(-(x * y), y, 1.0);
    c = fma(y * r, fma(r, 0.375, 0.5), y);
    s = t * c;
}

}  // namespace lrr
