// Rounding a double-double sum once, with a proof that the exact sum rounds the
// same way.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace cil {

__host__ __device__ inline __attribute__((always_inline)) void two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// Whether fl(hi + lo) = R, with the rest e, is the correctly rounded value of
// any sum within delta R + slack of hi + lo: no rounding boundary of R lies
// between.  Above R the boundary is half an ulp away, below as far, except below a
// power of two, where the spacing halves; either is tested, as the uncertainty may
// reach past R on the other side of e.  (2^-50: the roundings of this test.)  R = 0
// is taken as it is: a sum of squares whose parts all vanish.
__host__ __device__ inline __attribute__((always_inline)) bool dd_certain(double hi, double lo, double delta, double &R,
                                                                          double slack = 0.0)
{
    double e;
    two_sum(hi, lo, R, e);
    int ex;
    const double frac = frexp(R, &ex);                   // R = frac 2^ex, frac in [0.5, 1)
    const double up = ldexp(1.0, ex - 54), down = frac == 0.5 ? ldexp(1.0, ex - 55) : up;
    const double err = (delta * R + slack) * (1.0 + 0x1p-50);
    return std::isfinite(R) && ((e + err < up && err - e < down) || R == 0.0);
}

}  // namespace cil
