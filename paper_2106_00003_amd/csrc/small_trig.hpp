// sin and cos in float64 for |x| <= pi/4: plain Taylor polynomials, no range reduction.  Truncation error below 1e-17
// relative on that interval.
#pragma once
#include <hip/hip_runtime.h>

namespace givens {

__device__ __forceinline__ double cos_small(double x)
{
    const double z = x * x;
    double p = 1.0 / 20922789888000.0;                 // 1/16!
    p = fma(p, z, -1.0 / 87178291200.0);               // 1/14!
    p = fma(p, z, 1.0 / 479001600.0);                  // 1/12!
    p = fma(p, z, -1.0 / 3628800.0);                   // 1/10!
    p = fma(p, z, 1.0 / 40320.0);                      // 1/8!
    p = fma(p, z, -1.0 / 720.0);                       // 1/6!
    p = fma(p, z, 1.0 / 24.0);                         // 1/4!
    p = fma(p, z, -0.5);
    return fma(p, z, 1.0);
}
__device__ __forceinline__ double sin_small(double x)
{
    const double z = x * x;
    double p = 1.0 / 355687428096000.0;                // 1/17!
    p = fma(p, z, -1.0 / 1307674368000.0);             // 1/15!
    p = fma(p, z, 1.0 / 6227020800.0);                 // 1/13!
    p = fma(p, z, -1.0 / 39916800.0);                  // 1/11!
    p = fma(p, z, 1.0 / 362880.0);                     // 1/9!
    p = fma(p, z, -1.0 / 5040.0);                      // 1/7!
    p = fma(p, z, 1.0 / 120.0);                        // 1/5!
    p = fma(p, z, -1.0 / 6.0);
    return fma(p * z, x, x);
}

// cos and sine of an angle in float64, to 1e-16 up to 1e5 (reduced by multiples of pi / 2)
__device__ __forceinline__ double2 tile_sincos(double th)
{
    double s, c;
    if (fabs(th) <= 1.0e5) {
        const double k = rint(th * 0.63661977236758134308);
        const double r = fma(-k, 6.123233995736766036e-17, fma(-k, 1.5707963267948965580, th));
        const double sr = sin_small(r), cr = cos_small(r);
        const int quarter = (int)k & 3;
        s = quarter & 1 ? cr : sr;
        c = quarter & 1 ? sr : cr;
        if (quarter & 2) s = -s;
        if (quarter == 1 || quarter == 2) c = -c;
    } else {
        sincos(th, &s, &c);
    }
    double2 out;
    out.x = c;
    out.y = s;
    return out;
}

} // namespace givens
