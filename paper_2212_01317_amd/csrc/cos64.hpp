// FP64 cosine of a bond's angle difference.
#pragma once
#include <hip/hip_runtime.h>

namespace mpr {

// cos(2 pi q d).  q d is reduced in turns, which is exact, to r in [0, 1/4] with the rounding of the product as a tail, and
// the cosine is its Taylor polynomial in r^2 to (2 pi r)^20 (the rest is below 2e-17), the first term in two parts.  One
// straight line of about 30 FP64 operations; cos of the rounded 2 pi q d forms sine and cosine and selects.  Against 128-bit
// values for uniform angles: rms 2.9e-17 at q = 1/2 and 3.1e-17 at q = 0.3 (cos of the product: 6.9e-17, 4.3e-17).
__device__ __forceinline__ double cos_turns(double q, double d)
{
    const double h = q * d, tail = fma(q, d, -h);
    const double f = h - rint(h), a = fabs(f);
    const bool fold = a > 0.25;
    const double r = fold ? 0.5 - a : a;
    double rl = (f < 0.0) != fold ? -tail : tail;
    if (!(fabs(h) < 1e9)) rl = 0.0;            // (the tail is below 1e-7 turns up to here)
    const double y = r * r, yl = fma(r + r, rl, fma(r, r, -y));
    constexpr double c1 = -0x1.3bd3cc9be45dep+4, c1l = -0x1.698p-50;
    const double w = c1 * y;
    double p = 0x1.ef6e308d6d1c4p-9;
    p = fma(p, y, -0x1.2a0c591af8314p-5);
    p = fma(p, y, 0x1.20c62c2f2d7f5p-2);
    p = fma(p, y, -0x1.b6e24f44b128fp+0);
    p = fma(p, y, 0x1.f9d38a3763cc3p+2);
    p = fma(p, y, -0x1.a6d1f2a204a8cp+4);
    p = fma(p, y, 0x1.e1f506891babbp+5);
    p = fma(p, y, -0x1.55d3c7e3cbffap+6);
    p = fma(p, y, 0x1.03c1f081b5ac4p+6);
    const double e = fma(p, y * y, fma(c1, yl, fma(c1l, y, fma(c1, y, -w))));
    const double t = 1.0 + w, v = t + (((1.0 - t) + w) + e);
    return fold ? -v : v;
}

}  // namespace mpr
