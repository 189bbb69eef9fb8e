// The exact Metropolis decision on the 3D lattice.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace mpr {

// The exact decision with up to six neighbours, evaluated as the definition writes it (the oracle's order: back,
// up, left, right, down, front; absent neighbours excluded by `present`).  A loop: its twelve cosines side by side take 178
// registers, and a kernel that calls it then runs two waves per SIMD instead of six.
static __device__ __noinline__ bool exact64_6(float tp, float to, float nb, float nu, float nl, float nr, float nd, float nf,
                                              unsigned present, double two_pi_q, double J, float T, float u2)
{
    double acc = 0.0;
    const double dtp = (double)tp, dto = (double)to;
#pragma unroll 1
    for (int j = 0; j < 6; ++j) {
        if (!((present >> j) & 1u)) continue;
        const double n = (double)(j == 0 ? nb : j == 1 ? nu : j == 2 ? nl : j == 3 ? nr : j == 4 ? nd : nf);
        acc += cos(two_pi_q * (dtp - n)) - cos(two_pi_q * (dto - n));
    }
    const double dE = -J * acc;
    if ((double)T > 0.0) return (double)u2 < exp(-dE / (double)T);
    return dE <= 0.0;
}

}  // namespace mpr
