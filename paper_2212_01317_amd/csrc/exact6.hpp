// The exact Metropolis decision on the 3D lattice.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace mpr {

// The exact decision with up to six neighbours, evaluated as the definition writes it (the oracle's order: back,
// up, left, right, down, front; absent neighbours excluded by `present`).
static __device__ __noinline__ bool exact64_6(float tp, float to, float nb, float nu, float nl, float nr, float nd, float nf,
                                              unsigned present, double two_pi_q, double J, float T, float u2)
{
    double acc = 0.0;
    const double dtp = (double)tp, dto = (double)to;
    if (present & 1u) acc += cos(two_pi_q * (dtp - (double)nb)) - cos(two_pi_q * (dto - (double)nb));
    if (present & 2u) acc += cos(two_pi_q * (dtp - (double)nu)) - cos(two_pi_q * (dto - (double)nu));
    if (present & 4u) acc += cos(two_pi_q * (dtp - (double)nl)) - cos(two_pi_q * (dto - (double)nl));
    if (present & 8u) acc += cos(two_pi_q * (dtp - (double)nr)) - cos(two_pi_q * (dto - (double)nr));
    if (present & 16u) acc += cos(two_pi_q * (dtp - (double)nd)) - cos(two_pi_q * (dto - (double)nd));
    if (present & 32u) acc += cos(two_pi_q * (dtp - (double)nf)) - cos(two_pi_q * (dto - (double)nf));
    const double dE = -J * acc;
    if ((double)T > 0.0) return (double)u2 < exp(-dE / (double)T);
    return dE <= 0.0;
}

}  // namespace mpr
