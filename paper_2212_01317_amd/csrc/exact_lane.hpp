// The exact Metropolis decision of one lane, formed by several.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace mpr {

// exact64 of lane `src` by the first eight active lanes of the wave (there are as many): a cosine each.
static __device__ __noinline__ bool exact_of_lane(int src, float tp, float to, float nu, float nl, float nr, float nd, unsigned present,
                                           double two_pi_q, double J, float T, float u2)
{
    const unsigned long long act = __ballot(1);
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0));
    src = __builtin_amdgcn_readfirstlane(src);
    auto of = [&](float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src)); };
    const unsigned pres = (unsigned)__builtin_amdgcn_readlane((int)present, src);
    const float n = rank < 2 ? of(nu) : rank < 4 ? of(nl) : rank < 6 ? of(nr) : of(nd);
    const double c = cos(two_pi_q * ((double)(rank & 1 ? of(to) : of(tp)) - (double)n));
    const int lo = __double2loint(c), hi = __double2hiint(c);
    unsigned long long m = act;
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int l0 = __ffsll((long long)m) - 1;
        m &= m - 1;
        const int l1 = __ffsll((long long)m) - 1;
        m &= m - 1;
        const double d = __hiloint2double(__builtin_amdgcn_readlane(hi, l0), __builtin_amdgcn_readlane(lo, l0)) -
                         __hiloint2double(__builtin_amdgcn_readlane(hi, l1), __builtin_amdgcn_readlane(lo, l1));
        if ((pres >> j) & 1u) sum += d;
    }
    const double dE = -J * sum, t = (double)of(T);
    return t > 0.0 ? (double)of(u2) < exp(-dE / t) : dE <= 0.0;
}

}  // namespace mpr
