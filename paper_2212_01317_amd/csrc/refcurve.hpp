// Declarations of the multi-sweep kernel of the matching curve (refcurve.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mpr_internal.hpp"

namespace mpr {

// How the chains of a curve are cut: `strips` workgroups per chain (0: the chains do not fit, a launch per half-sweep), up
// to `depth` sweeps a launch.
struct RefPlan {
    int strips, depth, threads;
    int per_step;              // units (rows, planes) that the threads take at once, even
    bool field;                // cos and sin of every angle held next to it
};
RefPlan ref_plan(int dim, int L, int nT);

struct RefSweepArgs {
    const float* src;          // [nT][L^dim] state after sweep `sweep` - 1, or null: every angle is 1/2
    float* dst;                // [nT][L^dim] state after the launch; may be src with one strip per chain
    const float* Tgrid;
    int nT, L;
    int ns;                    // sweeps of this launch, 1 .. plan.depth
    uint32_t sweep;            // the first sweep's index
    uint32_t n_therm;          // later sweeps are measured
    uint32_t key0, key1;
    float q, delta_e;
    double two_pi_q;
    double* esum;              // [nT][strips] energies of the measured sweeps, summed
};
hipError_t launch_ref_sweeps(int dim, const RefPlan& p, const RefSweepArgs& a, hipStream_t s);
// e_out[T] = the chain's energies times inv_norm, over the n_meas measured sweeps
hipError_t launch_ref_mean(const double* esum, int strips, int nT, double inv_norm, double n_meas, double* e_out,
                           hipStream_t s);

}  // namespace mpr
