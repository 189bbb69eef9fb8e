// The start and the end of the chains in the realization-lane layout S[g][n][64] (realization r = 64 g + l), for the runs
// that sweep in that layout: the start is written straight into the lane buffers instead of into the [R][N] state and
// transposed.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "lattice3d.hpp"
#include "mpr_internal.hpp"

namespace mpr {

// the start of k_init (a.state and a.state2 unused) into out0, its samples into out1 too; the cubic lattice's into out.  Pad
// realizations r >= a.R get 0.  The buffers are aligned to 16 bytes.
hipError_t launch_lane_start(const InitArgs& a, float* out0, float* out1, hipStream_t s);
hipError_t launch_lane_start3(const Init3Args& a, float* out, hipStream_t s);
// parts of the energy of a start (mode as in InitArgs) of N sites
int lane_start_parts(int mode, int64_t N);
// the energy partials of k_energy_full (the same per-site terms, so the same integer sums) of that start, partial[R][nparts]:
// a block-mean start holds the same state in every realization, so realization 0's are formed and copied to the others
hipError_t launch_lane_start_energy(const InitArgs& a, const float* lanes, float q, long long* partial, int nparts,
                                    hipStream_t s);
hipError_t launch_lane_start_energy3(const Init3Args& a, const float* lanes, float q, long long* partial, int nparts,
                                     hipStream_t s);
// rows 1 .. R - 1 of partial[R][nparts] from row 0: the start energy of a start that every realization shares
hipError_t launch_rows_from_first(long long* partial, int nparts, int R, hipStream_t s);
// after a sampling sweep: acc[n] += the gap angles over the realizations in order (first: from 0), and/or the [R][N] state
hipError_t launch_lane_end(const float* S, const uint8_t* mask, int64_t N, int R, int first, float* out, double* acc,
                           hipStream_t s);

}  // namespace mpr
