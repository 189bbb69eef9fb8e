// Declarations of the double-checkerboard sweep (dc.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mpr_internal.hpp"

namespace mpr {

// Update lists of a call: per phase (block parity, colour) the row pairs with both sites free from the front of `cap` words
// and those with one from the back, with their numbers in count[phase][both, one].
struct DcPlan {
    uint32_t* list;      // [4][cap]
    uint32_t* count;     // [4][2]
    int64_t cap;         // H Mw
};
// Sec. 2.2.2 double-checkerboard sweep: four in-place phases per sweep over all realizations.
struct DcArgs {
    float* state;        // [R][H][W], updated in place
    const uint8_t* mask;
    const TBand* tb;     // temperatures with the tb_h x tb_w layout (blocks, or 1 x 1 per site)
    int64_t H, W;
    int lb_h, lb_w;      // the blocks of the checkerboard
    int tb_h, tb_w, nbx_t;
    int Mw, R;
    uint32_t real_offset, scene, key0, key1;
    float q, J, delta_e;
    double two_pi_q, Jd;
    DcPlan plan;
};
hipError_t launch_dc_plan(const DcArgs& a, hipStream_t s);
hipError_t launch_dc_sweep(const DcArgs& a, uint32_t sweep, hipStream_t s);

}  // namespace mpr
