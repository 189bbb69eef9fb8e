// Tile geometry of the batched tile sweep (its body is in sweep_body.hpp, its kernel in batched.hip).
#include <hip/hip_runtime.h>

#include "mpr_internal.hpp"

namespace mpr {

void fused_geometry(int64_t H, int64_t W, int R, int tile_h, int* ntx, int* nty, int* rchunk, int* nchunks)
{
    *ntx = (int)((W + 63) / 64);
    *nty = (int)((H + tile_h - 1) / tile_h);
    const int64_t ntiles = (int64_t)(*ntx) * (*nty);
    // enough workgroups to fill 256 CUs several times over; longer realization chunks amortise the setup
    int64_t rc = ntiles * (int64_t)R / 4096;
    if (rc < 1) rc = 1;
    if (rc > R) rc = R;
    if (rc > 64) rc = 64;
    *rchunk = (int)rc;
    *nchunks = (int)((R + rc - 1) / rc);
}

}  // namespace mpr
