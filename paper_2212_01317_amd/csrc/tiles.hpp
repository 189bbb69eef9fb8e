// Declarations of the multi-sweep tile kernel (tiles.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "items.hpp"
#include "mpr_internal.hpp"

namespace mpr {

// A launch advances every realization by up to `depth` sweeps.
struct TileGeom {
    int depth;
    int ntx, nty, ntiles;
    int rchunk, nchunks;       // realizations per workgroup
    size_t plan_words;         // 32-bit words of the plan (update lists of every tile)
};
TileGeom tile_geometry(int64_t H, int64_t W, int R);

struct TileArgs {
    const float* src;          // [R][H][W] state after sweep `sweep` - 1
    float* dst;                // [R][H][W] state after the last sweep of the launch (samples already in place)
    const uint8_t* mask;
    const TBand* Tb;           // temperatures with the lb_h x lb_w layout (1 x 1: one per site)
    uint32_t* plan;
    int H, W, lb_h, lb_w, nbx, ntx, ntiles, Mw, R, rchunk, nchunks;
    int ns;                    // sweeps of this launch, 1 .. depth
    int64_t HW;
    uint32_t sweep;            // the first sweep's index
    uint32_t real_offset, scene, key0, key1;
    float q, J, delta_e;
    double two_pi_q, Jd;
    float* snap;               // [ns][R][H][W]: the gap cells of every sweep's state too, or null (no energies then)
    long long* e_partial;      // [ns][R][ntiles] energy of each tile's colour-1 bonds (fixed point), or null
};
inline dim3 item_grid(uint32_t nwork)
{
    return dim3(nwork < kItemRow ? (nwork + 7u) / 8u * 8u : kItemRow, (nwork + kItemRow - 1u) / kItemRow);
}
// the plan of a call, from its mask and the sample angles of a.src (realization 0)
hipError_t launch_tile_plan(const TileArgs& a, hipStream_t s);
// a.ns sweeps, src -> dst
hipError_t launch_tile_sweeps(const TileArgs& a, hipStream_t s);
// one sweep (a.ns == 1, no snapshots) without a plan, src -> dst, with its own chunks of realizations (onesweep.hip)
hipError_t launch_one_sweep(const TileArgs& a, hipStream_t s);
// One scene of a batch: the arguments of a launch from its first state buffer to the second, and back.
struct TileScene {
    TileArgs a[2];
    double* e_real;            // [depth][R]
    double* series;            // [cap + 1]
    double* acc;
    double inv_norm;
};
// A launch over the scenes list[0 .. n) (device arrays): items prefix[i] .. prefix[i + 1] are scene list[i]'s.
struct TileBatch {
    const TileScene* scenes;
    const int* list;
    const uint32_t* prefix;
    int n, parity;             // a[parity]
    uint32_t sweep;
    int ns;
    bool table;                // every scene's temperatures fit the LDS table
};
bool tile_uses_table(const TileArgs& a);
// (`work`: the items of the list)
hipError_t launch_tile_batch_plan(const TileBatch& b, uint32_t work, hipStream_t s);
hipError_t launch_tile_batch(const TileBatch& b, uint32_t work, bool energy, hipStream_t s);
// the energies of that launch into each scene's series, and the means of sweep k into means[1 + (k - 1) % ring][n_scenes]
// (ring >= depth; row 0 is the starts')
hipError_t launch_tile_batch_energy(const TileBatch& b, double* means, int n_scenes, int ring, hipStream_t s);
hipError_t launch_tile_batch_accumulate(const TileBatch& b, bool first, int blocks, hipStream_t s);
// acc[n] += the gap angles of ns states [ns][R][HW], state by state, over the realizations in order; first: from 0
hipError_t launch_accumulate_n(const float* states, const uint8_t* mask, int64_t HW, int R, int ns, bool first,
                               double* acc, hipStream_t s);
// e_real[i][r] and e_out[i] (mean over the realizations in order) of ns sweeps, from partial [ns][R][nparts]; host: the
// means also go to host[i], in memory that the host reads while the stream runs, or null
hipError_t launch_energy_reduce_n(const long long* partial, int nparts, int R, int ns, double inv_norm, double* e_real,
                                  double* e_out, double* host, hipStream_t s);

}  // namespace mpr
