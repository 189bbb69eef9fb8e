// Declarations of the 3D lattice (lattice3d.hip), kept apart from mpr_internal.hpp so that the plane's kernels do
// not depend on them.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mpr_internal.hpp"

namespace mpr {

// ---- the 3D lattice (lattice3d.hip): grids D x H x W, site n = (z H + y) W + x, six neighbours, blocks
// lb_d x lb_h x lb_w ----
// The FP32 filter's bound on |dE_fp32 - dE_exact| / J with six neighbours: |(Cx, Sy)| <= 6 makes the terms of the
// plane's derivation 3/2 as large, about 2.3e-5 with every FP32 rounding; 2.75e-5 leaves margin.
constexpr float kDeltaE3 = 2.75e-5f;
constexpr int kB3 = 8;           // columns of a wave's two rows (163 VGPRs; three waves per SIMD have 168)
constexpr int kZSeg3 = 64;       // most planes of a wave's segment (a multiple of 4: window slot = plane & 3)
constexpr int kWaves3 = 3;       // waves per SIMD the 3D sweep is compiled for
constexpr int64_t kMargin3 = 1024;   // floats before and after the lane buffer that the sweep may read (and ignores)
// planes of a segment: about equal segments of at most kZSeg3, shortened while the device has too few waves
int lat3_zseg(int64_t D, int64_t H, int64_t W, int R);
struct Lat3Args {
    int D, H, W, R, Rp, Mw, nbands, nzseg, zseg;
    int nrows;                   // row pairs
    int lb_d, lb_h, lb_w, nbx, nby;
    uint32_t lbw_inv;            // ceil(2^32 / lb_w) for lb_w > 1
    uint32_t sweep, real_offset, scene, key0, key1;
    int colour;
    float q, J, delta_e;
    double two_pi_q, Jd;
};
int64_t lat3_blocks(int64_t D, int64_t H, int64_t W, int lb_d, int lb_h, int lb_w);
// S[b], N[b], Tsum[b], Nobs[b] of Eq. (2) per 3D block (bonds to the +x, +y, +z neighbour)
hipError_t launch_block_stats3(const float* t, const uint8_t* mask, int64_t D, int64_t H, int64_t W, int lb_d,
                               int lb_h, int lb_w, double two_pi_q, double J, double* S, int* N, double* Ts, int* No,
                               hipStream_t s);
struct Init3Args {
    const float* t;
    const uint8_t* mask;
    const double* Ts;
    const int* No;
    const float* gmean;
    int64_t D, H, W;
    int lb_d, lb_h, lb_w, nbx, nby;
    int R;
    uint32_t real_offset, scene, key0, key1;
    int mode;
};
// gap bits of each row's window columns: [(D H) nbands]
hipError_t launch_cells3(const uint8_t* mask, int64_t D, int64_t H, int64_t W, int nbands, uint32_t* cells,
                         hipStream_t s);
// one half-sweep (colour a.colour, all rows) of the lane-layout state [G][n][64], in place; with epart set, the
// fixed-point energy of each row pair's colour-1 sites goes to epart[r][(pair * nbands + band) * nzseg + zseg]; the
// buffer has kMargin3 floats on either side
hipError_t launch_sweep3(const Lat3Args& a, const uint32_t* cells, const TBand* tb, float* state, long long* epart,
                         hipStream_t s);
// the matching curve of the cubic lattice: periodic L^3, one chain per temperature
hipError_t launch_ref3_half(float* state, const float* Tgrid, int nT, int L, uint32_t sweep, int colour, float q,
                            float delta_e, uint32_t key0, uint32_t key1, double two_pi_q, hipStream_t s);
int ref3_energy_parts(int L);
hipError_t launch_ref3_energy(const float* state, int L, int nT, float q, double* partial, int nparts, hipStream_t s);

}  // namespace mpr
