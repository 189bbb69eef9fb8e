// Gradient of the realization-averaged prediction with respect to the block temperatures.
//
// For a density proportional to exp(-sum_b H_b / T_b) the derivative of an expectation is
// d<f>/dT_b = Cov(f, H_b) / T_b^2 (score function).  H_b is the part of Eq. (1) attributed to block b: every bond
// with at least one gap end, counted in the block of its gap end, one half in each block for a bond between two gaps
// of different blocks (bonds between samples are constant).  With one sampling sweep, E[zhat] = zmin + span E[t], so
// for a loss L(zhat) the estimate over R realizations is Cov_r(g_r, H_rb) / T_b^2 with g_r = sum_v w_v t_rv and
// w_v = dL/dzhat_v * span at gaps.  Everything here is FP64 and reduced in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "cos64.hpp"
#include "mpr_internal.hpp"

namespace mpr {

namespace {

template <class T>
__device__ __forceinline__ T wave_sum64(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The sums over a wave of eight values per lane, value k in the lanes with bits 5..3 equal to k: each exchange halves the
// values a lane keeps (10 exchanges; 48 one value at a time).
__device__ __forceinline__ double wave_sum8(const double* v, int lane)
{
    double a[4], b[2];
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = (h5 ? v[k + 4] : v[k]) + __shfl_xor(h5 ? v[k] : v[k + 4], 32, 64);
#pragma unroll
    for (int k = 0; k < 2; ++k) b[k] = (h4 ? a[k + 2] : a[k]) + __shfl_xor(h4 ? a[k] : a[k + 2], 16, 64);
    double c = (h3 ? b[1] : b[0]) + __shfl_xor(h3 ? b[0] : b[1], 8, 64);
    c += __shfl_xor(c, 4, 64);
    c += __shfl_xor(c, 2, 64);
    c += __shfl_xor(c, 1, 64);
    return c;
}

}  // namespace

// One wave per chunk of a block's rows and RG realizations, or (GROUP, RG = 1) a workgroup: partial H.  A bond inside the block
// is formed once, at its upper or left site, with weight 1 unless both ends are samples; a bond that leaves the block counts
// for the gap on this side, one half where the other end is a gap too.  The weights of a site serve the RG realizations.
// Bound by the FP64 cosines: 512 x 512, 1024 realizations, 32 x 32 blocks: 0.81 ms, 3.20 ms when a workgroup per realization
// formed every bond from both ends (1.62 with the bonds of the left and upper sides in the same loop, where a few lanes hold
// up each wave).
template <int RG, bool GROUP>
__global__ __launch_bounds__(256) void k_block_energy(const float* __restrict__ state, const uint8_t* __restrict__ mask,
                                                       StatsGeom g, double q, double J, int64_t HW, int R,
                                                       double* part /* [R][B * nchunk] */)
{
    const int64_t wg = blockIdx.x;                // block * nchunk + chunk
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr uint32_t step = GROUP ? 256 : 64;
    const uint32_t me = GROUP ? threadIdx.x : (uint32_t)lane;
    const int r0 = GROUP ? (int)blockIdx.y : ((int)blockIdx.y * 4 + wave) * RG;
    if (r0 >= R) return;
    const int b = (int)(wg / g.nchunk), c = (int)(wg % g.nchunk);
    const int by = b / g.nbx, bx = b % g.nbx;
    const int64_t yb = (int64_t)by * g.lb_h, ye = yb + g.lb_h < g.H ? yb + g.lb_h : g.H;
    const int64_t y0 = yb + (int64_t)c * g.G, y1 = y0 + g.G < ye ? y0 + g.G : ye;
    const int64_t x0 = (int64_t)bx * g.lb_w, x1 = x0 + g.lb_w < g.W ? x0 + g.lb_w : g.W;
    double acc[RG];
#pragma unroll
    for (int k = 0; k < RG; ++k) acc[k] = 0.0;
    if (y1 > y0) {
        const uint32_t cols = (uint32_t)(x1 - x0), sites = (uint32_t)(y1 - y0) * cols;
        for (uint32_t i = me; i < sites; i += step) {
            const uint32_t row = i / cols;
            const int64_t y = y0 + row, x = x0 + (i - row * cols), n = y * g.W + x;
            const bool gap = !mask[n];
            double wr = 0.0, wd = 0.0;
            if (x + 1 < g.W) {
                const bool other = !mask[n + 1];
                wr = x + 1 < x1 ? (gap || other ? 1.0 : 0.0) : gap ? (other ? 0.5 : 1.0) : 0.0;
            }
            if (y + 1 < g.H) {
                const bool other = !mask[n + g.W];
                wd = y + 1 < ye ? (gap || other ? 1.0 : 0.0) : gap ? (other ? 0.5 : 1.0) : 0.0;
            }
            // (all loads of a site before its cosines; a neighbour outside the grid is the site itself, with weight 0)
            const int64_t right = x + 1 < g.W ? 1 : 0, down = y + 1 < g.H ? g.W : 0;
            float t0[RG], tr[RG], td[RG];
#pragma unroll
            for (int k = 0; k < RG; ++k) {
                const float* s = state + (int64_t)(r0 + k < R ? r0 + k : R - 1) * HW + n;
                t0[k] = s[0];
                tr[k] = s[right];
                td[k] = s[down];
            }
            if (wr != 0.0) {
#pragma unroll
                for (int k = 0; k < RG; ++k) acc[k] += wr * cos_turns(q, (double)t0[k] - (double)tr[k]);
            }
            if (wd != 0.0) {
#pragma unroll
                for (int k = 0; k < RG; ++k) acc[k] += wd * cos_turns(q, (double)t0[k] - (double)td[k]);
            }
        }
        // the gaps at the block's left and upper sides, whose bond to the next block starts there
        const uint32_t n_left = x0 > 0 ? (uint32_t)(y1 - y0) : 0u, n_up = c == 0 && yb > 0 ? cols : 0u;
        for (uint32_t i = me; i < n_left + n_up; i += step) {
            const int64_t n = i < n_left ? (y0 + i) * g.W + x0 : yb * g.W + x0 + (i - n_left);
            const int64_t other = i < n_left ? -1 : -g.W;
            if (mask[n]) continue;
            const double wo = mask[n + other] ? 1.0 : 0.5;
#pragma unroll
            for (int k = 0; k < RG; ++k) {
                const float* s = state + (int64_t)(r0 + k < R ? r0 + k : R - 1) * HW + n;
                acc[k] += wo * cos_turns(q, (double)s[0] - (double)s[other]);
            }
        }
    }
    double sum;
    int k = 0;
    if constexpr (RG == 8) {
        sum = wave_sum8(acc, lane);
        k = lane >> 3;
        if (lane & 7) return;
    } else {
        sum = wave_sum64(acc[0]);
        if constexpr (GROUP) {
            __shared__ double lds[4];
            if (lane == 0) lds[wave] = sum;
            __syncthreads();
            if (threadIdx.x != 0) return;
            sum = ((lds[0] + lds[1]) + lds[2]) + lds[3];
        } else if (lane != 0) {
            return;
        }
    }
    if (r0 + k < R) part[(int64_t)(r0 + k) * gridDim.x + wg] = -J * sum;
}

// The same from the gap sites, each with its four bonds (one half of a bond to another gap), a workgroup per chunk and
// realization: where the sites of a wave lie in different rows every load takes a cache line per lane, and the samples' are
// not made.
__global__ __launch_bounds__(256) void k_block_energy_narrow(const float* __restrict__ state, const uint8_t* __restrict__ mask,
                                                              StatsGeom g, double q, double J, int64_t HW,
                                                              double* part /* [R][B * nchunk] */)
{
    __shared__ double lds[4];
    const int64_t wg = blockIdx.x;
    const int b = (int)(wg / g.nchunk), c = (int)(wg % g.nchunk);
    const int by = b / g.nbx, bx = b % g.nbx;
    const int64_t yb = (int64_t)by * g.lb_h, ye = yb + g.lb_h < g.H ? yb + g.lb_h : g.H;
    const int64_t y0 = yb + (int64_t)c * g.G, y1 = y0 + g.G < ye ? y0 + g.G : ye;
    const int64_t x0 = (int64_t)bx * g.lb_w, x1 = x0 + g.lb_w < g.W ? x0 + g.lb_w : g.W;
    const float* s = state + (int64_t)blockIdx.y * HW;
    double acc = 0.0;
    if (y1 > y0) {
        const uint32_t cols = (uint32_t)(x1 - x0), sites = (uint32_t)(y1 - y0) * cols;
        for (uint32_t i = threadIdx.x; i < sites; i += 256) {
            const uint32_t row = i / cols;
            const int64_t y = y0 + row, x = x0 + (i - row * cols), n = y * g.W + x;
            if (mask[n]) continue;
            const double t = (double)s[n];
            auto bond = [&](bool there, int64_t m) {
                if (there) acc += (mask[m] ? 1.0 : 0.5) * cos_turns(q, t - (double)s[m]);
            };
            bond(y > 0, n - g.W);
            bond(x > 0, n - 1);
            bond(x + 1 < g.W, n + 1);
            bond(y + 1 < g.H, n + g.W);
        }
    }
    acc = wave_sum64(acc);
    if ((threadIdx.x & 63u) == 0) lds[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + wg] = -J * (((lds[0] + lds[1]) + lds[2]) + lds[3]);
}

// The chunks of a block, added by P lanes (P a power of two), then across them.
__global__ __launch_bounds__(256) void k_block_energy_final(const double* part, int64_t n /* R * B */, int nchunk, int P,
                                                             double* Hrb /* [R][B] */)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, i = t / P;
    double s = 0.0;
    if (i < n)
        for (int c = (int)(t % P); c < nchunk; c += P) s += part[i * nchunk + c];
    for (int o = P >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (i < n && t % P == 0) Hrb[i] = s;
}

hipError_t launch_block_energy(const float* state, const uint8_t* mask, const StatsGeom& g, double two_pi_q,
                               double J, int R, double* part, double* Hrb, hipStream_t s)
{
    const int64_t nwg = g.B() * g.nchunk;
    const double q = (double)(float)(two_pi_q / (2.0 * kPi));        // (2 pi q, q an FP32 value)
    // columns of one or two sites, tall enough that a wave's sites lie in rows of their own: 512 x 512, R = 512, 512 x 1
    // blocks 5.28 / 2.91 ms, 512 x 2 2.40 / 2.19, 64 x 1 2.99 / 3.86, 512 x 4 1.16 / 1.33
    const bool narrow = g.lb_w <= 2 && g.W >= 16 && std::min<int64_t>(g.lb_h, g.H) >= 128 * g.lb_w;
    // eight realizations per wave where that leaves four waves per SIMD; else one, a wave each for small chunks and a
    // workgroup each for large ones, whose sites are a serial chain for a wave.  Wave / workgroup each: 1024 x 1024, R = 4,
    // 4 x 4 blocks 172 / 407 us, 16 x 16 33 / 40, 32 x 32 36 / 30; 154 x 148, R = 60, 32 x 32 20 / 14; 3 x 100000, R = 8,
    // 1 x 100000 2.54 / 0.69 ms
    const int64_t sites = std::min<int64_t>({g.lb_h, g.H, g.G}) * std::min<int64_t>(g.lb_w, g.W);
    if (narrow)
        hipLaunchKernelGGL(k_block_energy_narrow, dim3((unsigned)nwg, (unsigned)R), dim3(256), 0, s, state, mask, g, q, J,
                           g.H * g.W, part);
    else if (nwg * (R / 8) >= 4096)
        hipLaunchKernelGGL((k_block_energy<8, false>), dim3((unsigned)nwg, (unsigned)((R + 31) / 32)), dim3(256), 0, s, state, mask,
                           g, q, J, g.H * g.W, R, part);
    else if (sites <= 256 || (sites < 1024 && nwg * R >= 12288))
        hipLaunchKernelGGL((k_block_energy<1, false>), dim3((unsigned)nwg, (unsigned)((R + 3) / 4)), dim3(256), 0, s, state, mask,
                           g, q, J, g.H * g.W, R, part);
    else
        hipLaunchKernelGGL((k_block_energy<1, true>), dim3((unsigned)nwg, (unsigned)R), dim3(256), 0, s, state, mask,
                           g, q, J, g.H * g.W, R, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n = g.B() * R;
    int P = 1;
    while (P < 64 && P * 2 <= g.nchunk) P *= 2;
    hipLaunchKernelGGL(k_block_energy_final, dim3((unsigned)((n * P + 255) / 256)), dim3(256), 0, s, part, n, g.nchunk, P,
                       Hrb);
    return hipGetLastError();
}

// g_r = sum_v w_v t_rv with w_v = grad_zhat_v * span at gaps: one workgroup per (eight realizations, part of the grid), so
// that the weights are read once for eight states, V sites per load; then the parts of a realization are summed in order.
// Bound by reading the states: 512 x 512, 1024 realizations: 194 us, 525 us with a workgroup per realization.
template <int V>
__global__ __launch_bounds__(256) void k_grad_g_part(const float* __restrict__ state, const float* __restrict__ gz,
                                                      const uint8_t* __restrict__ mask, int64_t HW, int R,
                                                      const double* __restrict__ range, double* part /* [R][P] */)
{
    __shared__ double lds[4][8];
    typedef float fvec __attribute__((ext_vector_type(V)));
    typedef uint8_t bvec __attribute__((ext_vector_type(V)));
    const int r0 = (int)blockIdx.y * 8, lane = (int)(threadIdx.x & 63u);
    const int P = gridDim.x;
    const double span = range[1] - range[0];
    double acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0;
    for (int64_t n = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V; n < HW; n += (int64_t)P * 256 * V) {
        const bvec m = *reinterpret_cast<const bvec*>(mask + n);
        const fvec g = *reinterpret_cast<const fvec*>(gz + n);
        fvec s[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            s[k] = *reinterpret_cast<const fvec*>(state + (int64_t)(r0 + k < R ? r0 + k : R - 1) * HW + n);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (m[v]) continue;
            const double w = (double)g[v] * span;
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] += w * (double)s[k][v];
        }
    }
    const double sum = wave_sum8(acc, lane);
    if ((lane & 7) == 0) lds[threadIdx.x >> 6][lane >> 3] = sum;
    __syncthreads();
    const int k = (int)threadIdx.x;
    if (k < 8 && r0 + k < R)
        part[(int64_t)(r0 + k) * P + blockIdx.x] = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
}

__global__ __launch_bounds__(256) void k_grad_g_final(const double* part, int P, int R, double* g)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= R) return;
    double s = 0.0;
    for (int p = 0; p < P; ++p) s += part[(int64_t)r * P + p];
    g[r] = s;
}

// dT_b = [sum_r (g_r - mean g)(H_rb - mean H_b) / (R - 1)] / T_b^2 (0 when T_b = 0).  A workgroup takes eight blocks, 32 lanes
// each (realizations r % 32), in two passes (256 blocks, 1024 realizations: 21 us, 496 us with one thread per block).
__global__ __launch_bounds__(256) void k_grad_cov(const double* g, const double* Hrb, int R, int64_t B,
                                                   const float* T_blocks, double* dT)
{
    __shared__ double lds[2][4][8];
    const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6), k = lane & 7, first = (int)(threadIdx.x >> 3);
    const int64_t b = (int64_t)blockIdx.x * 8 + k, bc = b < B ? b : B - 1;
    // over the lanes of the same block, the same in each of them
    auto total = [&](double v, double (*l)[8]) {
        v += __shfl_xor(v, 8, 64);
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lane < 8) l[w][k] = v;
        __syncthreads();
        return ((l[0][k] + l[1][k]) + l[2][k]) + l[3][k];
    };
    double gm = 0.0, hm = 0.0;
    for (int r = first; r < R; r += 32) {
        gm += g[r];
        hm += Hrb[(int64_t)r * B + bc];
    }
    gm = total(gm, lds[0]) / (double)R;
    hm = total(hm, lds[1]) / (double)R;
    __syncthreads();
    double cov = 0.0;
    for (int r = first; r < R; r += 32) cov += (g[r] - gm) * (Hrb[(int64_t)r * B + bc] - hm);
    cov = total(cov, lds[0]) / (double)(R - 1);
    if (first != 0 || b >= B) return;
    const double T = (double)T_blocks[b];
    dT[b] = T > 0.0 ? cov / (T * T) : 0.0;
}

// The same with a thread per block, whose loads are rows of H_rb: for many blocks.
__global__ __launch_bounds__(256) void k_grad_cov_row(const double* g, const double* Hrb, int R, int64_t B,
                                                       const float* T_blocks, double* dT)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    double gm = 0.0, hm = 0.0;
    for (int r = 0; r < R; ++r) {
        gm += g[r];
        hm += Hrb[(int64_t)r * B + b];
    }
    gm /= (double)R;
    hm /= (double)R;
    double cov = 0.0;
    for (int r = 0; r < R; ++r) cov += (g[r] - gm) * (Hrb[(int64_t)r * B + b] - hm);
    cov /= (double)(R - 1);
    const double T = (double)T_blocks[b];
    dT[b] = T > 0.0 ? cov / (T * T) : 0.0;
}

int grad_parts(int64_t HW)
{
    int64_t p = (HW + 256 * 16 - 1) / (256 * 16);
    return (int)(p < 1 ? 1 : (p > 256 ? 256 : p));
}

hipError_t launch_temperature_grad(const float* state, const double* Hrb, const float* gz, const uint8_t* mask,
                                   int64_t HW, int R, int64_t B, const double* range, const float* T_blocks,
                                   double* part, double* g, double* dT, hipStream_t s)
{
    const int P = grad_parts(HW);
    const dim3 grid((unsigned)P, (unsigned)((R + 7) / 8));
    if (HW % 4 == 0 && (uintptr_t)state % 16 == 0 && (uintptr_t)gz % 16 == 0 && (uintptr_t)mask % 4 == 0)
        hipLaunchKernelGGL(k_grad_g_part<4>, grid, dim3(256), 0, s, state, gz, mask, HW, R, range, part);
    else
        hipLaunchKernelGGL(k_grad_g_part<1>, grid, dim3(256), 0, s, state, gz, mask, HW, R, range, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_grad_g_final, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, part, P, R, g);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // a thread per block where the blocks alone fill the device, or nearly and the realizations are few: lanes / threads at
    // 2^20 blocks, R = 8 150 / 25 us, at 2^18, R = 128 140 / 89, at 2^17, R = 16 29 / 18, R = 128 57 / 77, at 2^12, R = 512 20 / 126
    if (B >= 196608 || (B >= 65536 && R <= 32))
        hipLaunchKernelGGL(k_grad_cov_row, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, g, Hrb, R, B, T_blocks, dT);
    else
        hipLaunchKernelGGL(k_grad_cov, dim3((unsigned)((B + 7) / 8)), dim3(256), 0, s, g, Hrb, R, B, T_blocks, dT);
    return hipGetLastError();
}

}  // namespace mpr
