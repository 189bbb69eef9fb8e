// The start of the chains (Sec. 3.3: samples keep their angles, gaps the block mean of the samples or a uniform draw), the
// energy of the start, and the end of the chains (the sum over the realizations, the states as planes) in the
// realization-lane layout S[g][n][64], on the plane and on the cubic lattice.  The values and the per-site energy terms are
// those of k_init and k_energy_full.
#include <hip/hip_runtime.h>

#include "metropolis.hpp"
#include "mpr_internal.hpp"
#include "philox.hpp"
#include "rl_start.hpp"

namespace mpr {

namespace {

__device__ __forceinline__ int fix24(float x) { return __float2int_rn(x * 16777216.0f); }

// the angle of site n (row `row` of its plane or cube, column x) in a start without a random part
__device__ __forceinline__ float mean_start(const InitArgs& a, int64_t n, int64_t row, int64_t x)
{
    if (a.mask[n]) return a.t[n];
    const uint32_t b = (uint32_t)row / (uint32_t)a.lb_h * (uint32_t)a.nbx + (uint32_t)x / (uint32_t)a.lb_w;
    return a.No[b] > 0 ? (float)(a.Ts[b] / (double)a.No[b]) : *a.gmean;
}
__device__ __forceinline__ float mean_start(const Init3Args& a, int64_t n, int64_t row, int64_t x)
{
    if (a.mask[n]) return a.t[n];
    const int64_t z = row / a.H, y = row - z * a.H;
    const int64_t b = (z / a.lb_d * a.nby + y / a.lb_h) * a.nbx + x / a.lb_w;
    return a.No[b] > 0 ? (float)(a.Ts[b] / (double)a.No[b]) : *a.gmean;
}
__device__ __forceinline__ int64_t rows_of(const InitArgs& a) { return a.H; }
__device__ __forceinline__ int64_t rows_of(const Init3Args& a) { return a.D * a.H; }
__device__ __forceinline__ uint32_t row_colour(const InitArgs&, int64_t row) { return (uint32_t)row & 1u; }
__device__ __forceinline__ uint32_t row_colour(const Init3Args& a, int64_t row)
{
    const int64_t z = row / a.H;
    return (uint32_t)(z + (row - z * a.H)) & 1u;
}

// A wave takes 64 sites: each lane forms one site's angle, and the wave writes it to the group's 64 realizations, four sites
// a store (pad realizations r >= R get 0).  The second buffer gets the samples only: a sweep writes the gaps of its target.
// Bound by the writes: 4096 x 4096, R = 128, 40% samples: 2.2 ms for 12 GB, 6.4 ms when a wave went site by site with its
// scalar loads and its FP64 division in the chain and wrote both buffers in full.
template <class A>
__global__ __launch_bounds__(256) void k_lane_start_mean(A a, float* __restrict__ out0, float* __restrict__ out1)
{
    const int64_t N = rows_of(a) * a.W;
    const int g = blockIdx.y, l = (int)(threadIdx.x & 63u);
    const int64_t n0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64, n = n0 + l;
    if (n0 >= N) return;
    float v = 0.0f;
    int sample = 0;
    if (n < N) {
        const int64_t row = N <= 0xffffffffll ? (uint32_t)n / (uint32_t)a.W : n / a.W;
        v = mean_start(a, n, row, n - row * a.W);
        sample = a.mask[n];
    }
    const int r = g * 64 + 4 * (l & 15);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int from = 4 * j + (l >> 4);
        const float x = __shfl(v, from, 64);
        const int put = __shfl(sample, from, 64);
        if (n0 + from >= N) break;
        const float4 q = make_float4(r < a.R ? x : 0.0f, r + 1 < a.R ? x : 0.0f, r + 2 < a.R ? x : 0.0f,
                                     r + 3 < a.R ? x : 0.0f);
        const int64_t o = ((int64_t)g * N + n0 + from) * 64 + 4 * (l & 15);
        *reinterpret_cast<float4*>(out0 + o) = q;
        if (out1 && put) *reinterpret_cast<float4*>(out1 + o) = q;
    }
}

// A wave takes the four sites 4 m .. 4 m + 3 of a row at a time, each lane one realization: two Philox pairs, one per colour,
// serve them all.
template <class A>
__global__ __launch_bounds__(256) void k_lane_start_random(A a, float* __restrict__ out0, float* __restrict__ out1)
{
    const int64_t rows = rows_of(a), N = rows * a.W;
    const uint32_t Mw = (uint32_t)((a.W + 3) / 4);
    const int g = blockIdx.y, l = (int)(threadIdx.x & 63u), r = g * 64 + l;
    const int64_t wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int64_t i = (int64_t)blockIdx.x * 4 + wv; i < rows * Mw; i += (int64_t)gridDim.x * 4) {       // i < 2^32
        const uint32_t row = (uint32_t)i / Mw, m = (uint32_t)i - row * Mw;
        const uint32_t c = row_colour(a, row);
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (r < a.R) {
            const U4 w = philox_x3((uint32_t)i, 0u, a.real_offset + (uint32_t)r, ctr_word3(a.scene, TAG_INIT, c), a.key0,
                                   a.key1);
            const U4 u = philox_x3((uint32_t)i, 0u, a.real_offset + (uint32_t)r, ctr_word3(a.scene, TAG_INIT, c ^ 1u),
                                   a.key0, a.key1);
            v[0] = u24(w.x);
            v[1] = u24(u.x);
            v[2] = u24(w.z);
            v[3] = u24(u.z);
        }
        const int64_t n0 = (int64_t)row * a.W + 4 * m;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (4 * (int64_t)m + k >= a.W) break;
            const bool sample = a.mask[n0 + k] != 0;
            const float x = sample && r < a.R ? a.t[n0 + k] : v[k];
            const int64_t o = ((int64_t)g * N + n0 + k) * 64 + l;
            out0[o] = x;
            if (out1 && sample) out1[o] = x;
        }
    }
}

template <class T>
__device__ __forceinline__ T group_sum(T v, T* lds)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63u) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    return lds[0] + lds[1] + lds[2] + lds[3];
}

// Energy of a start without a random part, from the mask, the samples and the block means (a start that every realization
// shares: row 0 of the partials).  4096 x 4096: 194 us; read back from a group of 64 realizations 2.5 ms.
__global__ __launch_bounds__(256) void k_mean_start_energy(InitArgs a, float q, long long* __restrict__ partial)
{
    __shared__ long long lds[4];
    long long acc = 0;
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < a.H * a.W; n += (int64_t)gridDim.x * 256) {
        const int64_t y = (uint32_t)n / (uint32_t)a.W, x = n - y * a.W;
        const float tn = mean_start(a, n, y, x);
        float e = 0.0f;                                   // energy of the site's right and lower bonds / J
        if (x + 1 < a.W) e -= cos_rev(q * (tn - mean_start(a, n + 1, y, x + 1)));
        if (y + 1 < a.H) e -= cos_rev(q * (tn - mean_start(a, n + a.W, y + 1, x)));
        acc += fix24(e);
    }
    acc = group_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

__global__ __launch_bounds__(256) void k_mean_start_energy3(Init3Args a, float q, long long* __restrict__ partial)
{
    __shared__ long long lds[4];
    const int64_t HW = a.H * a.W, N = a.D * HW;
    long long acc = 0;
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < N; n += (int64_t)gridDim.x * 256) {
        const int64_t row = n / a.W, x = n - row * a.W, z = row / a.H, y = row - z * a.H;
        const float tn = mean_start(a, n, row, x);
        float e = 0.0f;
        if (x + 1 < a.W) e -= cos_rev(q * (tn - mean_start(a, n + 1, row, x + 1)));
        if (y + 1 < a.H) e -= cos_rev(q * (tn - mean_start(a, n + a.W, row + 1, x)));
        if (z + 1 < a.D) e -= cos_rev(q * (tn - mean_start(a, n + HW, row + a.H, x)));
        acc += fix24(e);
    }
    acc = group_sum(acc, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// Energy of any start, from the lanes: each wave walks sites (a grid stride), each lane sums its realization's terms; the
// four waves of a workgroup then add their lanes' sums.  (D = 1 on the plane.)
__global__ __launch_bounds__(256) void k_rl_energy_full(const float* __restrict__ lanes, int64_t D, int64_t H, int64_t W,
                                                        int R, float q, long long* __restrict__ partial)
{
    __shared__ long long s_red[4][64];
    const int64_t HW = H * W, N = D * HW;
    const int g = blockIdx.y, l = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const float* st = lanes + (int64_t)g * N * 64 + l;
    long long acc = 0;
    for (int64_t n = (int64_t)blockIdx.x * 4 + wv; n < N; n += (int64_t)gridDim.x * 4) {
        int64_t row, z = 0;                                   // on the scalar unit, in 32 bits where they hold the sites
        if (N <= 0xffffffffll) row = (uint32_t)n / (uint32_t)W;
        else row = n / W;
        const int64_t x = n - row * W;
        if (D > 1) z = row / H;
        const int64_t y = row - z * H;
        const float tn = st[n * 64];
        float e = 0.0f;                                   // energy of the bonds to the next column, row and plane / J
        if (x + 1 < W) e -= cos_rev(q * (tn - st[(n + 1) * 64]));
        if (y + 1 < H) e -= cos_rev(q * (tn - st[(n + W) * 64]));
        if (z + 1 < D) e -= cos_rev(q * (tn - st[(n + HW) * 64]));
        acc += fix24(e);
    }
    s_red[wv][l] = acc;
    __syncthreads();
    const int r = g * 64 + l;
    if (wv == 0 && r < R)
        partial[(int64_t)r * gridDim.x + blockIdx.x] = s_red[0][l] + s_red[1][l] + s_red[2][l] + s_red[3][l];
}

// rows 1 .. R - 1 of partial[R][nparts] from row 0
__global__ __launch_bounds__(256) void k_rows_from_first(long long* __restrict__ partial, int nparts, int R)
{
    const int64_t n = (int64_t)(R - 1) * nparts;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        partial[nparts + i] = partial[i % nparts];
}

// The end of a sampling sweep.  A workgroup takes 64 sites: per group of 64 realizations its waves read the sites' 256-byte
// realization rows into an LDS tile; with ACC lane n of the first wave adds site n's realizations in order r = 0 .. R - 1 to
// acc (the order of a loop over the realizations; the first sweep starts from 0), with OUT the other waves write the tile as
// rows of the [R][N] state.  Without OUT the samples are not read.  Bound by memory: 4096 x 4096, R = 128: 3.1 ms with both,
// 3.6 ms and 3.9 ms as two kernels, of which the sum read only the gaps.
template <bool OUT, bool ACC>
__global__ __launch_bounds__(256) void k_lane_end(const float* __restrict__ S, const uint8_t* __restrict__ mask, int64_t N,
                                                   int R, int first, float* __restrict__ out, double* __restrict__ acc)
{
    __shared__ float tile[64 * 65];                 // [site][realization], rows padded against bank conflicts
    const int64_t n0 = (int64_t)blockIdx.x * 64;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), l = (int)(threadIdx.x & 63u);
    const int64_t ns = n0 + l;
    const bool gap = ACC && ns < N && !mask[ns], mine = ACC && wv == 0 && ns < N;
    const unsigned long long gaps = __ballot(gap);
    double v = mine && gap && !first ? acc[ns] : 0.0;
    for (int g = 0; g * 64 < R; ++g) {
        float x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = 4 * j + wv;
            if (OUT ? n0 + i < N : (gaps >> i & 1) != 0) x[j] = S[((int64_t)g * N + n0 + i) * 64 + l];
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = 4 * j + wv;
            if (OUT ? n0 + i < N : (gaps >> i & 1) != 0) tile[i * 65 + l] = x[j];
        }
        __syncthreads();
        const int m = R - g * 64 < 64 ? R - g * 64 : 64;
        if (ACC && wv == 0) {
            if (gap) {
                int k = 0;
                for (; k + 16 <= m; k += 16) {
                    float y[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) y[j] = tile[l * 65 + k + j];
#pragma unroll
                    for (int j = 0; j < 16; ++j) v += (double)y[j];
                }
                for (; k < m; ++k) v += (double)tile[l * 65 + k];
            }
        } else if (OUT && ns < N) {
            for (int i = ACC ? wv - 1 : wv; i < m; i += ACC ? 3 : 4)
                out[(int64_t)(g * 64 + i) * N + ns] = tile[l * 65 + i];
        }
        __syncthreads();
    }
    if (mine && gap) acc[ns] = v;
    else if (mine && first) acc[ns] = 0.0;
}

template <class A>
hipError_t lane_start(const A& a, int64_t rows, float* out0, float* out1, hipStream_t s)
{
    const unsigned groups = (unsigned)((a.R + 63) / 64);
    if (a.mode == 1) {
        const int64_t blocks = (rows * a.W + 255) / 256;
        hipLaunchKernelGGL(k_lane_start_mean<A>, dim3((unsigned)blocks, groups), dim3(256), 0, s, a, out0, out1);
    } else {
        const int64_t blocks = (rows * ((a.W + 3) / 4) + 3) / 4;
        hipLaunchKernelGGL(k_lane_start_random<A>, dim3((unsigned)(blocks < 8192 ? blocks : 8192), groups), dim3(256), 0, s,
                           a, out0, out1);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lane_start(const InitArgs& a, float* out0, float* out1, hipStream_t s)
{
    return lane_start(a, a.H, out0, out1, s);
}

hipError_t launch_lane_start3(const Init3Args& a, float* out, hipStream_t s)
{
    return lane_start(a, a.D * a.H, out, nullptr, s);
}

// A random start is walked a site per wave and step, so that few parts are a serial chain (a call on 16^3, R = 64: 1.11 ms with
// 4096 sites a part, 0.33 ms with 32); in a shared start a thread has a site, and each part is copied for every realization.
int lane_start_parts(int mode, int64_t N)
{
    const int64_t per = mode == 1 ? 2048 : 32, p = (N + per - 1) / per;
    return (int)(p < 1 ? 1 : p > 4096 ? 4096 : p);
}

hipError_t launch_lane_start_energy(const InitArgs& a, const float* lanes, float q, long long* partial, int nparts,
                                    hipStream_t s)
{
    if (a.mode == 1) {
        hipLaunchKernelGGL(k_mean_start_energy, dim3((unsigned)nparts), dim3(256), 0, s, a, q, partial);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? e : launch_rows_from_first(partial, nparts, a.R, s);
    }
    hipLaunchKernelGGL(k_rl_energy_full, dim3((unsigned)nparts, (unsigned)((a.R + 63) / 64)), dim3(256), 0, s, lanes,
                       (int64_t)1, a.H, a.W, a.R, q, partial);
    return hipGetLastError();
}

hipError_t launch_lane_start_energy3(const Init3Args& a, const float* lanes, float q, long long* partial, int nparts,
                                     hipStream_t s)
{
    if (a.mode == 1) {
        hipLaunchKernelGGL(k_mean_start_energy3, dim3((unsigned)nparts), dim3(256), 0, s, a, q, partial);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? e : launch_rows_from_first(partial, nparts, a.R, s);
    }
    hipLaunchKernelGGL(k_rl_energy_full, dim3((unsigned)nparts, (unsigned)((a.R + 63) / 64)), dim3(256), 0, s, lanes, a.D,
                       a.H, a.W, a.R, q, partial);
    return hipGetLastError();
}

hipError_t launch_lane_end(const float* S, const uint8_t* mask, int64_t N, int R, int first, float* out, double* acc,
                           hipStream_t s)
{
    const dim3 grid((unsigned)((N + 63) / 64));
    if (out && acc) hipLaunchKernelGGL((k_lane_end<true, true>), grid, dim3(256), 0, s, S, mask, N, R, first, out, acc);
    else if (out) hipLaunchKernelGGL((k_lane_end<true, false>), grid, dim3(256), 0, s, S, mask, N, R, first, out, acc);
    else hipLaunchKernelGGL((k_lane_end<false, true>), grid, dim3(256), 0, s, S, mask, N, R, first, out, acc);
    return hipGetLastError();
}

hipError_t launch_rows_from_first(long long* partial, int nparts, int R, hipStream_t s)
{
    if (R <= 1 || nparts <= 0) return hipSuccess;
    const int64_t n = (int64_t)(R - 1) * nparts;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_rows_from_first, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, s, partial,
                       nparts, R);
    return hipGetLastError();
}

}  // namespace mpr
