// gfx950 kernels of the SV-MPR conditional simulation (Lach & Zukovic, arXiv 2212.01317).
//
// Built with -ffp-contract=off: every FP64 expression that must reproduce the published-formula arithmetic
// (map, bond energies, the exact Metropolis decision, prediction) is evaluated exactly as written; the FP32 hot
// path uses explicit fmaf where a fused multiply-add is wanted.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <cstdint>

#include "cos64.hpp"
#include "metropolis.hpp"

namespace mpr {

// ------------------------------------------------------------------------------------------------------------
// small device helpers
// ------------------------------------------------------------------------------------------------------------

template <class T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of one value per thread over a workgroup of NT threads; result valid in thread 0.  Fixed order.
template <int NT, class T>
__device__ __forceinline__ T block_sum(T v, T* lds /* NT / 64 entries */)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    T s = T(0);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) s += lds[i];
    }
    __syncthreads();
    return s;
}

// ------------------------------------------------------------------------------------------------------------
// Sec. 2.1: linear map of the samples onto angles
// ------------------------------------------------------------------------------------------------------------
constexpr int MAP_NT = 256;

int map_reduce_blocks(int64_t n)
{
    int64_t b = (n + (int64_t)MAP_NT * 16 - 1) / ((int64_t)MAP_NT * 16);
    return (int)(b < 1 ? 1 : (b > 2048 ? 2048 : b));
}

// The maps over all sites are bound by memory.  V sites at i: four per thread and load where the number of sites and every
// pointer allow it (4096 x 4096 sites: k_map_apply 37.5 -> 21.8 us, k_predict 79 -> 47, k_validate_part 44 -> 26), else one.
template <int V, class T>
__device__ __forceinline__ void load_v(const T* p, int64_t i, T* out)
{
    if constexpr (V == 4) {
        typedef T vec __attribute__((ext_vector_type(4)));
        const vec v = *reinterpret_cast<const vec*>(p + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) out[k] = v[k];
    } else {
        out[0] = p[i];
    }
}
template <int V, class T>
__device__ __forceinline__ void store_v(T* p, int64_t i, const T* in)
{
    if constexpr (V == 4) {
        typedef T vec __attribute__((ext_vector_type(4)));
        vec v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = in[k];
        *reinterpret_cast<vec*>(p + i) = v;
    } else {
        p[i] = in[0];
    }
}
template <class... P>
bool aligned4(int64_t n, const P*... p)
{
    return n % 4 == 0 && (((uintptr_t)p % (4 * sizeof(P)) == 0) && ...);
}

// min, max, count and non-finite count over a workgroup, in thread 0
__device__ __forceinline__ void map_reduce_group(float& mn, float& mx, unsigned long long& cnt, unsigned long long& bad)
{
    __shared__ float smn[MAP_NT / 64], smx[MAP_NT / 64];
    __shared__ unsigned long long sc[MAP_NT / 64], sb[MAP_NT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o, 64));
        mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    cnt = wave_sum(cnt);
    bad = wave_sum(bad);
    const int w = (int)(threadIdx.x >> 6);
    if ((threadIdx.x & 63u) == 0) {
        smn[w] = mn;
        smx[w] = mx;
        sc[w] = cnt;
        sb[w] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < MAP_NT / 64; ++i) {
            mn = fminf(mn, smn[i]);
            mx = fmaxf(mx, smx[i]);
            cnt += sc[i];
            bad += sb[i];
        }
    }
}

template <int V>
__global__ __launch_bounds__(MAP_NT) void k_map_reduce(const float* __restrict__ z, const uint8_t* __restrict__ mask,
                                                        int64_t n, float* pmin, float* pmax, unsigned long long* pcnt,
                                                        unsigned long long* pbad)
{
    float mn = INFINITY, mx = -INFINITY;
    unsigned cnt = 0, bad = 0;
    for (int64_t i = ((int64_t)blockIdx.x * MAP_NT + threadIdx.x) * V; i < n; i += (int64_t)gridDim.x * MAP_NT * V) {
        float zv[V];
        uint8_t m[V];
        load_v<V>(z, i, zv);
        load_v<V>(mask, i, m);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (!m[k]) continue;
            if (isfinite(zv[k])) {
                mn = fminf(mn, zv[k]);
                mx = fmaxf(mx, zv[k]);
            } else {
                ++bad;
            }
            ++cnt;
        }
    }
    unsigned long long c = cnt, b = bad;
    map_reduce_group(mn, mx, c, b);
    if (threadIdx.x == 0) {
        pmin[blockIdx.x] = mn;
        pmax[blockIdx.x] = mx;
        pcnt[blockIdx.x] = c;
        pbad[blockIdx.x] = b;
    }
}

__global__ __launch_bounds__(MAP_NT) void k_map_finalize(const float* pmin, const float* pmax,
                                                          const unsigned long long* pcnt,
                                                          const unsigned long long* pbad, int nblocks, double* range,
                                                          unsigned long long* counts)
{
    float mn = INFINITY, mx = -INFINITY;
    unsigned long long cnt = 0, bad = 0;
    for (int i = threadIdx.x; i < nblocks; i += MAP_NT) {
        mn = fminf(mn, pmin[i]);
        mx = fmaxf(mx, pmax[i]);
        cnt += pcnt[i];
        bad += pbad[i];
    }
    map_reduce_group(mn, mx, cnt, bad);
    if (threadIdx.x == 0) {
        range[0] = (double)mn;
        range[1] = (double)mx;
        counts[0] = cnt;
        counts[1] = bad;
    }
}

template <int V>
__global__ __launch_bounds__(MAP_NT) void k_map_apply(const float* __restrict__ z, const uint8_t* __restrict__ mask,
                                                       int64_t n, const double* __restrict__ range,
                                                       float* __restrict__ t)
{
    const int64_t i = ((int64_t)blockIdx.x * MAP_NT + threadIdx.x) * V;
    if (i >= n) return;
    const double zmin = range[0];
    const double span = range[1] - range[0];
    float zv[V], tv[V];
    uint8_t m[V];
    load_v<V>(z, i, zv);
    load_v<V>(mask, i, m);
#pragma unroll
    for (int k = 0; k < V; ++k) tv[k] = m[k] && span != 0.0 ? (float)(((double)zv[k] - zmin) / span) : 0.0f;
    store_v<V>(t, i, tv);
}

hipError_t launch_map_reduce(const float* z, const uint8_t* mask, int64_t n, float* pmin, float* pmax,
                             unsigned long long* pcnt, unsigned long long* pbad, int nblocks, hipStream_t s)
{
    if (aligned4(n, z, mask))
        hipLaunchKernelGGL(k_map_reduce<4>, dim3(nblocks), dim3(MAP_NT), 0, s, z, mask, n, pmin, pmax, pcnt, pbad);
    else
        hipLaunchKernelGGL(k_map_reduce<1>, dim3(nblocks), dim3(MAP_NT), 0, s, z, mask, n, pmin, pmax, pcnt, pbad);
    return hipGetLastError();
}

hipError_t launch_map_finalize(const float* pmin, const float* pmax, const unsigned long long* pcnt,
                               const unsigned long long* pbad, int nblocks, double* range, unsigned long long* counts,
                               hipStream_t s)
{
    hipLaunchKernelGGL(k_map_finalize, dim3(1), dim3(MAP_NT), 0, s, pmin, pmax, pcnt, pbad, nblocks, range, counts);
    return hipGetLastError();
}

hipError_t launch_map_apply(const float* z, const uint8_t* mask, int64_t n, const double* range, float* t,
                            hipStream_t s)
{
    const bool v4 = aligned4(n, z, mask, static_cast<const float*>(t));
    const int64_t nb = (n / (v4 ? 4 : 1) + MAP_NT - 1) / MAP_NT;
    if (v4) hipLaunchKernelGGL(k_map_apply<4>, dim3((unsigned)nb), dim3(MAP_NT), 0, s, z, mask, n, range, t);
    else hipLaunchKernelGGL(k_map_apply<1>, dim3((unsigned)nb), dim3(MAP_NT), 0, s, z, mask, n, range, t);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Eq. (2) per T-block (Sec. 2.2.2): sample-bond energies and counts, sample-angle sums and counts.
// One workgroup per (block, chunk of block rows); a second pass sums the chunks of a block in order.
// ------------------------------------------------------------------------------------------------------------
constexpr int STATS_NT = 256;

StatsGeom stats_geom(int64_t H, int64_t W, int lb_h, int lb_w)
{
    StatsGeom g;
    g.H = H;
    g.W = W;
    g.lb_h = lb_h;
    g.lb_w = lb_w;
    g.nbx = (int)((W + lb_w - 1) / lb_w);
    g.nby = (int)((H + lb_h - 1) / lb_h);
    const int64_t ew = lb_w < W ? lb_w : W;
    const int64_t eh = lb_h < H ? lb_h : H;
    // sites of a workgroup: 4096, or 1024 on small grids, where few workgroups run (one block of 128 x 128: 21.8 us as 4
    // workgroups, 8.2 us as 16)
    int64_t G = (H * W <= ((int64_t)1 << 20) ? 1024 : 4096) / ew;
    if (G < 1) G = 1;
    if (G > eh) G = eh;
    g.G = (int)G;
    g.nchunk = (int)((eh + G - 1) / G);
    return g;
}

// One chunk of a block (G of its rows) per workgroup.  Bound by the FP64 cosines: 4096 x 4096 sites in 32 x 32 blocks, 60%
// samples, 93 us (119 us with cos and a division of 64-bit indexes per site); the bytes alone are 18 us.
__global__ __launch_bounds__(STATS_NT) void k_block_stats(const float* __restrict__ t,
                                                           const uint8_t* __restrict__ mask, StatsGeom g,
                                                           double q, double J, int bonds, double* pS,
                                                           int* pN, double* pTs, int* pNo)
{
    __shared__ double lds_d[STATS_NT / 64], lds_t[STATS_NT / 64];
    __shared__ int lds_i[STATS_NT / 64], lds_o[STATS_NT / 64];
    const int b = blockIdx.x / g.nchunk, c = blockIdx.x % g.nchunk;
    const int by = b / g.nbx, bx = b % g.nbx;
    const int64_t yb = (int64_t)by * g.lb_h;
    int64_t y_start = yb + (int64_t)c * g.G;
    int64_t y_end = yb + (int64_t)(c + 1) * g.G;
    if (y_end > yb + g.lb_h) y_end = yb + g.lb_h;
    if (y_end > g.H) y_end = g.H;
    const int64_t x_start = (int64_t)bx * g.lb_w;
    int64_t x_end = x_start + g.lb_w;
    if (x_end > g.W) x_end = g.W;
    const int64_t rows = y_end - y_start, cols = x_end - x_start;
    double S = 0.0, Ts = 0.0;
    int N = 0, No = 0;
    if (rows > 0 && cols > 0) {
        const uint32_t sites = (uint32_t)(rows * cols), nc = (uint32_t)cols;      // rows * cols < 2^31
        for (uint32_t i = threadIdx.x; i < sites; i += STATS_NT) {
            const uint32_t r = i / nc;
            const int64_t y = y_start + r, x = x_start + (i - r * nc);
            const int64_t n = y * g.W + x;
            if (!mask[n]) continue;
            const double tn = (double)t[n];
            Ts += tn;
            ++No;
            if ((bonds & 1) && x + 1 < g.W && mask[n + 1]) {
                S += -J * cos_turns(q, tn - (double)t[n + 1]);
                ++N;
            }
            if ((bonds & 2) && y + 1 < g.H && mask[n + g.W]) {
                S += -J * cos_turns(q, tn - (double)t[n + g.W]);
                ++N;
            }
        }
    }
    S = wave_sum(S);
    Ts = wave_sum(Ts);
    N = wave_sum(N);
    No = wave_sum(No);
    const int w = (int)(threadIdx.x >> 6);
    if ((threadIdx.x & 63u) == 0) {
        lds_d[w] = S;
        lds_t[w] = Ts;
        lds_i[w] = N;
        lds_o[w] = No;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        pS[blockIdx.x] = ((lds_d[0] + lds_d[1]) + lds_d[2]) + lds_d[3];
        pN[blockIdx.x] = lds_i[0] + lds_i[1] + lds_i[2] + lds_i[3];
        pTs[blockIdx.x] = ((lds_t[0] + lds_t[1]) + lds_t[2]) + lds_t[3];
        pNo[blockIdx.x] = lds_o[0] + lds_o[1] + lds_o[2] + lds_o[3];
    }
}

// The chunks of a block, added by P lanes rather than one after another (P a power of two: chunk c by lane c % P), then
// across the lanes.
__global__ __launch_bounds__(256) void k_block_stats_final(const double* pS, const int* pN, const double* pTs,
                                                            const int* pNo, int64_t B, int nchunk, int P, double* S,
                                                            int* N, double* Ts, int* No)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x, b = g / P;
    const int lane = (int)(g % P);
    double s = 0.0, ts = 0.0;
    int nn = 0, no = 0;
    if (b < B) {
        for (int c = lane; c < nchunk; c += P) {
            const int64_t i = b * nchunk + c;
            s += pS[i];
            nn += pN[i];
            ts += pTs[i];
            no += pNo[i];
        }
    }
    for (int o = P >> 1; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        ts += __shfl_xor(ts, o, 64);
        nn += __shfl_xor(nn, o, 64);
        no += __shfl_xor(no, o, 64);
    }
    if (b >= B || lane != 0) return;
    if (S) S[b] = s;
    if (N) N[b] = nn;
    if (Ts) Ts[b] = ts;
    if (No) No[b] = no;
}

hipError_t launch_block_stats(const float* t, const uint8_t* mask, const StatsGeom& g, double two_pi_q, double J,
                              double* pS, int* pN, double* pTs, int* pNo, double* S, int* N, double* Ts, int* No,
                              hipStream_t s, int bonds)
{
    const int64_t B = g.B();
    const int64_t nwg = B * g.nchunk;
    const double q = (double)(float)(two_pi_q / (2.0 * kPi));        // (2 pi q, q an FP32 value)
    hipLaunchKernelGGL(k_block_stats, dim3((unsigned)nwg), dim3(STATS_NT), 0, s, t, mask, g, q, J, bonds, pS, pN, pTs,
                       pNo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int P = 1;
    while (P < 64 && P * 2 <= g.nchunk) P *= 2;
    hipLaunchKernelGGL(k_block_stats_final, dim3((unsigned)((B * P + 255) / 256)), dim3(256), 0, s, pS, pN, pTs, pNo, B,
                       g.nchunk, P, S, N, Ts, No);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Energy matching (Sec. 2.1, Sec. 2.2.2): inverse of the matching curve, median fill of blocks without bonds.
// ------------------------------------------------------------------------------------------------------------
// up[i] = the running maximum of the curve, first point first.
__device__ double curve_inverse(double e, const double* cT, const double* up, int n)
{
    if (e <= -1.0) return 0.0;
    if (e <= up[0]) {
        const double denom = up[0] + 1.0;
        return denom > 0.0 ? cT[0] * (e + 1.0) / denom : cT[0];
    }
    int lo = 0, hi = n;                       // the first point at or above e is in (lo, hi]; hi == n: there is none
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (up[mid] >= e) hi = mid;
        else lo = mid;
    }
    if (hi == n) return cT[n - 1];
    const double prev = up[hi - 1], cur = up[hi];
    const double lam = (e - prev) / (cur - prev);
    return exp((1.0 - lam) * log(cT[hi - 1]) + lam * log(cT[hi]));
}

// Bound by latency.  A curve of up to kCurveLds points is held in LDS as its running maximum, so that a block's search is a
// few LDS reads (121 points, 65536 blocks: 5 us, and 34 us for a walk along the curve in memory, which a longer curve
// still takes: each block then reads only the points up to its energy).
constexpr int kCurveLds = 1024;

__device__ double curve_inverse_walk(double e, const double* cT, const double* ce, int n)
{
    if (e <= -1.0) return 0.0;
    double prev = ce[0];
    if (e <= prev) {
        const double denom = prev + 1.0;
        return denom > 0.0 ? cT[0] * (e + 1.0) / denom : cT[0];
    }
    for (int i = 1; i < n; ++i) {
        const double cur = ce[i] > prev ? ce[i] : prev;
        if (cur >= e) {
            const double lam = (e - prev) / (cur - prev);
            return exp((1.0 - lam) * log(cT[i - 1]) + lam * log(cT[i]));
        }
        prev = cur;
    }
    return cT[n - 1];
}

__global__ __launch_bounds__(256) void k_calibrate(const double* S, const int* N, int64_t B, double J,
                                                    const double* cT, const double* ce, int nc, float* T_out,
                                                    double* e_out, int* nb_out)
{
    __shared__ double up[kCurveLds];
    __shared__ double wmax[4];
    if (nc <= kCurveLds) {
        // running maximum (x replaces it only if greater: a NaN after the first point is passed over, a NaN there stays)
        const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
        const double first = ce[0];
        double base = -INFINITY;
        for (int i0 = 0; i0 < nc; i0 += 256) {
            const int i = i0 + (int)threadIdx.x;
            double v = i < nc ? ce[i] : -INFINITY;
            if (!(v == v)) v = -INFINITY;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const double u = __shfl_up(v, o, 64);
                if (lane >= o && u > v) v = u;
            }
            if (lane == 63) wmax[w] = v;
            __syncthreads();
            double m = base;
            for (int j = 0; j < 4; ++j) {
                if (j < w && wmax[j] > v) v = wmax[j];
                if (wmax[j] > m) m = wmax[j];
            }
            if (base > v) v = base;
            if (i < nc) up[i] = first == first ? v : first;
            base = m;
            __syncthreads();
        }
    }
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    const int nb = N[b];
    double e = 0.0;
    float T = -1.0f;   // marker: filled by the median pass
    if (nb > 0) {
        e = S[b] / (J * (double)nb);
        T = (float)(J * (nc <= kCurveLds ? curve_inverse(e, cT, up, nc) : curve_inverse_walk(e, cT, ce, nc)));
    }
    T_out[b] = T;
    if (e_out) e_out[b] = e;
    if (nb_out) nb_out[b] = nb;
}

constexpr int MED_NT = 1024;

// One workgroup, bound by its LDS atomics and by L2 reads of 65536 blocks: 46 us, 96 us when one thread searched the 256 bins
// and the upper of two middle values took a second selection.  With a temperature in every block there is nothing to do.
// k-th smallest (0-based) of the T values of blocks with N > 0, by a 4-pass 8-bit radix select on the FP32 bit
// patterns (T >= 0, so the bit patterns are ordered like the values).
__device__ float radix_select(const float* T, const int* N, int64_t B, unsigned k, unsigned* hist, unsigned* sh)
{
    unsigned prefix = 0u, pmask = 0u;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        for (int i = threadIdx.x; i < 256; i += MED_NT) hist[i] = 0u;
        __syncthreads();
        for (int64_t b = threadIdx.x; b < B; b += MED_NT) {
            if (N[b] > 0) {
                const unsigned key = __float_as_uint(T[b]);
                if ((key & pmask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x < 64) {               // the bin of rank k: four bins per lane, prefix over the lanes
            const int l = (int)threadIdx.x;
            unsigned h[4], sum = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) sum += h[j] = hist[4 * l + j];
            unsigned end = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned u = __shfl_up(end, o, 64);
                if (l >= o) end += u;
            }
            unsigned cum = end - sum;
            if (cum <= k && k < end) {
                int d = 0;
                while (cum + h[d] <= k) cum += h[d++];
                sh[0] = prefix | (unsigned)(4 * l + d) << shift;
                sh[1] = k - cum;
            }
        }
        __syncthreads();
        prefix = sh[0];
        k = sh[1];
        pmask |= 255u << shift;
        __syncthreads();
    }
    return __uint_as_float(prefix);
}

__global__ __launch_bounds__(MED_NT) void k_median_fill(float* T, const int* N, int64_t B, unsigned* n_have)
{
    __shared__ unsigned hist[256];
    __shared__ unsigned sh[2];
    __shared__ unsigned scount[MED_NT / 64];
    unsigned cnt = 0;
    for (int64_t b = threadIdx.x; b < B; b += MED_NT) cnt += N[b] > 0 ? 1u : 0u;
    cnt = block_sum<MED_NT>(cnt, scount);
    if (threadIdx.x == 0) sh[0] = cnt;
    __syncthreads();
    const unsigned count = sh[0];
    __syncthreads();
    if (threadIdx.x == 0) *n_have = count;
    if (count == 0u || count == (unsigned)B) return;      // no temperature at all, or none to fill in
    const float lo = radix_select(T, N, B, (count - 1u) / 2u, hist, sh);
    float med = lo;
    if ((count & 1u) == 0u) {
        // the next value in order: lo again if it has further copies, else the least value above it
        unsigned upto = 0, above = 0xffffffffu;
        const unsigned klo = __float_as_uint(lo);
        for (int64_t b = threadIdx.x; b < B; b += MED_NT) {
            if (N[b] <= 0) continue;
            const unsigned key = __float_as_uint(T[b]);
            if (key <= klo) ++upto;
            else if (key < above) above = key;
        }
        if (threadIdx.x == 0) {
            sh[0] = 0u;
            sh[1] = 0xffffffffu;
        }
        __syncthreads();
        atomicAdd(&sh[0], upto);
        atomicMin(&sh[1], above);
        __syncthreads();
        const float hi = sh[0] > count / 2u ? lo : __uint_as_float(sh[1]);
        med = (float)(((double)lo + (double)hi) * 0.5);
    }
    for (int64_t b = threadIdx.x; b < B; b += MED_NT)
        if (N[b] == 0) T[b] = med;
}

hipError_t launch_calibrate(const double* S, const int* N, int64_t B, double J, const double* cT, const double* ce,
                            int nc, float* T_out, double* e_out, int* nb_out, unsigned* n_have, hipStream_t s)
{
    hipLaunchKernelGGL(k_calibrate, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, S, N, B, J, cT, ce, nc,
                       T_out, e_out, nb_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_median_fill, dim3(1), dim3(MED_NT), 0, s, T_out, N, B, n_have);
    return hipGetLastError();
}

// The mean over all samples, which starts the gaps of a block without samples: where every block has some it is not read
// and 0 is left in its place.  The block sums are added in block order, one sequential FP64 sum: a chunk is in LDS while
// the next is loaded, and one thread adds it (bound by the latency of the additions: 16384 blocks 529 us with the chunk in
// the lanes' registers).
constexpr int GM_CHUNK = 2048;

__global__ __launch_bounds__(256) void k_global_mean(const double* __restrict__ Ts, const int* __restrict__ No,
                                                      int64_t B, float* gmean)
{
    __shared__ double buf[2][GM_CHUNK];
    __shared__ long long s_cnt[4];
    __shared__ int s_empty;
    if (threadIdx.x == 0) s_empty = 0;
    __syncthreads();
    long long cnt = 0;
    bool empty = false;
    for (int64_t b = threadIdx.x; b < B; b += 256) {
        cnt += No[b];
        empty |= No[b] <= 0;
    }
    if (empty) s_empty = 1;
    cnt = block_sum<256>(cnt, s_cnt);         // (its barriers order s_empty)
    if (!s_empty) {
        if (threadIdx.x == 0) *gmean = 0.0f;
        return;
    }
    double sum = 0.0;
    auto fill = [&](int64_t b0, int k, int first) {
        for (int i = (int)threadIdx.x - first; i < GM_CHUNK; i += 256 - first)
            if (i >= 0) buf[k][i] = b0 + i < B ? Ts[b0 + i] : 0.0;
    };
    fill(0, 0, 0);
    __syncthreads();
    for (int64_t b0 = 0, c = 0; b0 < B; b0 += GM_CHUNK, ++c) {
        const int k = (int)(c & 1);
        if (threadIdx.x >= 64) {
            if (b0 + GM_CHUNK < B) fill(b0 + GM_CHUNK, k ^ 1, 64);
        } else if (threadIdx.x == 0) {
            const int m = B - b0 < GM_CHUNK ? (int)(B - b0) : GM_CHUNK;
            int i = 0;
            for (; i + 16 <= m; i += 16) {
                double x[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) x[j] = buf[k][i + j];
#pragma unroll
                for (int j = 0; j < 16; ++j) sum += x[j];
            }
            for (; i < m; ++i) sum += buf[k][i];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *gmean = cnt > 0 ? (float)(sum / (double)cnt) : 0.0f;
}

hipError_t launch_global_mean(const double* Ts, const int* No, int64_t B, float* gmean, hipStream_t s)
{
    hipLaunchKernelGGL(k_global_mean, dim3(1), dim3(256), 0, s, Ts, No, B, gmean);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_tpairs(const float* T, int64_t B, float J, float delta, TBand* tp)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    tp[b] = make_tband(T[b], J, delta);
}

hipError_t launch_tpairs(const float* T, int64_t B, float J, float delta, TBand* tp, hipStream_t s)
{
    hipLaunchKernelGGL(k_tpairs, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, T, B, J, delta, tp);
    return hipGetLastError();
}

// Directional coupling: per block {Tx, Ty} from T[b], T[B + b] raised to at least `floor`, the scales
// kx = J log2(e) / Tx, ky = J log2(e) / Ty of the two field components and the error band of the filter.
__global__ __launch_bounds__(256) void k_tpairs_directional(const float* __restrict__ T, int64_t B, float J,
                                                             float delta, float floor_T, TBandDir* __restrict__ out)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    out[b] = make_tband_directional(fmaxf(T[b], floor_T), fmaxf(T[B + b], floor_T), J, delta);
}

hipError_t launch_tpairs_directional(const float* T, int64_t B, float J, float delta, float floor_T, TBandDir* out,
                                     hipStream_t s)
{
    hipLaunchKernelGGL(k_tpairs_directional, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, T, B, J, delta,
                       floor_T, out);
    return hipGetLastError();
}

// out[i] = max(T[i], floor_T)
__global__ __launch_bounds__(256) void k_floor(float* __restrict__ T, int64_t n, float floor_T)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) T[i] = fmaxf(T[i], floor_T);
}

hipError_t launch_floor(float* T, int64_t n, float floor_T, hipStream_t s)
{
    hipLaunchKernelGGL(k_floor, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, T, n, floor_T);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Start of the chains (Sec. 3.3): block means of the sample angles (SV-MPR) or uniform draws (MPR).
// ------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init(InitArgs a)
{
    const int64_t HW = a.H * a.W;
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (n >= HW) return;
    const int64_t y = n / a.W, x = n % a.W;
    float v;
    if (a.mask[n]) {
        v = a.t[n];
    } else if (a.mode == 1) {
        const int64_t b = (y / a.lb_h) * a.nbx + (x / a.lb_w);
        v = a.No[b] > 0 ? (float)(a.Ts[b] / (double)a.No[b]) : *a.gmean;
    } else {
        const uint32_t Mw = (uint32_t)((a.W + 3) / 4);
        const uint32_t pair = (uint32_t)y * Mw + (uint32_t)(x >> 2);
        const uint32_t colour = (uint32_t)((x + y) & 1);
        const U4 w = philox4x32_10(pair, 0u, a.real_offset + (uint32_t)r, ctr_word3(a.scene, TAG_INIT, colour),
                                   a.key0, a.key1);
        v = u24(((x >> 1) & 1) ? w.z : w.x);
    }
    a.state[(int64_t)r * HW + n] = v;
    if (a.state2) a.state2[(int64_t)r * HW + n] = v;
}

hipError_t launch_init(const InitArgs& a, hipStream_t s)
{
    const int64_t HW = a.H * a.W;
    hipLaunchKernelGGL(k_init, dim3((unsigned)((HW + 255) / 256), (unsigned)a.R), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Whole-grid energy of the current states (used for e(0)): every site's right and lower bond, FP32 terms,
// FP64 per-workgroup sums.  partial layout [R][part].
constexpr int EN_NT = 256;

int energy_full_parts(int64_t H, int64_t W)
{
    const int64_t HW = H * W;
    int64_t p = (HW + EN_NT * 8 - 1) / (EN_NT * 8);
    return (int)(p < 1 ? 1 : (p > 4096 ? 4096 : p));
}

__device__ __forceinline__ int fix24(float x) { return __float2int_rn(x * 16777216.0f); }

__global__ __launch_bounds__(EN_NT) void k_energy_full(const float* __restrict__ state, int64_t H, int64_t W, float q,
                                                        float J, long long* partial)
{
    __shared__ long long s_red[EN_NT / 64];
    (void)J;
    const int r = blockIdx.y;
    const int64_t HW = H * W;
    const float* st = state + (int64_t)r * HW;
    // (32-bit indexes: H W < 2^31)
    const uint32_t Wu = (uint32_t)W, last = (uint32_t)(HW - W);
    long long acc = 0;
    for (uint32_t n = blockIdx.x * (uint32_t)EN_NT + threadIdx.x; n < (uint32_t)HW; n += gridDim.x * (uint32_t)EN_NT) {
        const uint32_t x = n - n / Wu * Wu;
        const float tn = st[n];
        float e = 0.0f;                                   // energy of the site's right and lower bonds / J
        if (x + 1 < Wu) e -= cos_rev(q * (tn - st[n + 1]));
        if (n < last) e -= cos_rev(q * (tn - st[n + Wu]));
        acc += fix24(e);
    }
    const long long tot = block_sum<EN_NT>(acc, s_red);
    if (threadIdx.x == 0) partial[(int64_t)r * gridDim.x + blockIdx.x] = tot;
}

hipError_t launch_energy_full(const float* state, int64_t H, int64_t W, int R, float q, float J, long long* partial,
                              int nparts, hipStream_t s)
{
    hipLaunchKernelGGL(k_energy_full, dim3((unsigned)nparts, (unsigned)R), dim3(EN_NT), 0, s, state, H, W, q, J,
                       partial);
    return hipGetLastError();
}

// e_real[r] = (sum over parts of partial[r][p]) * unit * inv_norm (integer sum: order-free), one workgroup per
// realization; then e_out = mean over realizations (in order).
__global__ __launch_bounds__(256) void k_energy_real(const long long* __restrict__ partial, int nparts,
                                                      double inv_norm, double* e_real)
{
    __shared__ long long s_red[4];
    const int r = blockIdx.x;
    const long long* row = partial + (int64_t)r * nparts;
    long long s = 0;
    for (int p = threadIdx.x; p < nparts; p += 256) s += row[p];
    s = block_sum<256>(s, s_red);
    if (threadIdx.x == 0) e_real[r] = ((double)s * kFixUnit) * inv_norm;
}

__global__ void k_energy_mean(const double* e_real, int R, double* e_out)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double s = 0.0;
    for (int r = 0; r < R; ++r) s += e_real[r];
    *e_out = s / (double)R;
}

hipError_t launch_energy_reduce(const long long* partial, int nparts, int R, double inv_norm, double* e_real,
                                double* e_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_energy_real, dim3((unsigned)R), dim3(256), 0, s, partial, nparts, inv_norm, e_real);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_energy_mean, dim3(1), dim3(64), 0, s, e_real, R, e_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Sampling (Sec. 2.1): acc[n] += sum over realizations (in order) of the gap angle; first pass starts from 0.
// ------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_accumulate(const float* __restrict__ state, const uint8_t* __restrict__ mask,
                                                     int64_t HW, int R, int first, double* __restrict__ acc)
{
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= HW) return;
    if (mask[n]) {
        if (first) acc[n] = 0.0;
        return;
    }
    double a = first ? 0.0 : acc[n];
    for (int r = 0; r < R; ++r) a += (double)state[(int64_t)r * HW + n];
    acc[n] = a;
}

hipError_t launch_accumulate(const float* state, const uint8_t* mask, int64_t HW, int R, int first, double* acc,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_accumulate, dim3((unsigned)((HW + 255) / 256)), dim3(256), 0, s, state, mask, HW, R, first,
                       acc);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Back-transform of the conditional mean (Sec. 2.1) and the validation measures (Eq. 3, Eq. 4).
// ------------------------------------------------------------------------------------------------------------
template <int V>
__global__ __launch_bounds__(256) void k_predict(const double* __restrict__ acc, const float* __restrict__ z,
                                                  const uint8_t* __restrict__ mask, int64_t n, int64_t n_samples,
                                                  const double* __restrict__ range, float* __restrict__ zhat)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= n) return;
    const double zmin = range[0], span = range[1] - range[0];
    float zv[V], out[V];
    uint8_t m[V];
    double a[V];
    load_v<V>(z, i, zv);
    load_v<V>(mask, i, m);
    load_v<V>(acc, i, a);
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const double tbar = a[k] / (double)n_samples;
        out[k] = m[k] ? zv[k] : (float)(zmin + span * tbar);
    }
    store_v<V>(zhat, i, out);
}

hipError_t launch_predict(const double* acc, const float* z, const uint8_t* mask, int64_t n, int64_t n_samples,
                          const double* range, float* zhat, hipStream_t s)
{
    if (aligned4(n, acc, z, mask, static_cast<const float*>(zhat)))
        hipLaunchKernelGGL(k_predict<4>, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, acc, z, mask, n,
                           n_samples, range, zhat);
    else
        hipLaunchKernelGGL(k_predict<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, acc, z, mask, n, n_samples,
                           range, zhat);
    return hipGetLastError();
}

constexpr int VAL_NT = 256;

int validate_blocks(int64_t n)
{
    int64_t b = (n + VAL_NT * 16 - 1) / (VAL_NT * 16);
    return (int)(b < 1 ? 1 : (b > 2048 ? 2048 : b));
}

template <int V>
__global__ __launch_bounds__(VAL_NT) void k_validate_part(const float* __restrict__ zhat,
                                                           const float* __restrict__ truth,
                                                           const uint8_t* __restrict__ ev, int64_t n, double* part)
{
    __shared__ double s_red[VAL_NT / 64];
    double sa = 0.0, s2 = 0.0, cnt = 0.0;
    for (int64_t i = ((int64_t)blockIdx.x * VAL_NT + threadIdx.x) * V; i < n; i += (int64_t)gridDim.x * VAL_NT * V) {
        uint8_t m[V];
        float a[V], b[V];
        load_v<V>(ev, i, m);
        load_v<V>(truth, i, a);
        load_v<V>(zhat, i, b);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (!m[k]) continue;
            const double e = (double)a[k] - (double)b[k];
            sa += fabs(e);
            s2 += e * e;
            cnt += 1.0;
        }
    }
    sa = block_sum<VAL_NT>(sa, s_red);
    s2 = block_sum<VAL_NT>(s2, s_red);
    cnt = block_sum<VAL_NT>(cnt, s_red);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x + 0] = sa;
        part[3 * blockIdx.x + 1] = s2;
        part[3 * blockIdx.x + 2] = cnt;
    }
}

// The partial sums by a whole workgroup (2048 of them: 4.7 us, and 221 us when one thread read them in turn).
__global__ __launch_bounds__(VAL_NT) void k_validate_final(const double* part, int nblocks, double* out)
{
    __shared__ double s_red[VAL_NT / 64];
    double sa = 0.0, s2 = 0.0, cnt = 0.0;
    for (int i = (int)threadIdx.x; i < nblocks; i += VAL_NT) {
        sa += part[3 * i];
        s2 += part[3 * i + 1];
        cnt += part[3 * i + 2];
    }
    sa = block_sum<VAL_NT>(sa, s_red);
    s2 = block_sum<VAL_NT>(s2, s_red);
    cnt = block_sum<VAL_NT>(cnt, s_red);
    if (threadIdx.x != 0) return;
    out[0] = cnt > 0.0 ? sa / cnt : 0.0;
    out[1] = cnt > 0.0 ? sqrt(s2 / cnt) : 0.0;
}

hipError_t launch_validate(const float* zhat, const float* truth, const uint8_t* ev, int64_t n, double* part,
                           int nblocks, double* out, hipStream_t s)
{
    if (aligned4(n, zhat, truth, ev))
        hipLaunchKernelGGL(k_validate_part<4>, dim3(nblocks), dim3(VAL_NT), 0, s, zhat, truth, ev, n, part);
    else
        hipLaunchKernelGGL(k_validate_part<1>, dim3(nblocks), dim3(VAL_NT), 0, s, zhat, truth, ev, n, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_validate_final, dim3(1), dim3(VAL_NT), 0, s, part, nblocks, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Matching curve: the unconditional MPR model on a periodic L x L lattice, one chain per temperature.
// ------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ref_fill(float* state, int64_t n, float v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) state[i] = v;
}

hipError_t launch_ref_fill(float* state, int64_t n, float v, hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, state, n, v);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_ref_half(RefArgs a)
{
    const int chain = blockIdx.y;
    const int p = blockIdx.x * 256 + threadIdx.x;
    const int L = a.L;
    if (p >= L * a.Mw) return;
    const int y = p / a.Mw, m = p - y * a.Mw;
    const int xa = 4 * m + ((y + a.colour) & 1);
    if (xa >= L) return;
    float* st = a.state + (int64_t)chain * L * L;
    const float T = a.Tgrid[chain];
    const TBand tb = make_tband(T, 1.0f, a.delta_e);
    const U4 w = philox_x3((uint32_t)p, a.sweep, (uint32_t)chain, ctr_word3(0u, TAG_REFLAT, a.colour), a.key0,
                               a.key1);
    const int yu = (y + L - 1) % L, yd = (y + 1) % L;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int x = xa + 2 * h;
        if (x >= L) break;
        const int xl = (x + L - 1) % L, xr = (x + 1) % L;
        float nb[4];
        nb[0] = st[yu * L + x];
        nb[1] = st[y * L + xl];
        nb[2] = st[y * L + xr];
        nb[3] = st[yd * L + x];
        float Cx = 0.0f, Sy = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float ang = a.q * nb[j];
            Cx += cos_rev(ang);
            Sy += sin_rev(ang);
        }
        const float to = st[y * L + x];
        const float co = cos_rev(a.q * to), so = sin_rev(a.q * to);
        const float tpv = u24(h ? w.z : w.x);
        const uint32_t wa = h ? w.w : w.y;
        const float u2 = u24(wa);
        const float cp = cos_rev(a.q * tpv), sp = sin_rev(a.q * tpv);
        const float X = fmaf(cp - co, Cx, (sp - so) * Sy);
        int dec = filter32(X, (float)(wa >> 8), tb, 1.0f, a.delta_e);
        if (dec < 0) dec = exact64(tpv, to, nb[0], nb[1], nb[2], nb[3], 15u, a.two_pi_q, 1.0, T, u2) ? 1 : 0;
        if (dec) st[y * L + x] = tpv;
    }
}

hipError_t launch_ref_half(const RefArgs& a, int nT, hipStream_t s)
{
    const int np = a.L * a.Mw;
    hipLaunchKernelGGL(k_ref_half, dim3((unsigned)((np + 255) / 256), (unsigned)nT), dim3(256), 0, s, a);
    return hipGetLastError();
}

int ref_energy_parts(int L)
{
    const int64_t n = (int64_t)L * L;
    int64_t p = (n + 256 * 8 - 1) / (256 * 8);
    return (int)(p < 1 ? 1 : (p > 1024 ? 1024 : p));
}

__global__ __launch_bounds__(256) void k_ref_energy(const float* __restrict__ state, int L, float q, double* partial)
{
    __shared__ double s_red[4];
    const int chain = blockIdx.y;
    const float* st = state + (int64_t)chain * L * L;
    double acc = 0.0;
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < (int64_t)L * L; n += (int64_t)gridDim.x * 256) {
        const int y = (int)(n / L), x = (int)(n - (int64_t)y * L);
        const float tn = st[n];
        const float e = -cos_rev(q * (tn - st[y * L + (x + 1) % L])) - cos_rev(q * (tn - st[((y + 1) % L) * L + x]));
        acc += (double)e;
    }
    const double tot = block_sum<256>(acc, s_red);
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * gridDim.y + chain] = tot;
}

hipError_t launch_ref_energy(const float* state, int L, int nT, float q, double* partial, int nparts, hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_energy, dim3((unsigned)nparts, (unsigned)nT), dim3(256), 0, s, state, L, q, partial);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_ref_accumulate(const double* partial, int nparts, int nT, double inv_norm,
                                                         double* e_sum, int first)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nT) return;
    double s = 0.0;
    for (int p = 0; p < nparts; ++p) s += partial[(int64_t)p * nT + i];
    const double e = s * inv_norm;
    e_sum[i] = first ? e : e_sum[i] + e;
}

hipError_t launch_ref_accumulate(const double* partial, int nparts, int nT, double inv_norm, double* e_sum, int first,
                                 hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_accumulate, dim3((unsigned)((nT + 255) / 256)), dim3(256), 0, s, partial, nparts, nT,
                       inv_norm, e_sum, first);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_ref_finish(const double* e_sum, int nT, double n_meas, double* e_out)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nT) return;
    e_out[i] = n_meas > 0.0 ? e_sum[i] / n_meas : 0.0;
}

hipError_t launch_ref_finish(const double* e_sum, int nT, double n_meas, double* e_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_finish, dim3((unsigned)((nT + 255) / 256)), dim3(256), 0, s, e_sum, nT, n_meas, e_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Sec. 2.2.3 (SST): the block map spread to the sites, then n_s passes of the mean over the (2 r_s + 1)^2 square
// around each site cut at the grid edges, in FP64 with the window summed row by row from the top left (the oracle's
// order), one rounding to FP32 at the end.
__global__ __launch_bounds__(256) void k_sst_spread(const float* T_blocks, int64_t H, int64_t W, int32_t lb_h,
                                                    int32_t lb_w, double* a)
{
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= H * W) return;
    const int64_t y = n / W, x = n - y * W, nbx = (W + lb_w - 1) / lb_w;
    a[n] = (double)T_blocks[(y / lb_h) * nbx + (x / lb_w)];
}

__global__ __launch_bounds__(256) void k_sst_pass(const double* __restrict__ a, double* __restrict__ b, int64_t H,
                                                  int64_t W, int32_t r)
{
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= H * W) return;
    const int64_t y = n / W, x = n - y * W;
    double sum = 0.0;
    int64_t cnt = 0;
    for (int64_t yy = y - r; yy <= y + r; ++yy) {
        if (yy < 0 || yy >= H) continue;
        for (int64_t xx = x - r; xx <= x + r; ++xx) {
            if (xx < 0 || xx >= W) continue;
            sum += a[yy * W + xx];
            ++cnt;
        }
    }
    b[n] = sum / (double)cnt;
}

__global__ __launch_bounds__(256) void k_sst_round(const double* a, int64_t n, float* out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (float)a[i];
}

// The passes of radius 1 and 2 fused: a workgroup loads a 64 x 32 tile with a ring of passes x R sites, straight from the
// block map in the first launch, runs the passes in LDS on a region that shrinks by R a pass, and writes the tile, as FP32
// after the last pass.  A thread makes four sites of a column from one walk down the rows, so each value is read from LDS
// once per column offset instead of once per window.  The sums keep the order of k_sst_pass (a site outside the grid
// adds 0).  4096^2, 32 x 32 blocks, five passes of radius 1:
// 648 us as seven kernels over two FP64 planes (0.27 GB a pass), 217 us fused (radius 2, five passes: 1222 / 335 us);
// bound by the LDS reads and FP64 additions and the barrier of each pass (256 / 384 / 768 threads: 272 / 399 / 226 us).
constexpr int kSstW = 64, kSstH = 32, kSstRing = 6, kSstNT = 512;
constexpr int kSstStride = kSstW + 2 * kSstRing + 1;

template <int R>
__global__ __launch_bounds__(kSstNT) void k_sst_fused(const float* __restrict__ T_blocks,
                                                      const double* __restrict__ in, int H, int W, int lb_h, int lb_w,
                                                      int passes, double* __restrict__ out, float* __restrict__ out32)
{
    constexpr int K = 4, N1 = 2 * R + 1;
    // (a column's last four sites may reach past the region: those rows are read and not used)
    __shared__ double buf[2][(kSstH + 2 * kSstRing + K) * kSstStride];
    const int ring = passes * R;
    const int rw = kSstW + 2 * ring, rh = kSstH + 2 * ring;
    const int ntx = (W + kSstW - 1) / kSstW;
    const int x0 = (int)(blockIdx.x % (unsigned)ntx) * kSstW - ring, y0 = (int)(blockIdx.x / (unsigned)ntx) * kSstH - ring;
    const int nbx = (W + lb_w - 1) / lb_w;
    for (int i = threadIdx.x; i < rw * rh; i += kSstNT) {
        const int ry = i / rw, rx = i - ry * rw, y = y0 + ry, x = x0 + rx;
        double v = 0.0;
        if (y >= 0 && y < H && x >= 0 && x < W)
            v = in ? in[(int64_t)y * W + x] : (double)T_blocks[(int64_t)(y / lb_h) * nbx + x / lb_w];
        buf[0][ry * kSstStride + rx] = v;
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p) {
        const double* const a = buf[p & 1];
        double* const b = buf[(p & 1) ^ 1];
        const int lo = (p + 1) * R, pw = rw - 2 * lo, ph = rh - 2 * lo;     // the region after this pass
        const unsigned inv = 65536u / (unsigned)pw + 1u;     // i / pw for i < 65536 / pw (at most 11 groups of columns)
        for (int i = threadIdx.x; i < pw * ((ph + K - 1) / K); i += kSstNT) {
            const int g = (int)(((unsigned)i * inv) >> 16), rx = lo + i - g * pw, ry = lo + g * K, x = x0 + rx;
            double v[K + 2 * R][2 * R + 1];
#pragma unroll
            for (int k = 0; k < K + 2 * R; ++k)
#pragma unroll
                for (int d = 0; d <= 2 * R; ++d)
                    v[k][d] = a[(ry - R + k) * kSstStride + rx - R + d];
            const int nx = (x + R < W - 1 ? x + R : W - 1) - (x - R > 0 ? x - R : 0) + 1;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                double sum = 0.0;
#pragma unroll
                for (int e = 0; e <= 2 * R; ++e)
#pragma unroll
                    for (int d = 0; d <= 2 * R; ++d) sum += v[k + e][d];
                const int y = y0 + ry + k;
                const int ny = (y + R < H - 1 ? y + R : H - 1) - (y - R > 0 ? y - R : 0) + 1;
                double m;
                if (nx == N1 && ny == N1) {
                    // the correctly rounded quotient: one Newton step on sum times the correctly rounded reciprocal
                    // (an infinite or NaN sum is its own quotient)
                    const double q = sum * (1.0 / (N1 * N1));
                    m = fma(fma(-(double)(N1 * N1), q, sum), 1.0 / (N1 * N1), q);
                    if (!(fabs(sum) < INFINITY)) m = sum;
                } else {
                    m = sum / (double)(ny * nx);
                }
                if (ry + k < lo + ph) b[(ry + k) * kSstStride + rx] = y >= 0 && y < H && x >= 0 && x < W ? m : 0.0;
            }
        }
        __syncthreads();
    }
    const double* const r = buf[passes & 1];
    for (int i = threadIdx.x; i < kSstW * kSstH; i += kSstNT) {
        const int ry = i / kSstW, rx = i % kSstW, y = y0 + ring + ry, x = x0 + ring + rx;
        if (y >= H || x >= W) continue;
        const double v = r[(ring + ry) * kSstStride + ring + rx];
        if (out32) out32[(int64_t)y * W + x] = (float)v;
        else out[(int64_t)y * W + x] = v;
    }
}

hipError_t launch_sst(const float* T_blocks, int64_t H, int64_t W, int32_t lb_h, int32_t lb_w, int32_t r_s,
                      int32_t n_s, double* a, double* b, float* out, hipStream_t s)
{
    // fused: windows whose ring fits the LDS, on tiles three eighths full (radius 2: a quarter), or all in one round (two a CU).
    // Emptier tiles cost the same each.  Five passes of radius 1, fused / a pass per launch: 1 x 2^20 sites 418 / 41 us,
    // 3 x 300001 127 / 63, 100001 x 20 98 / 98 (radius 2: 146 / 182).
    const int64_t ntiles = ((W + kSstW - 1) / kSstW) * ((H + kSstH - 1) / kSstH);
    if (n_s > 0 && (r_s == 1 || r_s == 2) && (ntiles <= 512 || H * W * 8 >= (r_s == 1 ? 3 : 2) * ntiles * kSstW * kSstH)) {
        const dim3 tiles((unsigned)ntiles);
        const double* in = nullptr;
        for (int32_t done = 0; done < n_s;) {
            const int p = n_s - done < kSstRing / r_s ? n_s - done : kSstRing / r_s;
            done += p;
            float* const o32 = done == n_s ? out : nullptr;
            if (r_s == 1)
                hipLaunchKernelGGL(k_sst_fused<1>, tiles, dim3(kSstNT), 0, s, T_blocks, in, (int)H, (int)W, lb_h, lb_w, p,
                                   a, o32);
            else
                hipLaunchKernelGGL(k_sst_fused<2>, tiles, dim3(kSstNT), 0, s, T_blocks, in, (int)H, (int)W, lb_h, lb_w, p,
                                   a, o32);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            in = a;
            a = b;
            b = const_cast<double*>(in);
        }
        return hipSuccess;
    }
    const int64_t n = H * W;
    const dim3 grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(k_sst_spread, grid, dim3(256), 0, s, T_blocks, H, W, lb_h, lb_w, a);
    hipError_t e = hipGetLastError();
    for (int32_t p = 0; p < n_s && e == hipSuccess; ++p) {
        hipLaunchKernelGGL(k_sst_pass, grid, dim3(256), 0, s, a, b, H, W, r_s);
        e = hipGetLastError();
        double* tmp = a;
        a = b;
        b = tmp;
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sst_round, grid, dim3(256), 0, s, a, n, out);
    return hipGetLastError();
}

}  // namespace mpr
