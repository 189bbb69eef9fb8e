// Double-checkerboard sweep (Sec. 2.2.2): the grid divided into the lb_h x lb_w blocks, coloured like a
// checkerboard by (block row + block column) % 2; one sweep = four in-place phases: colour 0 then colour 1 inside
// the even blocks, then the same inside the odd blocks.  Sites of one phase share no bond, so each phase updates
// the state in place.  The unit is a row pair of same-colour sites two columns apart (one Philox block, words 0-1 for the
// first site and 2-3 for the second, the counter of the single-checkerboard order); the (cos, sin) of the neighbours are
// computed from the stored angles; the decision is the FP32 filter with the exact FP64 test inside its error band, as in
// the other sweeps.
//
// The pairs of a phase depend on the mask and the blocks alone: their lists are built once per call, so that every lane of a
// phase has an update (a thread per pair of the grid idled on samples and on the blocks of the other parity, and paid five
// 64-bit divisions for each).  A thread decodes its pair once for several realizations.  700 x 900, R = 30, 16 x 16 blocks:
// 215 us per sweep with its energy, 270 us before; bound by the cache lines that four passes over the state touch.
#include <hip/hip_runtime.h>

#include "dc.hpp"
#include "exact_lane.hpp"
#include "metropolis.hpp"

namespace mpr {

namespace {

constexpr int kPlanNT = 1024;

__global__ __launch_bounds__(64) void k_dc_plan_clear(uint32_t* count)
{
    if (threadIdx.x < 8) count[threadIdx.x] = 0u;
}

// One thread per pair and colour.  A code is pair << 2 | its free sites of the phase.
__global__ __launch_bounds__(kPlanNT) void k_dc_plan(DcArgs a)
{
    constexpr int kWaves = kPlanNT / 64;
    __shared__ uint32_t base[4][kWaves];         // (parity, single) x wave: entries, then the wave's first
    const uint32_t p = blockIdx.x * (uint32_t)kPlanNT + threadIdx.x;
    const int colour = (int)blockIdx.y, wave = (int)(threadIdx.x >> 6);
    unsigned sm[2] = {0u, 0u};
    if ((int64_t)p < a.plan.cap) {
        const uint32_t y = p / (uint32_t)a.Mw, m = p - y * (uint32_t)a.Mw, by = y / (uint32_t)a.lb_h;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t x = 4 * m + ((y + (uint32_t)colour) & 1u) + 2 * h;
            if ((int64_t)x >= a.W || a.mask[(int64_t)y * a.W + x]) continue;
            sm[(by + x / (uint32_t)a.lb_w) & 1u] |= 1u << h;
        }
    }
    unsigned long long in[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const unsigned s = sm[c >> 1];
        in[c] = __ballot((c & 1) ? s == 1u || s == 2u : s == 3u);
        if ((threadIdx.x & 63u) == 0) base[c][wave] = (uint32_t)__popcll(in[c]);
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int c = (int)threadIdx.x;
        uint32_t sum = 0;
        for (int w = 0; w < kWaves; ++w) sum += base[c][w];
        uint32_t at = sum ? atomicAdd(&a.plan.count[(((c >> 1) * 2 + colour) << 1) + (c & 1)], sum) : 0u;
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t n = base[c][w];
            base[c][w] = at;
            at += n;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const unsigned s = sm[c >> 1];
        if (!((c & 1) ? s == 1u || s == 2u : s == 3u)) continue;
        const uint32_t i = base[c][wave] + __builtin_amdgcn_mbcnt_hi((uint32_t)(in[c] >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)in[c], 0));
        uint32_t* const list = a.plan.list + ((c >> 1) * 2 + colour) * a.plan.cap;
        list[(c & 1) ? a.plan.cap - 1 - i : (int64_t)i] = p << 2 | s;
    }
}

struct Cs {
    float t, c, s;
};

// One update: own angle `to`, neighbours in the order up, left, right, down with `present`.
__device__ __forceinline__ bool decide(const DcArgs& a, const TBand& tb, float to, const Cs& u, const Cs& l, const Cs& r,
                                       const Cs& d, unsigned present, float tp, uint32_t wa)
{
    const float Cx = ((u.c + l.c) + r.c) + d.c, Sy = ((u.s + l.s) + r.s) + d.s;
    const float ui = (float)(wa >> 8);
    const float cp = cos_rev(a.q * tp), sp = sin_rev(a.q * tp);
    const float co = cos_rev(a.q * to), so = sin_rev(a.q * to);
    const float X = fmaf(cp - co, Cx, (sp - so) * Sy);
    int dec = filter32(X, ui, tb, a.J, a.delta_e);
    // A wave full of updates mostly has one open decision or none: its cosines by eight lanes (256 x 256, R = 10, 20 sweeps
    // at 95 % gaps: 926 -> 851 us; 876 when half of a wave's lanes had no update and fewer waves waited for one)
    unsigned long long left = __ballot(dec < 0);
    if (left == 0) return dec > 0;
    const float u2 = ui * 5.9604644775390625e-8f;
    if (__popcll(__ballot(1)) >= 8 && __popcll(left) <= 4) {
        do {
            const int src = __ffsll((long long)left) - 1;
            left &= left - 1;
            const bool acc = exact_of_lane(src, tp, to, u.t, l.t, r.t, d.t, present, a.two_pi_q, a.Jd, tb.T, u2);
            if (((int)threadIdx.x & 63) == src) dec = acc ? 1 : 0;
        } while (left != 0);
    } else if (dec < 0) {
        dec = exact64(tp, to, u.t, l.t, r.t, d.t, present, a.two_pi_q, a.Jd, tb.T, u2) ? 1 : 0;
    }
    return dec > 0;
}

__global__ __launch_bounds__(256) void k_dc_phase(DcArgs a, uint32_t sweep, int colour, int phase, int rchunk)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x, both = a.plan.count[2 * phase], one = a.plan.count[2 * phase + 1];
    if (i >= both + one) return;
    const uint32_t* const list = a.plan.list + phase * a.plan.cap;
    const uint32_t code = i < both ? list[i] : list[a.plan.cap - 1 - (int64_t)(i - both)];
    const uint32_t p = code >> 2, y = p / (uint32_t)a.Mw, m = p - y * (uint32_t)a.Mw;
    const bool two = i < both, second = !two && (code & 2u);       // (second: the pair's second site alone)
    const uint32_t x = 4 * m + ((y + (uint32_t)colour) & 1u) + (second ? 2u : 0u), W = (uint32_t)a.W;
    const uint32_t n = y * W + x;                                  // H W < 2^31
    const TBand* const trow = a.tb + (int64_t)(y / (uint32_t)a.tb_h) * a.nbx_t;
    const TBand t0 = trow[x / (uint32_t)a.tb_w], t1 = two ? trow[(x + 2) / (uint32_t)a.tb_w] : t0;
    const bool pu = y > 0, pd = y + 1 < (uint32_t)a.H, pl = x > 0, pr = x + 1 < W, pr1 = x + 3 < W;
    const unsigned vert = (pu ? 1u : 0u) | (pd ? 8u : 0u);
    const uint32_t w3 = ctr_word3(a.scene, TAG_SWEEP, (uint32_t)colour);
    const int r0 = (int)blockIdx.y * rchunk, r1 = r0 + rchunk < a.R ? r0 + rchunk : a.R;
    // the angles of a realization: up, left, middle, down, own of the first site; up, right, down, own of the second.  Those of
    // the next realization are requested before this one's updates (other memory), a neighbour outside the grid reads the site.
    const uint32_t at[9] = {pu ? n - W : n,             pl ? n - 1 : n, pr ? n + 1 : n, pd ? n + W : n, n,
                            two && pu ? n + 2 - W : n, two && pr1 ? n + 3 : n, two && pd ? n + 2 + W : n, two ? n + 2 : n};
    float next[9];
    auto load = [&](int r) {
        const float* const st = a.state + (int64_t)r * a.H * a.W;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if (k < 5 || two) next[k] = st[at[k]];
    };
    load(r0);
    for (int r = r0; r < r1; ++r) {
        float v[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) v[k] = next[k];
        if (r + 1 < r1) load(r + 1);
        float* const st = a.state + (int64_t)r * a.H * a.W;
        auto field = [&](bool there, float t) {
            return there ? Cs{t, cos_rev(a.q * t), sin_rev(a.q * t)} : Cs{0.0f, 0.0f, 0.0f};
        };
        const U4 w = philox_x3(p, sweep, a.real_offset + (uint32_t)r, w3, a.key0, a.key1);
        const Cs mid = field(pr, v[2]);
        const float tp = u24(second ? w.z : w.x);
        if (decide(a, t0, v[4], field(pu, v[0]), field(pl, v[1]), mid, field(pd, v[3]), vert | (pl ? 2u : 0u) | (pr ? 4u : 0u),
                   tp, second ? w.w : w.y))
            st[n] = tp;
        if (two) {
            const float tp1 = u24(w.z);
            if (decide(a, t1, v[8], field(pu, v[5]), mid, field(pr1, v[6]), field(pd, v[7]), vert | 2u | (pr1 ? 4u : 0u), tp1,
                       w.w))
                st[n + 2] = tp1;
        }
    }
}

}  // namespace

hipError_t launch_dc_plan(const DcArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_dc_plan_clear, dim3(1), dim3(64), 0, s, a.plan.count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dc_plan, dim3((unsigned)((a.plan.cap + kPlanNT - 1) / kPlanNT), 2), dim3(kPlanNT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dc_sweep(const DcArgs& a, uint32_t sweep, hipStream_t s)
{
    // the number of entries is on the device: the grid covers all pairs, workgroups past the lists leave at once.  Up to
    // eight realizations a thread while about two rounds of threads are left (at most half the pairs are in a phase's list).
    const int64_t rc = a.plan.cap / 2 * a.R / (256 * 2048);
    const int rchunk = (int)(rc < 1 ? 1 : rc > 8 ? 8 : rc);
    const dim3 grid((unsigned)((a.plan.cap + 255) / 256), (unsigned)((a.R + rchunk - 1) / rchunk));
    for (int phase = 0; phase < 4; ++phase) {
        hipLaunchKernelGGL(k_dc_phase, grid, dim3(256), 0, s, a, sweep, phase & 1, phase, rchunk);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace mpr
