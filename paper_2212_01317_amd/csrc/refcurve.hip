// The matching curve's unconditional chains (Sec. 2.1: every site free, periodic, J = 1, one chain per temperature), with
// several sweeps per launch on a lattice, or a strip of it, that stays in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "metropolis.hpp"
#include "refcurve.hpp"

namespace mpr {

namespace {

constexpr int kRefMaxNT = 1024;
constexpr int kRefQueue = 8;                   // undecided updates that a wave settles at once (3D: the first four)
constexpr int kRefQueueWords = kRefMaxNT / 64 * kRefQueue;
constexpr int kRefSteps = 16;                  // unit steps of a half-sweep at most: two bits each of a thread's open updates
// words left for the lattice beside the queue and the sums, of 160 KB, and with two and four workgroups on a core
constexpr int kRefLds = 40960 - 32 - kRefQueueWords;
constexpr int kRefLdsHalf = 20480 - 32 - kRefQueueWords, kRefLdsSmall = 10240 - 32 - kRefQueueWords;

template <class T>
__device__ __forceinline__ T wave_total(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// What the updates of one colour need besides the lattice.
struct RefHalf {
    int L, per_step, units, base, b0, colour;
    bool whole;
    uint32_t sweep, chain, key0, key1;
    float q, T;
    double two_pi_q;
};

// The updates that the FP32 test left open: bit 2 i + h of `left` is site h of the thread's i-th unit.  Each round takes one of
// every thread that has any, eight (3D: four) threads a pass, and eight (sixteen) lanes form the FP64 cosines of one update.
// Not inlined: its registers are then not the sweep's.
template <int DIM>
__device__ __noinline__ void ref_settle(uint32_t left, RefHalf a, float* t, float2* f, uint32_t* q)
{
    constexpr int NB = 2 * DIM, TL = DIM == 2 ? 8 : 16;
    const int L = a.L, Mw = (L + 3) / 4, RS = 4 * Mw, PU = DIM == 2 ? Mw : L * Mw, US = 4 * PU;
    const int lane = (int)(threadIdx.x & 63u), term = lane % TL, nb = min(term >> 1, NB - 1);
    auto col = [&](int x) { return (x & 3) * Mw + (x >> 2); };
    for (;;) {
        const unsigned long long open = __ballot(left != 0);
        if (open == 0) break;
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(open >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)open, 0));
        const int n = min(__popcll(open), 64 / TL);
        if (left != 0 && rank < n) {
            const int bit = __ffs((int)left) - 1;
            q[rank] = threadIdx.x | (uint32_t)bit << 16;
            left &= left - 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int item = lane / TL;
        const uint32_t code = q[min(item, n - 1)];
        const int tid = (int)(code & 0xffffu), bit = (int)(code >> 16);
        const int first = tid / PU, in_unit = tid - first * PU, y = DIM == 2 ? 0 : in_unit / Mw, m = in_unit - y * Mw;
        const int u = a.b0 + first + (bit >> 1) * a.per_step, g = (a.base + u) % L;
        const U4 w = philox4x32_10((uint32_t)(g * PU + in_unit), a.sweep, a.chain, ctr_word3(0u, TAG_REFLAT, (uint32_t)a.colour),
                                   a.key0, a.key1);
        const int x = 4 * m + ((g + y + a.colour) & 1) + 2 * (bit & 1);
        const float tp = u24(bit & 1 ? w.z : w.x), u2 = u24(bit & 1 ? w.w : w.y);
        int un = u, yn = y, xn = x;            // the term's neighbour: back, up, left, right, down, front
        if (nb == 0) un = a.whole && u == 0 ? L - 1 : u - 1;
        else if (nb == NB - 1) un = a.whole && u == L - 1 ? 0 : u + 1;
        else if (nb == DIM - 1) xn = x == 0 ? L - 1 : x - 1;
        else if (nb == DIM) xn = x == L - 1 ? 0 : x + 1;
        else if (nb == 1) yn = y == 0 ? L - 1 : y - 1;
        else yn = y == L - 1 ? 0 : y + 1;
        const int c = u * US + y * RS + col(x);
        const double cs = cos(a.two_pi_q * ((double)(term & 1 ? t[c] : tp) - (double)t[un * US + yn * RS + col(xn)]));
        const double d = cs - __shfl_xor(cs, 1, 64);                   // even lanes: proposed less present
        double sum = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) sum += __shfl(d, item * TL + 2 * j, 64);
        const double dE = -1.0 * sum;
        const bool accept = (double)a.T > 0.0 ? (double)u2 < exp(-dE / (double)a.T) : dE <= 0.0;
        if (accept && term == 0 && item < n) {
            t[c] = tp;
            if (f) f[c] = make_float2(cos_rev(a.q * tp), sin_rev(a.q * tp));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();       // the queue is read before the next round writes it
    }
}

// A workgroup advances one strip of one chain.  The unit is a row (2D) or a plane (3D).  The strip's units are in LDS with a
// ring of 2 ns units before and 2 ns + 1 behind, the last for the bonds of the strip's last unit; each half-sweep spoils the
// outermost unit on each side, and the next is made one unit less wide.  One strip per chain needs no ring and any number of
// sweeps.
//
// A row is held as its columns of the four residues mod 4, one after another: the two sites of a Philox pair have the same
// two residues in every lane of a row, so that lanes read consecutive words.  A thread keeps its place in the unit and steps
// over an even number of units, which keeps its colour's columns too: the loop is Philox, the field and the test, and bound by
// their instructions.  With FIELD the cosine and sine of every angle are held next to it, written when an update is accepted,
// instead of formed for each of its neighbours.
//
// The updates that the FP32 test leaves open wait until the wave's units are done (updates of one colour do not see each
// other): a call per update made the waves of a workgroup wait for one lane's FP64 functions several times a half-sweep.
//
// 121 chains of 128 x 128, 450 sweeps (300 measured): 11.5 ms with two launches a sweep and two more for its energies, 4.7 ms;
// a pair takes about 1000 cycles of a SIMD's issue, a third of it Philox, at four waves.
template <int DIM, bool FIELD, int WORDS>
__global__ __launch_bounds__(kRefMaxNT) void k_ref_sweeps(RefSweepArgs a, int strips, int per_step)
{
    constexpr int NB = 2 * DIM;                // neighbours
    __shared__ __attribute__((aligned(16))) float lds[WORDS];
    __shared__ uint32_t queue[kRefQueueWords];
    __shared__ double red[kRefMaxNT / 64];
    const int L = a.L, Mw = (L + 3) / 4, RS = 4 * Mw, NT = (int)blockDim.x, tid = (int)threadIdx.x, lane = tid & 63;
    const int PU = DIM == 2 ? Mw : L * Mw, US = 4 * PU;      // pairs and LDS words of a unit
    const int chain = (int)blockIdx.x / strips, strip = (int)blockIdx.x - chain * strips;
    const bool whole = strips == 1;
    const int u0 = (int)((int64_t)strip * L / strips), own = (int)((int64_t)(strip + 1) * L / strips) - u0;
    const int ring = whole ? 0 : 2 * a.ns;
    const int units = own + (whole ? 0 : 2 * ring + 1);
    int base = (u0 - ring) % L;                // the lattice unit of LDS unit 0
    if (base < 0) base += L;
    float* const t = lds;
    float2* const f = reinterpret_cast<float2*>(lds + units * US);     // US is a multiple of four
    uint32_t* const q = queue + __builtin_amdgcn_readfirstlane(tid >> 6) * kRefQueue;

    // the thread's place: unit `first` of each step, row y of it (3D), columns 4 m .. 4 m + 3
    const int first = tid / PU, in_unit = tid - first * PU;
    const int y = DIM == 2 ? 0 : in_unit / Mw, m = in_unit - y * Mw;
    const bool active = first < per_step;
    const int row = y * RS;
    const int row_u = DIM == 2 ? 0 : (y == 0 ? L - 1 : y - 1) * RS, row_d = DIM == 2 ? 0 : (y == L - 1 ? 0 : y + 1) * RS;
    auto col = [&](int x) { return (x & 3) * Mw + (x >> 2); };
    const int64_t n_chain = (int64_t)L * L * (DIM == 3 ? L : 1), n_unit = DIM == 2 ? L : L * L;

    if (active) {
        const float* src = a.src ? a.src + chain * n_chain + y * L : nullptr;
        for (int u = first; u < units; u += per_step) {
            const int g = (base + u) % L;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int x = 4 * m + r;
                if (x >= L) break;
                const float v = src ? src[g * n_unit + x] : 0.5f;
                const int o = u * US + row + r * Mw + m;
                t[o] = v;
                if (FIELD) f[o] = make_float2(cos_rev(a.q * v), sin_rev(a.q * v));
            }
        }
    }
    __syncthreads();

    const TBand tb = make_tband(a.Tgrid[chain], 1.0f, a.delta_e);
    const int step_mod = per_step % L;
    double acc = 0.0;
    for (int k = 0; k < a.ns; ++k) {
        const uint32_t sweep = a.sweep + (uint32_t)k;
        for (int colour = 0; colour < 2; ++colour) {
            const int step = 2 * k + colour, b0 = whole ? 0 : 1 + step, b1 = whole ? units : units - 1 - step;
            int u = b0 + first;
            int g = (base + u) % L;
            const int x0 = 4 * m + ((g + y + colour) & 1);
            uint32_t left = 0, bit = 1;
            if (active) {
                // columns of the pair and of the sites beside and between (x0 < L, as L is even)
                const bool second = x0 + 2 < L;
                const int c0 = row + col(x0), c1 = second ? row + col(x0 + 2) : c0;
                const int x_l = row + col(x0 == 0 ? L - 1 : x0 - 1), x_m = row + col(x0 + 1 == L ? 0 : x0 + 1);
                const int x_r = second ? row + col(x0 + 3 == L ? 0 : x0 + 3) : x_m;
                for (; u < b1; u += per_step) {
                    const int o = u * US, o_p = whole && u == 0 ? (L - 1) * US : o - US;
                    const int o_n = whole && u == L - 1 ? 0 : o + US;
                    const U4 w = philox_x3((uint32_t)(g * PU + in_unit), sweep, (uint32_t)chain,
                                           ctr_word3(0u, TAG_REFLAT, (uint32_t)colour), a.key0, a.key1);
                    g += step_mod;
                    if (g >= L) g -= L;
                    float Cx[2], Sy[2], co[2], so[2];
                    int at[2][NB];             // back, up, left, right, down, front: the order of the sums, exact test too
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int c = h ? c1 : c0;
                        at[h][0] = o_p + c;
                        if (DIM == 3) at[h][1] = o + c - row + row_u;
                        at[h][DIM - 1] = o + (h ? x_m : x_l);
                        at[h][DIM] = o + (h ? x_r : x_m);
                        if (DIM == 3) at[h][4] = o + c - row + row_d;
                        at[h][NB - 1] = o_n + c;
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int c = o + (h ? c1 : c0);
                        Cx[h] = Sy[h] = 0.0f;
#pragma unroll
                        for (int i = 0; i <= NB; ++i) {
                            const int p = i < NB ? at[h][i] : c;
                            float2 v;
                            if (FIELD) {
                                v = f[p];
                            } else {
                                const float an = a.q * t[p];
                                v = make_float2(cos_rev(an), sin_rev(an));
                            }
                            if (i < NB) {
                                Cx[h] += v.x;
                                Sy[h] += v.y;
                            } else {
                                co[h] = v.x;
                                so[h] = v.y;
                            }
                        }
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int c = o + (h ? c1 : c0);
                        const uint32_t wt = h ? w.z : w.x, wa = h ? w.w : w.y;
                        const float tp = u24(wt), an = a.q * tp;
                        const float cp = cos_rev(an), sp = sin_rev(an);
                        const float X = fmaf(cp - co[h], Cx[h], (sp - so[h]) * Sy[h]);
                        int dec = filter32(X, (float)(wa >> 8), tb, 1.0f, a.delta_e);
                        if (h && !second) dec = 0;
                        if (dec < 0) left |= bit << h;
                        if (dec > 0) {
                            t[c] = tp;
                            if (FIELD) f[c] = make_float2(cp, sp);
                        }
                    }
                    bit <<= 2;
                }
            }
            if (__ballot(left != 0) != 0)
                ref_settle<DIM>(left, RefHalf{L, per_step, units, base, b0, colour, whole, sweep, (uint32_t)chain, a.key0,
                                              a.key1, a.q, tb.T, a.two_pi_q}, t, FIELD ? f : nullptr, q);
            __syncthreads();
        }
        if (sweep > a.n_therm) {               // the bonds of the strip's sites to the right, down (and to the front)
            if (active) {
                for (int u = ring + first; u < ring + own; u += per_step) {
                    const int o = u * US + row + m, o_n = (whole && u == L - 1 ? 0 : (u + 1) * US) + row + m;
                    const int o_d = DIM == 2 ? o_n : u * US + row_d + m;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int x = 4 * m + r;
                        if (x >= L) break;
                        const float tn = t[o + r * Mw];
                        const float right = t[x == L - 1 ? u * US + row : r == 3 ? o + 1 : o + (r + 1) * Mw];
                        if (DIM == 2) {
                            const float e = -cos_rev(a.q * (tn - right)) - cos_rev(a.q * (tn - t[o_d + r * Mw]));
                            acc += (double)e;
                        } else {
                            acc -= (double)cos_rev(a.q * (tn - right));
                            acc -= (double)cos_rev(a.q * (tn - t[o_d + r * Mw]));
                            acc -= (double)cos_rev(a.q * (tn - t[o_n + r * Mw]));
                        }
                    }
                }
            }
            __syncthreads();
        }
    }

    if (active) {
        float* dst = a.dst + chain * n_chain + y * L;
        for (int u = ring + first; u < ring + own; u += per_step) {
            const int g = (base + u) % L;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * m + r < L) dst[g * n_unit + 4 * m + r] = t[u * US + row + r * Mw + m];
        }
    }
    if (a.sweep + (uint32_t)a.ns - 1u > a.n_therm) {
        acc = wave_total(acc);
        if (lane == 0) red[tid >> 6] = acc;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int w = 0; w < (NT >> 6); ++w) s += red[w];
            double* e = a.esum + blockIdx.x;
            *e = a.sweep <= a.n_therm + 1u ? s : *e + s;       // (this launch holds the first measured sweep)
        }
    }
}

__global__ __launch_bounds__(256) void k_ref_mean(const double* esum, int strips, int nT, double inv_norm, double n_meas,
                                                   double* e_out)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nT) return;
    double s = 0.0;
    for (int p = 0; p < strips; ++p) s += esum[(int64_t)i * strips + p];
    e_out[i] = s * inv_norm / n_meas;
}

// LDS words of a workgroup's units
int64_t ref_words(int dim, int L, int strips, int depth, bool field)
{
    const int64_t US = (int64_t)((L + 3) / 4 * 4) * (dim == 3 ? L : 1);
    const int64_t units = strips == 1 ? L : (L + strips - 1) / strips + 4 * depth + 1;
    return units * US * (field ? 3 : 1);
}

}  // namespace

// A half-sweep of one pair per thread and less is bound by latency: such chains stay whole (2D L = 64: 777 us for 150 sweeps of
// 121 chains, in two strips 835).  Otherwise as many strips as there are cores for them, as long as they are 16 rows or four
// planes: the ring is then at most as much again (L = 128, 121 chains: 1610 us in two strips of 8 sweeps a launch, 1730 of 4,
// four strips 1956, whole without the field 2352; 16 chains: 2336 whole, 1512, 1119, 964 in two, four and eight strips; 3D
// L = 32, 121 chains: 5440 whole, 4665 in two strips; 16 chains: 5434, 2287 in eight).  Launches of one half-sweep each:
// 3912 / 2352 us in 2D, 8723 / 4310 in 3D; they remain where no strip fits (L > 1024, 3D L > 44, states over 1 GiB).
RefPlan ref_plan(int dim, int L, int nT)
{
    RefPlan p{0, 0, 0, 0, true};
    auto fits = [&](int strips, int depth, bool field) {
        const int PU = (L + 3) / 4 * (dim == 3 ? L : 1);
        const int units = (L + strips - 1) / strips + (strips > 1 ? 4 * depth : 0);
        if (ref_words(dim, L, strips, depth, field) > kRefLds || 2 * PU > kRefMaxNT) return false;
        p.strips = strips;
        p.depth = depth;
        p.field = field;
        p.per_step = std::min(kRefMaxNT / PU, units + 1) & ~1;
        p.threads = (p.per_step * PU + 63) / 64 * 64;
        return units <= kRefSteps * p.per_step;
    };
    constexpr int kWhole = 64;                 // sweeps of a launch without a ring
    const int most = std::max(1, dim == 3 ? L / 4 : L / 16);
    const bool two_states = (int64_t)nT * L * L * (dim == 3 ? L : 1) <= (int64_t)1 << 28;
    for (int S = L <= (dim == 3 ? 20 : 64) ? 1 : std::max(1, std::min(256 / nT, most)); S <= most; ++S) {
        if (S == 1) {
            if (fits(1, kWhole, true) || fits(1, kWhole, false)) return p;
            continue;
        }
        if (!two_states) break;
        const int deep = dim == 3 ? 3 : std::max(4, std::min(8, L / S / 4)), least = dim == 3 ? 2 : 4;
        for (bool field : {true, false})
            if (fits(S, deep, field) || fits(S, least, field)) return p;
    }
    p.strips = 0;
    return p;
}

hipError_t launch_ref_sweeps(int dim, const RefPlan& p, const RefSweepArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)(a.nT * p.strips)), nt((unsigned)p.threads);
    const int64_t words = ref_words(dim, a.L, p.strips, p.depth, p.field);
#define MPR_REF(D, F, W) hipLaunchKernelGGL((k_ref_sweeps<D, F, W>), grid, nt, 0, s, a, p.strips, p.per_step)
#define MPR_REF_W(D, F)                                            \
    do {                                                           \
        if (words <= kRefLdsSmall) MPR_REF(D, F, kRefLdsSmall);    \
        else if (words <= kRefLdsHalf) MPR_REF(D, F, kRefLdsHalf); \
        else MPR_REF(D, F, kRefLds);                               \
    } while (0)
    if (dim == 3 && p.field) MPR_REF_W(3, true);
    else if (dim == 3) MPR_REF_W(3, false);
    else if (p.field) MPR_REF_W(2, true);
    else MPR_REF_W(2, false);
#undef MPR_REF_W
#undef MPR_REF
    return hipGetLastError();
}

hipError_t launch_ref_mean(const double* esum, int strips, int nT, double inv_norm, double n_meas, double* e_out,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_ref_mean, dim3((unsigned)((nT + 255) / 256)), dim3(256), 0, s, esum, strips, nT, inv_norm, n_meas,
                       e_out);
    return hipGetLastError();
}

}  // namespace mpr
