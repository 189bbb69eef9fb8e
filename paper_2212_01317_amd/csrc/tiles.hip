// Several red/black Metropolis sweeps of one tile in one launch (Sec. 2.2.2 single checkerboard), for runs with few
// realizations.  The update, its random numbers (keyed by site, sweep and realization) and its decision are those of
// every other sweep kernel, so the chains are the same bit for bit.
//
// A workgroup owns a 64 x 32 tile of one realization at a time.  It loads the tile and a ring of 2 kD sites (kD = the
// plan's depth) and runs up to kD sweeps on it without a word from the neighbouring tiles: a sweep's colour 1 needs
// colour 0 one site further out, and that the previous sweep one site further still, so the part of the region that
// holds the true state shrinks by two sites a sweep and is the tile itself after the last.  Sites of the ring are
// updated by every tile that needs them, with the same random numbers and inputs, hence to the same bits.
//
// Why: with few realizations a sweep is bound by what surrounds the updates, not by them.  One launch per sweep pays
// the launch, the staging of the tile (samples, lists, temperatures) and one pass over the state each time.  Here a
// launch pays them once for kD sweeps; the ring costs updates instead, of which the device has many to spare.
//
// The update lists depend on the mask alone and are built once per call (k_tile_plan): per tile and colour, the pairs
// (two same-colour sites four columns apart, one Philox block) with both sites free and the pairs with one, each
// sorted by the number of sweeps a site's ring distance still admits, so that sweep i of n takes a prefix of the list.
//
// LDS: per colour and row the cells of that colour are contiguous, so a pair's neighbourhood is five vector reads at
// immediate offsets of one index.  A cell that is not loaded (outside the grid, or beyond ring 2 ns) has (cos, sin) = (0, 0),
// which no angle has.  A pair stands in the bucket of the site that is needed longer, so its other site is updated once more
// than it is needed, from cells that may not be loaded; nothing that still matters reads it after that.
#include <hip/hip_runtime.h>

#include "exact_lane.hpp"
#include "metropolis.hpp"
#include "tiles.hpp"

namespace mpr {

namespace {

constexpr int kTW = 64;                // tile width
constexpr int kTH = 32;                // tile height
constexpr int kD = 5;                  // depth: sweeps a launch can run
constexpr int kNT = 512;               // threads of a sweep workgroup
constexpr int kTabCap = 128;           // temperature blocks a region may touch for the LDS table

struct Tl {
    static constexpr int HALO = 2 * kD;
    static constexpr int RH = kTH + 2 * HALO, RW = kTW + 2 * HALO;
    static constexpr int LEAD = 2 + (kD & 1);                // pairs start on an even cell: 16-byte reads
    static constexpr int CW = RW / 2 + 6;                   // cells per colour and row, pads included
    static constexpr int CELLS = RH * CW;                   // cells per colour
    static constexpr int GL = (HALO + 3) / 4;               // groups of four columns left of the tile
    static constexpr int NG = kTW / 4 + 2 * GL;
    static constexpr int CAP = (RH - 2) * NG;               // pairs of one colour
    static constexpr int ECAP = kTH * kTW / 2;
    static constexpr int CPT = (RH * RW + kNT - 1) / kNT;   // region cells per thread
    // plan of a tile, in 32-bit words: header, the two colours' lists (full pairs from the front, single sites from
    // the back), the colour-1 sample sites that border a gap (two per word)
    static constexpr int HDR = 32;
    static constexpr int WORDS = HDR + 2 * CAP + ECAP / 2;
    static_assert((kD + LEAD) % 2 == 0, "pair alignment");
    static_assert(CW % 2 == 0 && CELLS <= 4096 && RH <= 64, "code fields");
    static_assert(4 * kD + 3 <= HDR, "header");
};
// header words: [(colour * 2 + single) * kD + k] = entries of buckets 0 .. k; then the border samples, e_const (lo, hi)
// list code: bits 0-11 lowest cell read (of the pair or of the single site), 12-17 its row, 18-24 temperature-table
// entry, 25 (single) which site of the pair

struct TileBox {
    int tx0, ty0, by0, bx0, nby, nbx;
};

__device__ __forceinline__ TileBox tile_box(const TileArgs& a, int tile)
{
    using C = Tl;
    TileBox b;
    b.tx0 = (tile % a.ntx) * kTW;
    b.ty0 = (tile / a.ntx) * kTH;
    const int y0 = b.ty0 - C::HALO > 0 ? b.ty0 - C::HALO : 0, x0 = b.tx0 - C::HALO > 0 ? b.tx0 - C::HALO : 0;
    const int y1 = b.ty0 + kTH + C::HALO < a.H ? b.ty0 + kTH + C::HALO - 1 : a.H - 1;
    const int x1 = b.tx0 + kTW + C::HALO < a.W ? b.tx0 + kTW + C::HALO - 1 : a.W - 1;
    b.by0 = y0 / a.lb_h;
    b.bx0 = x0 / a.lb_w;
    b.nby = y1 / a.lb_h - b.by0 + 1;
    b.nbx = x1 / a.lb_w - b.bx0 + 1;
    return b;
}

// sites outside the tile, row plus column distance: the least number of colour phases before a site can reach the tile
__device__ __forceinline__ int ring(int yrel, int xrel)
{
    const int dy = yrel < 0 ? -yrel : (yrel >= kTH ? yrel - kTH + 1 : 0);
    const int dx = xrel < 0 ? -xrel : (xrel >= kTW ? xrel - kTW + 1 : 0);
    return dy + dx;
}

__device__ __forceinline__ int to_fix(float x) { return __float2int_rn(x * 16777216.0f); }
__device__ __forceinline__ bool here(float2 cs) { return cs.x != 0.0f || cs.y != 0.0f; }

// ---- the plan: one workgroup per tile ----
template <bool TABLE>
__device__ __forceinline__ void tile_plan(const TileArgs& a, int tile)
{
    using C = Tl;
    __shared__ uint8_t kind[C::RH * C::RW];        // 0 not loaded, 1 gap, 2 sample
    __shared__ int cnt[4 * kD], pos[4 * kD];
    __shared__ int n_border;
    __shared__ long long esum[4];
    const int tid = (int)threadIdx.x;
    const TileBox b = tile_box(a, tile);
    uint32_t* const plan = a.plan + (size_t)tile * C::WORDS;
    for (int i = tid; i < C::RH * C::RW; i += 256) {
        const int yl = i / C::RW, xl = i % C::RW;
        const int gy = b.ty0 - C::HALO + yl, gx = b.tx0 - C::HALO + xl;
        uint8_t k = 0;
        if (gy >= 0 && gy < a.H && gx >= 0 && gx < a.W && ring(yl - C::HALO, xl - C::HALO) <= C::HALO)
            k = a.mask[(int64_t)gy * a.W + gx] ? 2 : 1;
        kind[i] = k;
    }
    if (tid < 4 * kD) cnt[tid] = 0;
    if (tid == 0) n_border = 0;
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        for (int i = tid; i < 2 * C::CAP; i += 256) {
            const int colour = i >= C::CAP ? 1 : 0, ic = i - colour * C::CAP;
            const int yl = 1 + ic / C::NG, ml = ic % C::NG;
            const int delta = (yl + colour) & 1;
            unsigned sm = 0;
            int bucket = kD;
            for (int h = 0; h < 2; ++h) {
                const int xl = 4 * (ml - C::GL) + delta + 2 * h + C::HALO;
                if (xl < 0 || xl >= C::RW || kind[yl * C::RW + xl] != 1) continue;
                const int d = (ring(yl - C::HALO, xl - C::HALO) + colour) >> 1;   // sweeps that must follow
                if (d >= kD) continue;                                           // read only
                sm |= 1u << h;
                if (d < bucket) bucket = d;
            }
            if (!sm) continue;
            const int single = sm == 3u ? 0 : 1, slot = (colour * 2 + single) * kD + bucket;
            if (pass == 0) {
                atomicAdd(&cnt[slot], 1);
                continue;
            }
            const int h = sm == 2u ? 1 : 0;
            const int xl = 4 * (ml - C::GL) + delta + 2 * h + C::HALO;
            const int q = yl - colour;                                       // row of the lowest cell read
            const unsigned cell = (unsigned)(q * C::CW + (xl >> 1) + C::LEAD);
            unsigned tix = 0;
            if (TABLE)
                tix = (unsigned)(((b.ty0 - C::HALO + yl) / a.lb_h - b.by0) * b.nbx +
                                 ((b.tx0 - C::HALO + xl) / a.lb_w - b.bx0));
            const unsigned code = cell | (unsigned)q << 12 | tix << 18 | (single ? (unsigned)h << 25 : 0u);
            const int p = atomicAdd(&pos[slot], 1);
            plan[C::HDR + colour * C::CAP + (single ? C::CAP - 1 - p : p)] = code;
        }
        __syncthreads();
        if (pass == 0 && tid < 4) {
            int run = 0;
            for (int k = 0; k < kD; ++k) {
                pos[tid * kD + k] = run;
                run += cnt[tid * kD + k];
                plan[tid * kD + k] = (uint32_t)run;
            }
        }
        __syncthreads();
    }
    // colour-1 sample sites of the tile: with a gap neighbour they are listed, the others' energy is constant
    uint16_t* const border = reinterpret_cast<uint16_t*>(plan + C::HDR + 2 * C::CAP);
    long long e_const = 0;
    for (int i = tid; i < C::ECAP; i += 256) {
        const int y = i / (kTW / 2), gy = b.ty0 + y;
        const int x = 2 * (i % (kTW / 2)) + ((y + 1) & 1), gx = b.tx0 + x;
        if (gy >= a.H || gx >= a.W) continue;
        const int yl = y + C::HALO, xl = x + C::HALO;
        const uint8_t* k = kind + yl * C::RW + xl;
        if (k[0] != 2) continue;
        if (k[-C::RW] == 1 || k[-1] == 1 || k[1] == 1 || k[C::RW] == 1) {
            border[atomicAdd(&n_border, 1)] = (uint16_t)((yl - 1) * C::CW + (xl >> 1) + C::LEAD);
            continue;
        }
        const float* t = a.src + (int64_t)gy * a.W + gx;
        auto cs = [&](int step, int64_t off) {
            if (!k[step]) return make_float2(0.0f, 0.0f);
            const float ang = a.q * t[off];
            return make_float2(cos_rev(ang), sin_rev(ang));
        };
        const float2 o = cs(0, 0), u = cs(-C::RW, -(int64_t)a.W), l = cs(-1, -1), r = cs(1, 1),
                     d = cs(C::RW, (int64_t)a.W);
        const float Cx = ((u.x + l.x) + r.x) + d.x;
        const float Sy = ((u.y + l.y) + r.y) + d.y;
        e_const += to_fix(-fmaf(o.x, Cx, o.y * Sy));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e_const += __shfl_xor(e_const, off, 64);
    if ((tid & 63) == 0) esum[tid >> 6] = e_const;
    __syncthreads();
    if (tid == 0) {
        const unsigned long long e = (unsigned long long)(((esum[0] + esum[1]) + esum[2]) + esum[3]);
        plan[4 * kD] = (uint32_t)n_border;
        plan[4 * kD + 1] = (uint32_t)e;
        plan[4 * kD + 2] = (uint32_t)(e >> 32);
    }
}

template <bool TABLE>
__global__ __launch_bounds__(256) void k_tile_plan(TileArgs a)
{
    tile_plan<TABLE>(a, (int)blockIdx.x);
}

// ---- the sweeps ----
struct alignas(16) TileLds {
    using C = Tl;
    float2 cs[2 * C::CELLS];               // (cos, sin) of 2 pi q t, colour 0 then colour 1
    float t[2 * C::CELLS];                 // angles
    uint32_t list[2 * C::CAP];
    uint16_t border[C::ECAP];
    TBand tab[kTabCap];                    // temperatures of the blocks the region touches
    int brow[C::RH], bcol[C::RW];          // without the table: row and column parts of a site's temperature index
    int count[4 * kD];                      // the plan's entry counts
    unsigned long long red[kD];
};

// One update from the LDS neighbourhood: the proposal, the field of the neighbours and the filter's margin r (accept
// iff r < 0) and tolerance (|r| <= tol: the exact test decides), as in the realization-lane sweep (rl_sweep.hip).
struct Trial {
    float tp, cp, sp, ui, Cx, Sy, r, tol;
};

__device__ __forceinline__ Trial trial(const TileArgs& a, float2 o, float2 u, float2 l, float2 rt, float2 d, uint32_t wp,
                                       uint32_t wa, const TBand& tb)
{
    Trial x;
    x.Cx = ((u.x + l.x) + rt.x) + d.x;
    x.Sy = ((u.y + l.y) + rt.y) + d.y;
    x.tp = u24(wp);
    x.ui = (float)(wa >> 8);
    const float ang = a.q * x.tp;
    x.cp = cos_rev(ang);
    x.sp = sin_rev(ang);
    const float X = fmaf(x.cp - o.x, x.Cx, (x.sp - o.y) * x.Sy);
    const float w24 = exp2_fast(fminf(fmaf(X, tb.kappa, 24.0f), 25.0f));
    const bool tpos = tb.T > 0.0f;
    x.r = tpos ? x.ui - w24 : -a.J * X;
    x.tol = tpos ? fmaf(w24, fmaf(fabsf(X), tb.kb, tb.band), 0.015625f) : a.delta_e;
    return x;
}

// The exact decision for the lanes inside the band (r becomes -1 or 1).  Mostly one lane of a wave is, and the workgroup
// waits for it: its eight FP64 cosines are then formed by eight lanes (128 x 128, R = 10, 200 sweeps: 1.08 -> 1.01 ms;
// 2048 x 2048, R = 10, 40 sweeps: 6.60 -> 6.41 ms).  With more than four, or fewer than eight lanes active, each decides its
// own: eight cosines each, but all of them at once.
__device__ __forceinline__ void settle(Trial& x, const float* t, const TileArgs& a, float2 u, float2 l, float2 rt,
                                       float2 d, float T, int i_own, int i_u, int i_l, int i_r, int i_d)
{
    const bool open = fabsf(x.r) <= x.tol;
    unsigned long long left = __ballot(open);
    if (left == 0) return;
    const unsigned pres = (here(u) ? 1u : 0u) | (here(l) ? 2u : 0u) | (here(rt) ? 4u : 0u) | (here(d) ? 8u : 0u);
    // (angles are not negative; without the fabsf the kernels take three more registers and are 1 % slower)
    const float own = t[i_own], tu = fabsf(t[i_u]), tl = fabsf(t[i_l]), tr = fabsf(t[i_r]), td = fabsf(t[i_d]);
    const float u2 = x.ui * 5.9604644775390625e-8f;
    if (__popcll(__ballot(1)) >= 8 && __popcll(left) <= 4) {
        do {
            const int src = __ffsll((long long)left) - 1;
            left &= left - 1;
            const bool acc = exact_of_lane(src, x.tp, own, tu, tl, tr, td, pres, a.two_pi_q, a.Jd, T, u2);
            if (((int)threadIdx.x & 63) == src) x.r = acc ? -1.0f : 1.0f;
        } while (left != 0);
    } else if (open) {
        x.r = exact64(x.tp, own, tu, tl, tr, td, pres, a.two_pi_q, a.Jd, T, u2) ? -1.0f : 1.0f;
    }
}

// writes an accepted proposal; returns the energy / J of the site's bonds after the update (fixed point) if ENERGY
template <bool ENERGY>
__device__ __forceinline__ int commit(const Trial& x, float* t, float2* cs, float2 o, int i_own)
{
    const bool acc = x.r < 0.0f;
    if (acc) {
        t[i_own] = x.tp;
        cs[i_own] = make_float2(x.cp, x.sp);
    }
    return ENERGY ? to_fix(-fmaf(acc ? x.cp : o.x, x.Cx, (acc ? x.sp : o.y) * x.Sy)) : 0;
}

// offsets, in cells from the lowest cell a colour-COLOUR site reads: the site, the cells above and below it, and the
// other colour's cells in its row
template <int COLOUR>
struct Off {
    using C = Tl;
    static constexpr int OWN = COLOUR == 0 ? 0 : C::CELLS + C::CW;
    static constexpr int UP = COLOUR == 0 ? C::CELLS - C::CW : 0;
    static constexpr int DN = COLOUR == 0 ? C::CELLS + C::CW : 2 * C::CW;
    static constexpr int MID = COLOUR == 0 ? C::CELLS : C::CW;
};

// the temperature of a site without the LDS table: q the row of its lowest cell, b that cell
template <int COLOUR>
__device__ __forceinline__ TBand site_temperature(const TileLds& L, const TileArgs& a, int b, int q)
{
    using C = Tl;
    const int xl = 2 * (b - q * C::CW - C::LEAD) + (q & 1);
    return a.Tb[L.brow[q + COLOUR] + L.bcol[xl]];
}

// One colour of one sweep: full pairs list[0 .. np), single sites list[CAP - n1 .. CAP) and, with the energy, the ne
// border samples (they read colour-0 cells only, which are current).  Returns the energy of the entries below own_p,
// own_1 (those of the tile).
template <int COLOUR, bool TABLE, bool ENERGY>
__device__ __forceinline__ int tile_colour(TileLds& L, const TileArgs& a, int np, int n1, int own_p, int own_1,
                                           int ne, uint32_t sweep, uint32_t ctr, uint32_t r, int tid)
{
    using C = Tl;
    using O = Off<COLOUR>;
    const uint32_t w3 = ctr_word3(a.scene, TAG_SWEEP, (uint32_t)COLOUR);
    const int mwr = a.Mw - C::CW / 2;
    float2* const cs = L.cs;
    const uint32_t* const list = L.list + COLOUR * C::CAP;
    int e = 0;
    int v = tid;
    for (; v < np; v += kNT) {
        const uint32_t code = list[v];
        const int b = (int)(code & 4095u), q = (int)((code >> 12) & 63u);
        const int hb = b + O::MID + (q & 1);
        const TBand t0 = TABLE ? L.tab[(code >> 18) & 127u] : site_temperature<COLOUR>(L, a, b, q);
        const TBand t1 = TABLE ? t0 : site_temperature<COLOUR>(L, a, b + 1, q);
        const float4 own = *reinterpret_cast<const float4*>(&cs[b + O::OWN]);
        const float4 up = *reinterpret_cast<const float4*>(&cs[b + O::UP]);
        const float4 dn = *reinterpret_cast<const float4*>(&cs[b + O::DN]);
        const float2 x0 = cs[hb - 1], x1 = cs[hb], x2 = cs[hb + 1];
        asm volatile("" ::: "memory");          // the reads above are issued before the Philox rounds
        const U4 w = philox_x3((uint32_t)__mul24(q, mwr) + (uint32_t)(b >> 1) + ctr, sweep, r, w3, a.key0, a.key1);
        // the two sites share no bond: both trials first, so that their chains of operations overlap
        const float2 o0 = make_float2(own.x, own.y), o1 = make_float2(own.z, own.w);
        const float2 u0 = make_float2(up.x, up.y), u1 = make_float2(up.z, up.w);
        const float2 d0 = make_float2(dn.x, dn.y), d1 = make_float2(dn.z, dn.w);
        Trial y0 = trial(a, o0, u0, x0, x1, d0, w.x, w.y, t0), y1 = trial(a, o1, u1, x1, x2, d1, w.z, w.w, t1);
        if (__ballot(fabsf(y0.r) <= y0.tol || fabsf(y1.r) <= y1.tol)) {
            settle(y0, L.t, a, u0, x0, x1, d0, t0.T, b + O::OWN, b + O::UP, hb - 1, hb, b + O::DN);
            settle(y1, L.t, a, u1, x1, x2, d1, t1.T, b + 1 + O::OWN, b + 1 + O::UP, hb, hb + 1, b + 1 + O::DN);
        }
        const int e0 = commit<ENERGY>(y0, L.t, cs, o0, b + O::OWN);
        const int e1 = commit<ENERGY>(y1, L.t, cs, o1, b + 1 + O::OWN);
        if (ENERGY && v < own_p) e += e0 + e1;
    }
    for (v -= np; v < n1; v += kNT) {
        const uint32_t code = list[C::CAP - 1 - v];
        const int b = (int)(code & 4095u), q = (int)((code >> 12) & 63u);
        const int hb = b + O::MID + (q & 1);
        const TBand tb = TABLE ? L.tab[(code >> 18) & 127u] : site_temperature<COLOUR>(L, a, b, q);
        const float2 o = cs[b + O::OWN], u = cs[b + O::UP], d = cs[b + O::DN], l = cs[hb - 1], rt = cs[hb];
        asm volatile("" ::: "memory");
        const U4 w = philox_x3((uint32_t)__mul24(q, mwr) + (uint32_t)(b >> 1) + ctr, sweep, r, w3, a.key0, a.key1);
        const bool h = (code >> 25) & 1u;
        Trial y = trial(a, o, u, l, rt, d, h ? w.z : w.x, h ? w.w : w.y, tb);
        if (__ballot(fabsf(y.r) <= y.tol))
            settle(y, L.t, a, u, l, rt, d, tb.T, b + O::OWN, b + O::UP, hb - 1, hb, b + O::DN);
        const int e0 = commit<ENERGY>(y, L.t, cs, o, b + O::OWN);
        if (ENERGY && v < own_1) e += e0;
    }
    if (ENERGY) {
        for (v -= n1; v < ne; v += kNT) {
            const int b = (int)L.border[v];
            const int hb = b + O::MID + ((b / C::CW) & 1);
            const float2 o = cs[b + O::OWN], u = cs[b + O::UP], d = cs[b + O::DN], l = cs[hb - 1], rt = cs[hb];
            const float Cx = ((u.x + l.x) + rt.x) + d.x;
            const float Sy = ((u.y + l.y) + rt.y) + d.y;
            e += to_fix(-fmaf(o.x, Cx, o.y * Sy));
        }
    }
    return e;
}

// sum over the 16 lanes of a row, in every lane of it
__device__ __forceinline__ int row_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false);     // row_ror 8, 4, 2, 1
    x += __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false);
    return x;
}

// Item `work` of a run: a tile and a chunk of its realizations.  ENERGY and SNAP are never both set: energies belong to the
// sweeps up to equilibrium, snapshots to the sampling ones.
template <bool TABLE, bool ENERGY, bool SNAP>
__device__ __forceinline__ void tile_item(TileLds& L, TileArgs a, uint32_t work)
{
    using C = Tl;
    const int tile = (int)(work % (uint32_t)a.ntiles);
    const int r0 = (int)(work / (uint32_t)a.ntiles) * a.rchunk;
    const int r1 = r0 + a.rchunk < a.R ? r0 + a.rchunk : a.R;
    const int tid = (int)threadIdx.x;
    const TileBox box = tile_box(a, tile);
    const uint32_t* const plan = a.plan + (size_t)tile * C::WORDS;

    // ---- staging: cells outside, lists, temperatures, samples ----
    // The tile's cells are requested first, their loads run under the rest (256 x 256, R = 10: 26.5 us for five sweeps, 27.2
    // when the cells were loaded after the lists had arrived; of either, 7 us are launch and staging).
    // my cells: bits 0-15 LDS cell, 16 gap, 17 of the tile; offset within a realization (H W < 2^31)
    uint32_t cell[C::CPT];
    int off[C::CPT];
    const float* __restrict__ src0 = a.src + (int64_t)r0 * a.HW;
    float pre[C::CPT];
    uint8_t sample[C::CPT];
#pragma unroll
    for (int k = 0; k < C::CPT; ++k) {
        const int i = tid + k * kNT;
        const int yl = i / C::RW, xl = i % C::RW;
        const int gy = box.ty0 - C::HALO + yl, gx = box.tx0 - C::HALO + xl;
        const int d = ring(yl - C::HALO, xl - C::HALO);
        cell[k] = 0u;
        off[k] = 0;
        pre[k] = 0.0f;
        sample[k] = 0;
        if (yl < C::RH && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W && d <= 2 * a.ns) {
            cell[k] = (uint32_t)(((yl + xl) & 1) * C::CELLS + yl * C::CW + (xl >> 1) + C::LEAD) | 1u << 16 |
                      (d == 0 ? 1u << 17 : 0u);
            off[k] = gy * a.W + gx;
            pre[k] = src0[off[k]];
            sample[k] = a.mask[off[k]];
        }
    }
    for (int i = tid; i < 2 * C::CELLS; i += kNT) {
        L.cs[i] = make_float2(0.0f, 0.0f);
        L.t[i] = 0.0f;
    }
    for (int c = 0; c < 2; ++c) {
        const int np = (int)plan[(2 * c) * kD + a.ns - 1], n1 = (int)plan[(2 * c + 1) * kD + a.ns - 1];
        for (int i = tid; i < np; i += kNT) L.list[c * C::CAP + i] = plan[C::HDR + c * C::CAP + i];
        for (int i = tid; i < n1; i += kNT)
            L.list[(c + 1) * C::CAP - 1 - i] = plan[C::HDR + (c + 1) * C::CAP - 1 - i];
    }
    if (tid < 4 * kD) L.count[tid] = (int)plan[tid];
    const int ne = ENERGY ? (int)plan[4 * kD] : 0;
    if (ENERGY) {
        const uint16_t* const border = reinterpret_cast<const uint16_t*>(plan + C::HDR + 2 * C::CAP);
        for (int i = tid; i < ne; i += kNT) L.border[i] = border[i];
        if (tid < kD) L.red[tid] = 0ull;
    }
    if (TABLE) {
        if (tid < box.nby * box.nbx)
            L.tab[tid] = a.Tb[(int64_t)(box.by0 + tid / box.nbx) * a.nbx + box.bx0 + tid % box.nbx];
    } else {
        if (tid < C::RH) {
            const int gy = box.ty0 - C::HALO + tid;
            L.brow[tid] = gy >= 0 && gy < a.H ? (gy / a.lb_h) * a.nbx : 0;
        } else if (tid >= 128 && tid < 128 + C::RW) {
            const int gx = box.tx0 - C::HALO + tid - 128;
            L.bcol[tid - 128] = gx >= 0 && gx < a.W ? gx / a.lb_w : 0;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C::CPT; ++k) {
        if (sample[k] != 0) {
            const int li = (int)(cell[k] & 0xffffu);
            const float ang = a.q * pre[k];
            L.t[li] = pre[k];
            L.cs[li] = make_float2(cos_rev(ang), sin_rev(ang));
            cell[k] = 0u;
            off[k] = 0;
        }
    }
    // the random-stream counter of a pair is row Mw + group; with b its lowest cell and q that cell's row, the group is
    // b / 2 - q CW / 2 counted from the region's own first
    const uint32_t ctr0 = (uint32_t)(box.ty0 - C::HALO) * (uint32_t)a.Mw + (uint32_t)(box.tx0 / 4) -
                          (uint32_t)((kD + C::LEAD) / 2);
    const long long e_const =
        ENERGY ? (long long)((unsigned long long)plan[4 * kD + 2] << 32 | (unsigned long long)plan[4 * kD + 1]) : 0;

    for (int r = r0; r < r1; ++r) {
        // opaque per realization: 32-bit offsets from a uniform base, not 64-bit addresses kept across the loop
#pragma unroll
        for (int k = 0; k < C::CPT; ++k) asm volatile("" : "+v"(off[k]));
#pragma unroll
        for (int k = 0; k < C::CPT; ++k) {
            if (cell[k] >> 16) {
                const int li = (int)(cell[k] & 0xffffu);
                const float ang = a.q * pre[k];
                L.t[li] = pre[k];
                L.cs[li] = make_float2(cos_rev(ang), sin_rev(ang));
            }
        }
        __syncthreads();
        if (r + 1 < r1) {                     // the next realization's gap cells, while this one is updated
            const float* __restrict__ srcn = a.src + (int64_t)(r + 1) * a.HW;
#pragma unroll
            for (int k = 0; k < C::CPT; ++k)
                if (cell[k] >> 16) pre[k] = srcn[(uint32_t)off[k]];
        }
        const uint32_t rg = a.real_offset + (uint32_t)r;
        for (int i = 0; i < a.ns; ++i) {
            const int k = a.ns - 1 - i;       // sweeps that follow
            const uint32_t sweep = a.sweep + (uint32_t)i;
            auto count = [&](int list, int bucket) { return __builtin_amdgcn_readfirstlane(L.count[list * kD + bucket]); };
            tile_colour<0, TABLE, false>(L, a, count(0, k), count(1, k), 0, 0, 0, sweep, ctr0, rg, tid);
            __syncthreads();
            int e = tile_colour<1, TABLE, ENERGY>(L, a, count(2, k), count(3, k), count(2, 0), count(3, 0), ne, sweep,
                                                     ctr0 + (uint32_t)a.Mw, rg, tid);
            if (ENERGY) {
                // integers, so the order does not matter: sums of 16 lanes in two halves, then one LDS add per row
                const int lo = row_sum(e & 0xffff), hi = row_sum(e >> 16);
                if ((tid & 15) == 0) atomicAdd(&L.red[i], (unsigned long long)((long long)hi * 65536 + lo));
            }
            __syncthreads();
            if (SNAP) {
                float* __restrict__ snap = a.snap + ((int64_t)i * a.R + r) * a.HW;
#pragma unroll
                for (int j = 0; j < C::CPT; ++j)
                    if (cell[j] >> 17) snap[(uint32_t)off[j]] = L.t[cell[j] & 0xffffu];
                __syncthreads();              // before the next sweep changes the cells
            }
        }
        float* __restrict__ dst = a.dst + (int64_t)r * a.HW;
#pragma unroll
        for (int k = 0; k < C::CPT; ++k)
            if (cell[k] >> 17) dst[(uint32_t)off[k]] = L.t[cell[k] & 0xffffu];
        if (ENERGY && tid < a.ns) {
            a.e_partial[((int64_t)tid * a.R + r) * a.ntiles + tile] = e_const + (long long)L.red[tid];
            L.red[tid] = 0ull;
        }
    }
}

template <bool TABLE, bool ENERGY, bool SNAP>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_tile_sweeps(TileArgs a)
{
    __shared__ TileLds L;
    const uint32_t work = item_of(blockIdx.x, blockIdx.y, kItemRow, (uint32_t)a.ntiles * (uint32_t)a.nchunks);
    if (work != kNoItem) tile_item<TABLE, ENERGY, SNAP>(L, a, work);
}

// A pointer read from memory, known to be global: flat accesses would wait for the LDS as well.
template <class T>
__device__ __forceinline__ T* in_global(T* p)
{
    return (T*)(__attribute__((address_space(1))) T*)(uint64_t)p;
}

// The arguments of the scene that item `work` of a batch belongs to; returns the scene's first item.
__device__ __forceinline__ uint32_t batch_args(const TileBatch& b, uint32_t work, TileArgs* args)
{
    int lo = 0, hi = b.n;                     // prefix[lo] <= work < prefix[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (b.prefix[mid] <= work) lo = mid;
        else hi = mid;
    }
    // the scene's arguments through the constant address space: scalar loads
    using CU = const __attribute__((address_space(4))) uint32_t;
    const uint64_t ad = (uint64_t)(b.scenes[b.list[lo]].a + b.parity);
    const CU* p = (const CU*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)ad) |
                              (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(ad >> 32)) << 32);
    static_assert(sizeof(TileArgs) % 4 == 0, "read in words");
    uint32_t words[sizeof(TileArgs) / 4];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(TileArgs) / 4); ++i) words[i] = p[i];
    TileArgs& a = *args;
    __builtin_memcpy(&a, words, sizeof a);
    a.src = in_global(a.src);
    a.dst = in_global(a.dst);
    a.mask = in_global(a.mask);
    a.Tb = in_global(a.Tb);
    a.plan = in_global(a.plan);
    a.e_partial = in_global(a.e_partial);
    return b.prefix[lo];
}

// The plans of all scenes in one launch: the items of a scene's first chunk of realizations.
template <bool TABLE>
__global__ __launch_bounds__(256) void k_tile_batch_plan(TileBatch b)
{
    const uint32_t work = item_of(blockIdx.x, blockIdx.y, kItemRow, b.prefix[b.n]);
    if (work == kNoItem) return;
    TileArgs a;
    const uint32_t tile = work - batch_args(b, work, &a);
    if (tile < (uint32_t)a.ntiles) tile_plan<TABLE>(a, (int)tile);
}

// The scenes of a batch in one launch: items are numbered through the scenes of the list.  As in a single call up to five
// sweeps stay in LDS, so that a launch, the staging and the pass over the states are paid once for them; a persistent queue
// of (scene, tile, chunk) items with one sweep per launch and a graph of five launches a sweep took, for 60 sweeps at most,
// 10.5 / 19.8 ms at 24 scenes of 64 .. 512 a side and R = 8 / 32 (4.7 / 11.8 so), 45.4 ms at 12 scenes of 256 .. 1024 and
// R = 32 (27.5), 14.3 ms at 200 scenes of 16 .. 64 and R = 10 (11.4, of it most in the starts' small launches).  The scenes
// still running advance in step, so a check reads all means in one copy.
template <bool TABLE, bool ENERGY>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_tile_batch(TileBatch b)
{
    __shared__ TileLds L;
    const uint32_t work = item_of(blockIdx.x, blockIdx.y, kItemRow, b.prefix[b.n]);
    if (work == kNoItem) return;
    TileArgs a;
    const uint32_t first = batch_args(b, work, &a);
    a.sweep = b.sweep;
    a.ns = b.ns;
    tile_item<TABLE, ENERGY, false>(L, a, work - first);
}

// acc of the listed scenes += the gap angles of the state after the launch, over the realizations in order.
__global__ __launch_bounds__(256) void k_tile_batch_accumulate(TileBatch b, int first)
{
    const TileScene& d = b.scenes[b.list[blockIdx.y]];
    const float* const st = d.a[b.parity].dst;
    const uint8_t* const mask = d.a[0].mask;
    const int64_t HW = d.a[0].HW;
    const int R = d.a[0].R;
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < HW; n += (int64_t)gridDim.x * 256) {
        if (mask[n]) {
            if (first) d.acc[n] = 0.0;
            continue;
        }
        double v = first ? 0.0 : d.acc[n];
        int r = 0;
        for (; r + 8 <= R; r += 8) {          // eight loads in flight, added in order
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = st[(int64_t)(r + k) * HW + n];
#pragma unroll
            for (int k = 0; k < 8; ++k) v += (double)x[k];
        }
        for (; r < R; ++r) v += (double)st[(int64_t)r * HW + n];
        d.acc[n] = v;
    }
}

// Sampling: one launch for the states of several sweeps (acc[n] is the sum over the states and, within a state, over the
// realizations in order, as with one launch per sweep).  Launches and latency bound the small grids it is for: 128 x 128,
// R = 10, 100 + 100 sweeps take 2.15 ms with a launch of both kernels per sampling sweep, 1.20 ms with one per five and
// 1.09 ms with a sum (and a reduction of energies) per twenty.
__global__ __launch_bounds__(256) void k_accumulate_n(const float* __restrict__ states, const uint8_t* __restrict__ mask,
                                                       int64_t HW, int64_t rows, int first, double* __restrict__ acc)
{
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= HW) return;
    if (mask[n]) {
        if (first) acc[n] = 0.0;
        return;
    }
    double v = first ? 0.0 : acc[n];
    const float* p = states + n;
    int64_t i = 0;
    for (; i + 16 <= rows; i += 16) {         // sixteen loads in flight, added in order
        float x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = p[(i + k) * HW];
#pragma unroll
        for (int k = 0; k < 16; ++k) v += (double)x[k];
    }
    for (; i < rows; ++i) v += (double)p[i * HW];
    acc[n] = v;
}

// ---- energies of several sweeps ----
__global__ __launch_bounds__(256) void k_energy_real_n(const long long* __restrict__ partial, int nparts, int R,
                                                        double inv_norm, double* e_real)
{
    __shared__ long long red[4];
    const int64_t row = (int64_t)blockIdx.y * R + blockIdx.x;
    long long s = 0;
    for (int p = (int)threadIdx.x; p < nparts; p += 256) s += partial[row * nparts + p];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) e_real[row] = ((double)(((red[0] + red[1]) + red[2]) + red[3]) * kFixUnit) * inv_norm;
}

// mean over the realizations, added in order: 64 at a time, one load per lane and reads of fixed lanes, which do not depend on
// the sum (and to host memory, for a host that waits for the value)
__device__ __forceinline__ void ordered_mean(const double* e_real, int R, double* out, double* host)
{
    const int lane = (int)(threadIdx.x & 63u);
    double sum = 0.0;
    for (int r0 = 0; r0 < R; r0 += 64) {
        const double v = r0 + lane < R ? e_real[r0 + lane] : 0.0;
        const int lo = __double2loint(v), hi = __double2hiint(v);
        const int m = R - r0 < 64 ? R - r0 : 64;
#pragma unroll
        for (int j = 0; j < 64; ++j)
            if (j < m) sum += __hiloint2double(__builtin_amdgcn_readlane(hi, j), __builtin_amdgcn_readlane(lo, j));
    }
    if (lane != 0) return;
    const double mean = sum / (double)R;
    *out = mean;
    if (host) __hip_atomic_store(host, mean, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(64) void k_energy_mean_n(const double* e_real, int R, double* e_out, double* host)
{
    ordered_mean(e_real + (int64_t)blockIdx.x * R, R, e_out + blockIdx.x, host ? host + blockIdx.x : nullptr);
}

// The energies of a launch of a batch: a workgroup per (scene of the list, sweep); sweep k's means also go to
// means[1 + (k - 1) % ring][scene].
__global__ __launch_bounds__(1024) void k_tile_batch_energy(TileBatch b, double* means, int n_scenes, int ring)
{
    const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6), scene = b.list[blockIdx.x];
    const TileScene& d = b.scenes[scene];
    const int R = d.a[0].R, nparts = d.a[0].ntiles;
    double* const er = d.e_real + (int64_t)blockIdx.y * R;
    for (int r = wv; r < R; r += 16) {
        const long long* const row = d.a[0].e_partial + ((int64_t)blockIdx.y * R + r) * nparts;
        long long s = 0;
        for (int p = lane; p < nparts; p += 64) s += row[p];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) er[r] = ((double)s * kFixUnit) * d.inv_norm;
    }
    __syncthreads();
    const int64_t k = (int64_t)b.sweep + blockIdx.y;
    if (wv == 0) ordered_mean(er, R, d.series + k, means + (1 + (k - 1) % ring) * n_scenes + scene);
}

// Both steps in one workgroup per sweep, where the partials are few: one wave per realization at a time.
__global__ __launch_bounds__(1024) void k_energy_small(const long long* __restrict__ partial, int nparts, int R,
                                                        double inv_norm, double* e_real, double* e_out, double* host)
{
    const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6);
    double* const er = e_real + (int64_t)blockIdx.x * R;
    for (int r = wv; r < R; r += 16) {
        const long long* const row = partial + ((int64_t)blockIdx.x * R + r) * nparts;
        long long s = 0;
        for (int p = lane; p < nparts; p += 64) s += row[p];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) er[r] = ((double)s * kFixUnit) * inv_norm;
    }
    __syncthreads();
    if (wv == 0) ordered_mean(er, R, e_out + blockIdx.x, host ? host + blockIdx.x : nullptr);
}

}  // namespace

TileGeom tile_geometry(int64_t H, int64_t W, int R)
{
    TileGeom g;
    g.depth = kD;
    g.ntx = (int)((W + kTW - 1) / kTW);
    g.nty = (int)((H + kTH - 1) / kTH);
    g.ntiles = g.ntx * g.nty;
    // Two workgroups fit a CU, 512 the device: realizations are put into one workgroup (they share its staging) while
    // about two rounds of workgroups are left.  512 x 512, R = 32: 46.9 / 42.8 / 39.3 / 38.9 us per sweep at 4096 /
    // 2048 / 1024 / 512 workgroups; 300 x 2000, R = 20 (320 tiles): 60.3 us at 1024 and 74.1 us at 512.
    const int64_t rc = (int64_t)g.ntiles * R / 1024;
    g.rchunk = (int)(rc < 1 ? 1 : (rc > R ? R : rc));
    if (g.rchunk > 64) g.rchunk = 64;
    g.nchunks = (R + g.rchunk - 1) / g.rchunk;
    g.plan_words = (size_t)g.ntiles * Tl::WORDS;
    return g;
}

namespace {

// the LDS temperature table: pairs inside one block (block columns of whole groups of four) and few enough blocks
bool tile_table(const TileArgs& a)
{
    using C = Tl;
    const int64_t ny = (C::RH - 2) / a.lb_h + 2, nx = (C::RW - 2) / a.lb_w + 2;
    return a.lb_w % 4 == 0 && ny * nx <= kTabCap;
}

}  // namespace

hipError_t launch_tile_plan(const TileArgs& a, hipStream_t s)
{
    if (tile_table(a)) hipLaunchKernelGGL((k_tile_plan<true>), dim3((unsigned)a.ntiles), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_tile_plan<false>), dim3((unsigned)a.ntiles), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tile_sweeps(const TileArgs& a, hipStream_t s)
{
    const dim3 grid = item_grid((uint32_t)a.ntiles * (uint32_t)a.nchunks);
#define MPR_TILES(TAB, EN, SN) hipLaunchKernelGGL((k_tile_sweeps<TAB, EN, SN>), grid, dim3(kNT), 0, s, a)
    if (tile_table(a)) {
        if (a.e_partial) MPR_TILES(true, true, false);
        else if (a.snap) MPR_TILES(true, false, true);
        else MPR_TILES(true, false, false);
    } else {
        if (a.e_partial) MPR_TILES(false, true, false);
        else if (a.snap) MPR_TILES(false, false, true);
        else MPR_TILES(false, false, false);
    }
#undef MPR_TILES
    return hipGetLastError();
}

bool tile_uses_table(const TileArgs& a) { return tile_table(a); }

hipError_t launch_tile_batch_plan(const TileBatch& b, uint32_t work, hipStream_t s)
{
    if (b.n <= 0 || work == 0) return hipSuccess;
    if (b.table) hipLaunchKernelGGL(k_tile_batch_plan<true>, item_grid(work), dim3(256), 0, s, b);
    else hipLaunchKernelGGL(k_tile_batch_plan<false>, item_grid(work), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_tile_batch(const TileBatch& b, uint32_t work, bool energy, hipStream_t s)
{
    if (b.n <= 0 || work == 0) return hipSuccess;
    const dim3 grid = item_grid(work);
#define MPR_TILES(TAB, EN) hipLaunchKernelGGL((k_tile_batch<TAB, EN>), grid, dim3(kNT), 0, s, b)
    if (b.table) {
        if (energy) MPR_TILES(true, true);
        else MPR_TILES(true, false);
    } else {
        if (energy) MPR_TILES(false, true);
        else MPR_TILES(false, false);
    }
#undef MPR_TILES
    return hipGetLastError();
}

hipError_t launch_tile_batch_energy(const TileBatch& b, double* means, int n_scenes, int ring, hipStream_t s)
{
    if (b.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_batch_energy, dim3((unsigned)b.n, (unsigned)b.ns), dim3(1024), 0, s, b, means, n_scenes,
                       ring);
    return hipGetLastError();
}

hipError_t launch_tile_batch_accumulate(const TileBatch& b, bool first, int blocks, hipStream_t s)
{
    for (int at = 0; at < b.n; at += 65535) {              // (grid.y)
        TileBatch part = b;
        part.list = b.list + at;
        const int n = b.n - at < 65535 ? b.n - at : 65535;
        hipLaunchKernelGGL(k_tile_batch_accumulate, dim3((unsigned)blocks, (unsigned)n), dim3(256), 0, s, part, first ? 1 : 0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_accumulate_n(const float* states, const uint8_t* mask, int64_t HW, int R, int ns, bool first,
                               double* acc, hipStream_t s)
{
    hipLaunchKernelGGL(k_accumulate_n, dim3((unsigned)((HW + 255) / 256)), dim3(256), 0, s, states, mask, HW,
                       (int64_t)R * ns, first ? 1 : 0, acc);
    return hipGetLastError();
}

hipError_t launch_energy_reduce_n(const long long* partial, int nparts, int R, int ns, double inv_norm, double* e_real,
                                  double* e_out, double* host, hipStream_t s)
{
    if ((int64_t)((nparts + 63) / 64) * ((R + 15) / 16) <= 8) {        // (loads of a wave, one after another)
        hipLaunchKernelGGL(k_energy_small, dim3((unsigned)ns), dim3(1024), 0, s, partial, nparts, R, inv_norm, e_real,
                           e_out, host);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_energy_real_n, dim3((unsigned)R, (unsigned)ns), dim3(256), 0, s, partial, nparts, R, inv_norm,
                       e_real);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_energy_mean_n, dim3((unsigned)ns), dim3(64), 0, s, e_real, R, e_out, host);
    return hipGetLastError();
}

}  // namespace mpr
