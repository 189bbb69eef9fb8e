// The 3D lattice: the method on a D x H x W grid (the extension to three dimensions named in Sec. 4).  Reading: the
// same Hamiltonian (Eq. 1) over the six nearest neighbours of the simple cubic lattice with open boundaries, the
// checkerboard colours c = (x + y + z) mod 2, temperature blocks lb_d x lb_h x lb_w, and the plane's random stream
// with the row index z H + y in place of y and the colour (x + y + z) mod 2.
//
// The sweep keeps the realization-lane layout of the plane, S[g][n][64] with n = (z H + y) W + x, but is a pair of
// half-sweeps (one launch per colour): a colour-c half-sweep reads only colour-(1 - c) neighbours, which it does not
// change, so it runs in place, with no ring of redundant updates and no second buffer, and a rejected proposal
// writes nothing.  A wave owns the columns [x0, x0 + 8) of two rows y0, y0 + 1 (y0 even) and a segment of planes of
// one group of 64 realizations, and streams along z on its own: no barrier and no exchange with other waves.
//
// What a plane needs: the (cos, sin) of the other colour's cells of the two rows, five a row with the one beside the
// band (they are also the neighbours along z of the next and the previous plane's updates, and of each other's row, so
// each is computed once), and for the cells that are updated the angles of the cell itself and of the one neighbour
// outside the two rows, whose (cos, sin) are taken at the update, for gap cells only.  With y0 even the updated
// columns depend on the plane and the launch's colour alone, so the loop has one form, four planes long.
//
// The exact decisions wait until the wave's streaming is over: the neighbours of an undecided site do not change in this
// half-sweep and the site keeps its angle, so only its place and the lanes in question are noted (in LDS, and the
// streaming pauses to settle them if they become many).  Settling them on the spot is a function call with the whole
// window live across it, for which the call's convention costs a second register for most of them.
//
// Measured (160^3, p = 0.6, R = 128; a sweep with its energy): 2.64 ms with four waves sharing rows through LDS behind a
// barrier per plane and the exact test called on the spot, 1.46 ms with this layout at two waves per SIMD, 1.30 ms at
// three and without the loads of sample cells that nothing reads (256^3, R = 64: 5.26 / 2.90 / 2.70 ms).  Bounds: at two waves
// per SIMD a colour-0 half-sweep read 2.45 GB (the state is 2.1 GB) in 0.67 ms, near what a copy reaches, with the VALU
// busy 59 % of the time.
//
// Every load of a step is issued a step ahead, and the new angles of a plane are stored a step late, right after the
// next loads have arrived: the arrival's wait (the counter retires in order) then finds stores a step old instead of
// ones just issued.
//
// The update (independent uniform proposal, FP32 filter with its error band, exact FP64 decision inside the band,
// in the oracle's neighbour order back, up, left, right, down, front) and the fixed-point energy of the colour-1
// sites (every bond has one colour-1 end) follow the plane's kernels.
#include <hip/hip_runtime.h>

#include "metropolis.hpp"
#include "cos64.hpp"
#include "exact6.hpp"
#include "lattice3d.hpp"
#include "mpr_internal.hpp"
#include "philox_lane.hpp"

namespace mpr {

namespace {

constexpr int kW3 = kB3 + 2;        // window columns x0 - 1 .. x0 + kB3
constexpr uint32_t kQueue3 = 64;   // undecided updates a wave notes; four planes add at most 32
static_assert(kB3 == 8, "two Philox pairs a row and plane");

__device__ __forceinline__ int fix24(float x) { return __float2int_rn(x * 16777216.0f); }

template <class T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NT, class T>
__device__ __forceinline__ T block_sum(T v, T* lds)
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

// philox_site with the round keys formed on the scalar unit: the sixteen key registers of RoundKeys are what keeps
// this kernel from a third wave per SIMD.
__device__ __forceinline__ U4 philox_site_s(uint32_t site, uint32_t w3k1, const PhiloxLane& L, uint32_t k0, uint32_t k1)
{
    asm volatile("" : "+s"(k0), "+s"(k1));
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)site;
    const uint32_t n2u = (uint32_t)(p0 >> 32) ^ w3k1, c3u = (uint32_t)p0;
    const uint64_t q1 = (uint64_t)0xCD9E8D57u * (uint64_t)n2u;
    uint32_t c0 = (uint32_t)(q1 >> 32) ^ L.lc1;
    uint32_t c1 = (uint32_t)q1;
    uint32_t c2 = c3u ^ L.lph;
    uint32_t c3 = L.lpl;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t a0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t a1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        const uint32_t n0 = xor3((uint32_t)(a1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(a0 >> 32), c3, k1);
        c1 = (uint32_t)a1;
        c3 = (uint32_t)a0;
        c0 = n0;
        c2 = n2;
    }
    return U4{c0, c1, c2, c3};
}

// exact64_6 of the first four lanes of `left` by the whole wave, sixteen lanes a decision with a cosine each; true in those of
// the four that accept.  Mostly one lane is open and 63 wait: a cosine and an exponential in a row instead of twelve and one
// (160^3, R = 128, 15 sweeps: 22.2 -> 21.9 ms).
__device__ __noinline__ bool exact6_round(unsigned long long left, float tp, float to, float nb, float nu, float nl, float nr,
                                          float nd, float nf, unsigned present, double two_pi_q, double J, float T, float u2)
{
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(left >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)left, 0));
    const bool mine = ((left >> lane) & 1ull) != 0 && rank < 4;
    // lane 16 k learns the k-th of them (lane 63 takes what the others send), and its sixteen lanes from it
    const int from = __builtin_amdgcn_ds_permute((mine ? rank * 16 : 63) * 4, lane);
    const int src = __builtin_amdgcn_ds_bpermute((lane & ~15) * 4, from) * 4, term = lane & 15;
    auto of = [&](float x) { return __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(x))); };
    const float n0 = of(nb), n1 = of(nu), n2 = of(nl), n3 = of(nr), n4 = of(nd), n5 = of(nf);
    const float p = of(tp), o = of(to), u = of(u2);
    const float n = term < 2 ? n0 : term < 4 ? n1 : term < 6 ? n2 : term < 8 ? n3 : term < 10 ? n4 : n5;
    const double c = cos(two_pi_q * ((double)(term & 1 ? o : p) - (double)n));
    const double d = c - __shfl_xor(c, 1, 64);           // even lanes: proposed less present
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const double dj = __shfl(d, (lane & ~15) + 2 * j, 64);
        if ((present >> j) & 1u) sum += dj;
    }
    const double dE = -J * sum;
    const bool acc = (double)T > 0.0 ? (double)u < exp(-dE / (double)T) : dE <= 0.0;
    return __builtin_amdgcn_ds_bpermute((mine ? rank * 16 : 0) * 4, acc ? 1 : 0) != 0 && mine;
}

// What the streaming reads of the launch arguments; settling reads the others again from the argument segment, so that
// they hold no scalar registers (and no lanes of spill registers) meanwhile.
struct Loop3 {
    int D, lb_d;
    uint32_t key0, key1;
    float q, J, delta_e;
    // one temperature column per site (AL == false) only
    int W, lb_w;
    uint32_t lbw_inv;
};

// C: the launch's colour.  AL: one temperature column per band (blocks a multiple of 8 wide, or one block).
// With P = (z + C) & 1 the updated columns are x0 + 2k + P in row 0 (y0) and x0 + 2k + 1 - P in row 1 (y0 + 1),
// k = 0 .. 3; the other colour's cells o[row][i], i = 0 .. 4, are at x0 + P - 1 + 2i and x0 - P + 2i.
template <int C, bool ENERGY, bool AL>
struct Wave3 {
    Loop3 a;
    char* S;                           // this wave's group of realizations
    int x0, y0, zs, ze;
    uint32_t lane4, real, w3k1;
    PhiloxLane pl;
    int64_t oz, wplane;                // byte offset of (current plane, row y0, column x0) in the group; bytes per plane
    int d1, dU, dD;                    // byte offsets of rows y0 + 1, y0 - 1, y0 + 2 from row y0 (0: absent)
    uint32_t site, site1, siteP;       // stream counter of the current plane's row y0; to row y0 + 1, to the next plane
    const uint32_t* cells;             // gap bits of the current plane's row y0; words to row y0 + 1, to the next plane
    uint32_t cell1, cellP;
    const TBand *t0, *t1;              // temperatures of the two rows in the current block plane (AL: of the band)
    int64_t tP;                        // temperatures per block plane
    uint32_t colmask;                  // window columns inside the grid
    int bzr;                           // the current plane's place in its temperature block
    uint4* queue;                      // LDS [kQueue3]: undecided updates (plane, row and cell, lanes)
    uint32_t nq;                       // their number
    TBand T0, T1;                      // AL: the two rows' temperatures
    float c[4][2][5], s[4][2][5];      // (cos, sin) of the other colour's cells by slot (plane & 3)
    float oa[2][5];                    // their angles as loaded, until they arrive
    float own[2][2][4], out[2][2][4];  // by plane parity: angles of the updated cells, of their outer neighbours
    float pend[2][4];                  // new angles of the last plane (negative: rejected)
    uint32_t pgap[2];                  // its gap bits (0: nothing pending)
    uint32_t gap[2], ngap[2];          // gap bits of the plane to be updated next and of the one after it
    long long e_acc;

    __device__ __forceinline__ float ld(int64_t off, int j) const
    {
        return *reinterpret_cast<const float*>(S + off + j * 256 + lane4);
    }
    template <class T>
    static __device__ __forceinline__ const T* uniform(const T* p)
    {
        const uint64_t ad = (uint64_t)p;
        return (const T*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)ad) |
                          ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(ad >> 32)) << 32));
    }
    // (through the constant address space: scalar loads whatever the compiler can prove about aliasing)
    static __device__ __forceinline__ uint32_t word(const uint32_t* p)
    {
        return *(const __attribute__((address_space(4))) uint32_t*)uniform(p);
    }

    // the other colour's cells of the plane at byte offset o.  Columns beside the grid are read too: the buffer has a
    // margin, and the arrival clears them.
    template <int P>
    __device__ __forceinline__ void request_others(int64_t o)
    {
        const int64_t o1 = o + d1;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            oa[0][i] = ld(o, P - 1 + 2 * i);
            oa[1][i] = ld(o1, 2 * i - P);
        }
    }

    // the updated cells of the plane at byte offset o and their neighbours in rows y0 - 1 and y0 + 2; without the energy
    // those of its gap cells only (bits g0, g1), a fifth of the half-sweep's reads at 40 % samples
    template <int B, int P>
    __device__ __forceinline__ void request_own(int64_t o, uint32_t g0, uint32_t g1)
    {
        const int64_t o1 = o + d1, oU = o + dU, oD = o + dD;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j0 = 2 * k + P, j1 = 2 * k + 1 - P;
            if (ENERGY || ((g0 >> (j0 + 1)) & 1u)) {
                own[B][0][k] = ld(o, j0);
                out[B][0][k] = ld(oU, j0);
            } else {
                own[B][0][k] = out[B][0][k] = __builtin_nondeterministic_value(0.0f);
            }
            if (ENERGY || ((g1 >> (j1 + 1)) & 1u)) {
                own[B][1][k] = ld(o1, j1);
                out[B][1][k] = ld(oD, j1);
            } else {
                own[B][1][k] = out[B][1][k] = __builtin_nondeterministic_value(0.0f);
            }
        }
    }
    // gap bits of the plane whose row y0 has its word at p
    __device__ __forceinline__ void request_gaps(const uint32_t* p)
    {
        ngap[0] = word(p);
        ngap[1] = d1 ? word(p + cell1) : 0u;
    }

    // the requested cells of plane z enter slot SL; (0, 0) outside the grid
    template <int SL, int P>
    __device__ __forceinline__ void arrive(int z)
    {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const float t = a.q * oa[r][i];
                c[SL][r][i] = cos_rev(t);
                s[SL][r][i] = sin_rev(t);
                oa[r][i] = __builtin_nondeterministic_value(0.0f);
            }
        if (z < 0 || z >= a.D) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int i = 0; i < 5; ++i) c[SL][r][i] = s[SL][r][i] = 0.0f;
        } else {
            if (d1 == 0) {
#pragma unroll
                for (int i = 0; i < 5; ++i) c[SL][1][i] = s[SL][1][i] = 0.0f;
            }
            if (colmask != (1u << kW3) - 1u) {
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    if (!((colmask >> (P + 2 * i)) & 1u)) c[SL][0][i] = s[SL][0][i] = 0.0f;
                    if (!((colmask >> (1 - P + 2 * i)) & 1u)) c[SL][1][i] = s[SL][1][i] = 0.0f;
                }
            }
        }
    }

    // stores the accepted angles of the pending plane (at byte offset off), whose row-0 columns are 2k + P
    template <int P>
    __device__ __forceinline__ void flush(int64_t off)
    {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (pgap[r] == 0u) continue;
            const int64_t o = off + (r ? d1 : 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = 2 * k + (r ? 1 - P : P);
                if (((pgap[r] >> (j + 1)) & 1u) && pend[r][k] >= 0.0f)
                    *reinterpret_cast<float*>(S + o + j * 256 + lane4) = pend[r][k];
            }
            pgap[r] = 0u;
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)               // dead until the next plane writes them
#pragma unroll
            for (int k = 0; k < 4; ++k) pend[r][k] = __builtin_nondeterministic_value(0.0f);
    }

    // a temperature entry (scalar load through the constant space)
    static __device__ __forceinline__ TBand entry(const TBand* e)
    {
        const __attribute__((address_space(4))) uint32_t* p =
            (const __attribute__((address_space(4))) uint32_t*)uniform(e);
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = p[i];
        TBand t;
        __builtin_memcpy(&t, w, sizeof(TBand));
        return t;
    }
    __device__ __forceinline__ int block_column(int x) const
    {
        const int xc = x < a.W ? x : a.W - 1;       // a pair's second column may lie past the grid (not updated)
        return a.lb_w == 1 ? xc : (int)__umulhi((uint32_t)xc, a.lbw_inv);
    }
    __device__ __forceinline__ void load_temperatures()
    {
        T0 = entry(t0);
        T1 = entry(t1);
    }

    // the field of the six neighbours (back, up, left, right, down, front) of updated cell k of row R
    template <int S0, int P, int R>
    __device__ __forceinline__ void field(int k, float* Cx, float* Sy) const
    {
        constexpr int SP = (S0 + 3) & 3, SN = (S0 + 1) & 3;
        const int iz = R == 0 ? k + P : k + 1 - P;          // the cell at the same column in the planes z -+ 1
        float co = 0.0f, so = 0.0f;
        if ((R == 0 ? dU : dD) != 0) {
            const float t = a.q * out[S0 & 1][R][k];
            co = cos_rev(t);
            so = sin_rev(t);
        }
        const float cu = R == 0 ? co : c[S0][0][iz], su = R == 0 ? so : s[S0][0][iz];
        const float cd = R == 0 ? c[S0][1][iz] : co, sd = R == 0 ? s[S0][1][iz] : so;
        *Cx = ((((c[SP][R][iz] + cu) + c[S0][R][k]) + c[S0][R][k + 1]) + cd) + c[SN][R][iz];
        *Sy = ((((s[SP][R][iz] + su) + s[S0][R][k]) + s[S0][R][k + 1]) + sd) + s[SN][R][iz];
    }

    // one Metropolis update of cell k of row R on plane z; returns its bonds' energy / J (fixed point) if ENERGY
    template <int S0, int P, int R>
    __device__ __forceinline__ int update(const TBand& T, int z, int k, uint32_t wp, uint32_t wa)
    {
        float Cx, Sy;
        field<S0, P, R>(k, &Cx, &Sy);
        const float tp = u24(wp);
        const float ui = (float)(wa >> 8);
        const float angp = a.q * tp;
        const float cp = cos_rev(angp), sp = sin_rev(angp);
        const float ango = a.q * own[S0 & 1][R][k];
        const float co = cos_rev(ango), so = sin_rev(ango);
        const float X = fmaf(cp - co, Cx, (sp - so) * Sy);
        const float w24 = exp2_fast(fminf(fmaf(X, T.kappa, 24.0f), 25.0f));
        const bool tpos = __float_as_int(T.T) > 0;
        float r = tpos ? ui - w24 : -a.J * X;
        const float tol = tpos ? fmaf(w24, fmaf(fabsf(X), T.kb, T.band), 0.015625f) : a.delta_e;
        const bool need = fabsf(r) <= tol;
        const uint64_t lanes = __builtin_amdgcn_ballot_w64(need);
        if (lanes != 0) {                     // undecided for now: as if rejected
            if (lane4 == 0u)
                queue[nq] = make_uint4((uint32_t)z, (uint32_t)(R * 4 + k), (uint32_t)lanes, (uint32_t)(lanes >> 32));
            ++nq;
            r = need ? 1.0f : r;
        }
        const bool acc = r < 0.0f;
        pend[R][k] = acc ? tp : -1.0f;
        return ENERGY ? fix24(-fmaf(acc ? cp : co, Cx, (acc ? sp : so) * Sy)) : 0;
    }

    // The undecided update of queue entry i: the trial of update() from the angles in memory, decided by the exact test.
    __device__ __forceinline__ void settle(uint32_t i, const TBand* tb)
    {
        auto seg = __builtin_amdgcn_kernarg_segment_ptr();      // the launch's Lat3Args is its first argument
        asm volatile("" : "+s"(seg));
        const auto& A = *(const __attribute__((address_space(4))) Lat3Args*)seg;
        const int D = A.D, H = A.H, W = A.W;
        const int64_t wrow = (int64_t)W * 256;
        const uint4 qe = queue[i];
        const int z = __builtin_amdgcn_readfirstlane((int)qe.x), rk = __builtin_amdgcn_readfirstlane((int)qe.y);
        const int R = rk >> 2, k = rk & 3, P = (z + C) & 1;
        const int y = y0 + R, j = 2 * k + (R == 0 ? P : 1 - P), x = x0 + j;
        const bool pb = z > 0, pu = y > 0, pl_ = x > 0, pr = x + 1 < W, pd = y + 1 < H, pf = z + 1 < D;
        char* const p = S + (((int64_t)z * H + y) * W + x) * 256 + lane4;
        auto at = [&](int64_t off) { return *reinterpret_cast<const float*>(p + off); };
        const float to = at(0), nb = at(pb ? -wplane : 0), nu = at(pu ? -wrow : 0), nl = at(pl_ ? -256 : 0),
                    nr = at(pr ? 256 : 0), nd = at(pd ? wrow : 0), nf = at(pf ? wplane : 0);
        const uint32_t pair = ((uint32_t)z * (uint32_t)H + (uint32_t)y) * (uint32_t)A.Mw + (uint32_t)(x0 / 4 + (k >> 1));
        const U4 w = philox_site_s(pair, w3k1, pl, a.key0, a.key1);
        const float tp = u24((k & 1) ? w.z : w.x);
        const float u2 = u24((k & 1) ? w.w : w.y);
        const unsigned present = (pb ? 1u : 0u) | (pu ? 2u : 0u) | (pl_ ? 4u : 0u) | (pr ? 8u : 0u) | (pd ? 16u : 0u) |
                                 (pf ? 32u : 0u);
        const TBand T = entry(tb + ((int64_t)(z / A.lb_d) * A.nby + y / A.lb_h) * A.nbx + x / A.lb_w);
        bool acc = false;
        uint64_t left = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)qe.w) << 32 |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)qe.z);
        do {
            acc |= exact6_round(left, tp, to, nb, nu, nl, nr, nd, nf, present, A.two_pi_q, A.Jd, T.T, u2);
            for (int n = 0; n < 4; ++n) left &= left - 1;        // (of 0: 0)
        } while (left != 0);
        if (acc) *reinterpret_cast<float*>(p) = tp;
        if (ENERGY) {
            auto cosq = [&](bool here, float t) { return here ? cos_rev(a.q * t) : 0.0f; };
            auto sinq = [&](bool here, float t) { return here ? sin_rev(a.q * t) : 0.0f; };
            const float Cx = ((((cosq(pb, nb) + cosq(pu, nu)) + cosq(pl_, nl)) + cosq(pr, nr)) + cosq(pd, nd)) +
                             cosq(pf, nf);
            const float Sy = ((((sinq(pb, nb) + sinq(pu, nu)) + sinq(pl_, nl)) + sinq(pr, nr)) + sinq(pd, nd)) +
                             sinq(pf, nf);
            const int before = fix24(-fmaf(cos_rev(a.q * to), Cx, sin_rev(a.q * to) * Sy));
            const int after = fix24(-fmaf(cos_rev(a.q * tp), Cx, sin_rev(a.q * tp) * Sy));
            if (acc) e_acc += after - before;
        }
    }

    // the updates of row R on plane z, then the energy of the colour's sample sites
    template <int S0, int P, int R>
    __device__ __forceinline__ int row(int z)
    {
        const uint32_t g = gap[R];
        const uint32_t base = site + (R == 0 ? 0u : site1);
        int e = 0;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int j0 = 4 * m + (R == 0 ? P : 1 - P), j1 = j0 + 2;
            const bool g0 = (g >> (j0 + 1)) & 1u, g1 = (g >> (j1 + 1)) & 1u;
            if (!(g0 || g1)) continue;
            TBand Ta, Tb;
            if (AL) {
                Ta = R == 0 ? T0 : T1;
                Tb = Ta;
            } else {
                int xb = x0;
                asm volatile("" : "+s"(xb));
                Ta = entry((R == 0 ? t0 : t1) + block_column(xb + j0));
                Tb = entry((R == 0 ? t0 : t1) + block_column(xb + j1));
            }
            const U4 w = philox_site_s(base + (uint32_t)m, w3k1, pl, a.key0, a.key1);
            if (g0) e += update<S0, P, R>(Ta, z, 2 * m, w.x, w.y);
            if (g1) e += update<S0, P, R>(Tb, z, 2 * m + 1, w.z, w.w);
        }
        if (ENERGY && (R == 0 || d1 != 0)) {
            const uint32_t smp = colmask & ~g;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = 2 * k + (R == 0 ? P : 1 - P);
                if (!((smp >> (j + 1)) & 1u)) continue;
                float Cx, Sy;
                field<S0, P, R>(k, &Cx, &Sy);
                const float t = a.q * own[S0 & 1][R][k];
                e += fix24(-fmaf(cos_rev(t), Cx, sin_rev(t) * Sy));
            }
        }
        return e;
    }

    // one step (S0 = z & 3): plane z + 1 arrives, plane z - 1 is stored, the next loads are issued (planes past the grid
    // are replaced by the current one; they are cleared at the arrival or never used), plane z is updated
    template <int S0>
    __device__ __forceinline__ void step(int z)
    {
        constexpr int P = (S0 + C) & 1, SN = (S0 + 1) & 3;
        arrive<SN, 1 - P>(z + 1);
        flush<1 - P>(oz - wplane);
        const uint32_t g0 = ngap[0], g1 = ngap[1];
        const bool more = z + 1 < a.D;
        request_others<P>(z + 2 < a.D ? oz + 2 * wplane : oz);
        request_own<(S0 + 1) & 1, 1 - P>(more ? oz + wplane : oz, g0, g1);
        request_gaps(z + 2 < a.D ? cells + 2 * cellP : cells);
        int e = row<S0, P, 0>(z);
        e += row<S0, P, 1>(z);
        if (ENERGY) e_acc += e;
        pgap[0] = gap[0];
        pgap[1] = gap[1];
        gap[0] = g0;
        gap[1] = g1;
        oz += wplane;
        site += siteP;
        cells += cellP;
        if (++bzr == a.lb_d) {
            bzr = 0;
            t0 += tP;
            t1 += tP;
            if (AL && z + 1 < ze) load_temperatures();
        }
    }

    // planes [zb, ze) (zb a multiple of 4), in one stretch unless the queue fills: returns the plane reached.  oz, site,
    // cells, t0, t1 and bzr are those of plane zb.
    __device__ __forceinline__ int stretch(int zb)
    {
        constexpr int P = C & 1;
        nq = 0u;
        pl = philox_lane(real, sweep_index, a.key0, a.key1);
        pgap[0] = pgap[1] = 0u;
        if (AL) load_temperatures();
        request_others<1 - P>(zb > 0 ? oz - wplane : oz);
        arrive<3, 1 - P>(zb - 1);
        request_others<P>(oz);
        arrive<0, P>(zb);
        request_others<1 - P>(zb + 1 < a.D ? oz + wplane : oz);
        request_gaps(cells);
        gap[0] = ngap[0];
        gap[1] = ngap[1];
        request_own<0, P>(oz, gap[0], gap[1]);
        request_gaps(zb + 1 < a.D ? cells + cellP : cells);
        do {
            step<0>(zb++);
            if (zb < ze) step<1>(zb++);
            if (zb < ze) step<2>(zb++);
            if (zb < ze) step<3>(zb++);
        } while (zb < ze && nq <= kQueue3 - 32u);
        if ((zb - 1 + C) & 1) flush<1>(oz - wplane);     // the pending plane is zb - 1
        else flush<0>(oz - wplane);
        return zb;
    }
    uint32_t sweep_index;
};

// One launch is one colour of a sweep over all rows; a workgroup is one wave, work items (band, row pair, plane segment,
// group of realizations).
template <int C, bool ENERGY, bool AL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves3, kWaves3))) void k_sweep3(
    Lat3Args a, const uint32_t* __restrict__ cells, const TBand* __restrict__ tb, float* state,
    long long* __restrict__ epart)
{
    // XCD-aware order: workgroup g runs on XCD g % 8; consecutive items (adjacent bands, then adjacent rows, which read
    // each other's edge cells) go to the same XCD.
    const uint32_t N = (uint32_t)a.nrows * (uint32_t)a.nbands * (uint32_t)a.nzseg * (uint32_t)(a.Rp / 64);
    const uint32_t g = blockIdx.x, xcd = g & 7u, k = g >> 3;
    const uint32_t per = N >> 3, rem = N & 7u;
    const uint32_t item = xcd < rem ? xcd * (per + 1u) + k : rem * (per + 1u) + (xcd - rem) * per + k;
    if (item >= N) return;
    const uint32_t band = item % (uint32_t)a.nbands;
    uint32_t rest = item / (uint32_t)a.nbands;
    const uint32_t rows = rest % (uint32_t)a.nrows;
    rest /= (uint32_t)a.nrows;
    const uint32_t zseg = rest % (uint32_t)a.nzseg;
    const uint32_t rg = rest / (uint32_t)a.nzseg;
    const int64_t n_all = (int64_t)a.D * a.H * a.W;
    __shared__ uint4 queue[kQueue3];
    Wave3<C, ENERGY, AL> w;
    w.a = Loop3{a.D, a.lb_d, a.key0, a.key1, a.q, a.J, a.delta_e, a.W, a.lb_w, a.lbw_inv};
    w.S = reinterpret_cast<char*>(state) + (int64_t)rg * n_all * 256;
    w.queue = queue;
    w.x0 = (int)band * kB3;
    w.y0 = 2 * (int)rows;
    w.zs = (int)zseg * a.zseg;
    w.ze = w.zs + a.zseg < a.D ? w.zs + a.zseg : a.D;
    w.lane4 = threadIdx.x * 4u;
    const int lane = (int)(rg * 64 + threadIdx.x);
    w.real = a.real_offset + (uint32_t)lane;
    w.w3k1 = ctr_word3(a.scene, TAG_SWEEP, (uint32_t)C) ^ a.key1;
    w.sweep_index = a.sweep;
    const int wrow = a.W * 256;                       // sides up to 65535
    const bool has1 = w.y0 + 1 < a.H;
    w.wplane = (int64_t)a.H * wrow;
    w.d1 = has1 ? wrow : 0;
    w.dU = w.y0 > 0 ? -wrow : 0;
    w.dD = w.y0 + 2 < a.H ? 2 * wrow : 0;
    w.site1 = (uint32_t)a.Mw;
    w.siteP = (uint32_t)a.H * (uint32_t)a.Mw;
    w.cell1 = (uint32_t)a.nbands;
    w.cellP = (uint32_t)a.H * (uint32_t)a.nbands;
    w.tP = (int64_t)a.nby * a.nbx;
    w.colmask = 0u;
    for (int j = 0; j < kW3; ++j) {
        const int x = w.x0 - 1 + j;
        if (x >= 0 && x < a.W) w.colmask |= 1u << j;
    }
    w.colmask = __builtin_amdgcn_readfirstlane(w.colmask);
    w.e_acc = 0;
    const int bcol = AL ? w.block_column(w.x0) : 0;
    for (int z = w.zs; z < w.ze;) {
        const int64_t plane = (int64_t)z * a.H + w.y0;
        w.oz = (plane * a.W + w.x0) * 256;
        w.site = (uint32_t)plane * (uint32_t)a.Mw + (uint32_t)(w.x0 / 4);
        w.cells = cells + plane * a.nbands + band;
        const int bz = z / a.lb_d;
        w.bzr = z % a.lb_d;
        w.t0 = tb + ((int64_t)bz * a.nby + w.y0 / a.lb_h) * a.nbx + bcol;
        w.t1 = has1 ? tb + ((int64_t)bz * a.nby + (w.y0 + 1) / a.lb_h) * a.nbx + bcol : w.t0;
        z = w.stretch(z);
        // the notes are written by lane 0 and read by the wave, and written again after that
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t i = 0; i < w.nq; ++i) w.settle(i, tb);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (ENERGY && lane < a.R)
        epart[(int64_t)lane * ((int64_t)a.nrows * a.nbands * a.nzseg) + ((int64_t)rows * a.nbands + band) * a.nzseg +
              zseg] = w.e_acc;
}

// gap bits of each row's window columns (x0 - 1 .. x0 + kB3)
__global__ __launch_bounds__(256) void k_cells3(const uint8_t* __restrict__ mask, int64_t rows, int W, int nbands,
                                                 uint32_t* __restrict__ cells)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= rows * nbands) return;
    const int64_t r = i / nbands;
    const int band = (int)(i % nbands);
    uint32_t g = 0u;
    for (int j = 0; j < kW3; ++j) {
        const int x = band * kB3 - 1 + j;
        if (x >= 0 && x < W && !mask[r * W + x]) g |= 1u << j;
    }
    cells[i] = g;
}

// Eq. (2) per 3D block: one workgroup per block, its sites in a fixed order per thread, a fixed-order reduction

// (one workgroup per block, of 1024 threads for the larger ones; 160^3 in 32^3 blocks: 117 us, 336 us with 256 threads, cos
// and 64-bit divisions for every site)
template <int ST3_NT>
__global__ __launch_bounds__(ST3_NT) void k_block_stats3(const float* __restrict__ t, const uint8_t* __restrict__ mask,
                                                          int64_t D, int64_t H, int64_t W, int lb_d, int lb_h,
                                                          int lb_w, int nbx, int nby, double q, double J,
                                                          double* S, int* N, double* Ts, int* No)
{
    __shared__ double lds_d[ST3_NT / 64];
    __shared__ int lds_i[ST3_NT / 64];
    const int64_t b = blockIdx.x;
    const int bx = (int)(b % nbx), by = (int)((b / nbx) % nby), bz = (int)(b / ((int64_t)nbx * nby));
    const int64_t z0 = (int64_t)bz * lb_d, y0 = (int64_t)by * lb_h, x0 = (int64_t)bx * lb_w;
    const int64_t nz = (z0 + lb_d < D ? lb_d : D - z0), ny = (y0 + lb_h < H ? lb_h : H - y0),
                  nx = (x0 + lb_w < W ? lb_w : W - x0);
    const int64_t HW = H * W;
    double s = 0.0, ts = 0.0;
    int n = 0, no = 0;
    const bool in32 = nz * ny * nx <= 0xffffffffll;
    for (int64_t i = threadIdx.x; i < nz * ny * nx; i += ST3_NT) {
        const int64_t row = in32 ? (uint32_t)i / (uint32_t)nx : i / nx;
        const int64_t dz = in32 ? (uint32_t)row / (uint32_t)ny : row / ny;
        const int64_t z = z0 + dz, y = y0 + (row - dz * ny), x = x0 + (i - row * nx);
        const int64_t p = z * HW + y * W + x;
        if (!mask[p]) continue;
        const double tp = (double)t[p];
        ts += tp;
        ++no;
        if (x + 1 < W && mask[p + 1]) {
            s += -J * cos_turns(q, tp - (double)t[p + 1]);
            ++n;
        }
        if (y + 1 < H && mask[p + W]) {
            s += -J * cos_turns(q, tp - (double)t[p + W]);
            ++n;
        }
        if (z + 1 < D && mask[p + HW]) {
            s += -J * cos_turns(q, tp - (double)t[p + HW]);
            ++n;
        }
    }
    s = block_sum<ST3_NT>(s, lds_d);
    ts = block_sum<ST3_NT>(ts, lds_d);
    n = block_sum<ST3_NT>(n, lds_i);
    no = block_sum<ST3_NT>(no, lds_i);
    if (threadIdx.x == 0) {
        S[b] = s;
        N[b] = n;
        Ts[b] = ts;
        No[b] = no;
    }
}

// one half-sweep of the periodic reference lattice (every site free, J = 1), one chain per temperature: a thread
// per same-colour pair of a row, the neighbours read from memory
__global__ __launch_bounds__(256) void k_ref3_half(float* state, const float* Tgrid, int L, uint32_t sweep, int colour,
                                                    float q, float delta_e, uint32_t key0, uint32_t key1,
                                                    double two_pi_q)
{
    const int chain = blockIdx.y;
    const int Mw = (L + 3) / 4;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t rows = (int64_t)L * L;
    if (p >= rows * Mw) return;
    const int64_t row = p / Mw;
    const int m = (int)(p - row * Mw);
    const int z = (int)(row / L), y = (int)(row % L);
    const int xa = 4 * m + ((y + z + colour) & 1);
    if (xa >= L) return;
    const int64_t L2 = (int64_t)L * L;
    float* st = state + (int64_t)chain * L2 * L;
    const float T = Tgrid[chain];
    const TBand tbd = make_tband(T, 1.0f, delta_e);
    const U4 w = philox4x32_10((uint32_t)p, sweep, (uint32_t)chain, ctr_word3(0u, TAG_REFLAT, (uint32_t)colour), key0,
                               key1);
    const int zb = (z + L - 1) % L, zf = (z + 1) % L, yu = (y + L - 1) % L, yd = (y + 1) % L;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int x = xa + 2 * h;
        if (x >= L) break;
        const int xl = (x + L - 1) % L, xr = (x + 1) % L;
        float nb[6];
        nb[0] = st[zb * L2 + (int64_t)y * L + x];
        nb[1] = st[z * L2 + (int64_t)yu * L + x];
        nb[2] = st[z * L2 + (int64_t)y * L + xl];
        nb[3] = st[z * L2 + (int64_t)y * L + xr];
        nb[4] = st[z * L2 + (int64_t)yd * L + x];
        nb[5] = st[zf * L2 + (int64_t)y * L + x];
        float Cx = 0.0f, Sy = 0.0f;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const float an = q * nb[j];
            Cx += cos_rev(an);
            Sy += sin_rev(an);
        }
        const int64_t o = z * L2 + (int64_t)y * L + x;
        const float to = st[o];
        const float co = cos_rev(q * to), so = sin_rev(q * to);
        const float tpv = u24(h ? w.z : w.x);
        const uint32_t wa = h ? w.w : w.y;
        const float cp = cos_rev(q * tpv), sp = sin_rev(q * tpv);
        const float X = fmaf(cp - co, Cx, (sp - so) * Sy);
        int dec = filter32(X, (float)(wa >> 8), tbd, 1.0f, delta_e);
        if (dec < 0)
            dec = exact64_6(tpv, to, nb[0], nb[1], nb[2], nb[3], nb[4], nb[5], 63u, two_pi_q, 1.0, T, u24(wa)) ? 1 : 0;
        if (dec) st[o] = tpv;
    }
}

// per (part, chain): the sum over the part's sites of the energies of their +x, +y, +z bonds (periodic), FP64
__global__ __launch_bounds__(256) void k_ref3_energy(const float* __restrict__ state, int L, float q, double* partial)
{
    __shared__ double s_red[4];
    const int chain = blockIdx.y;
    const int64_t L2 = (int64_t)L * L, L3 = L2 * L;
    const float* st = state + (int64_t)chain * L3;
    double acc = 0.0;
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < L3; n += (int64_t)gridDim.x * 256) {
        const int64_t z = n / L2, y = (n / L) % L, x = n % L;
        const float tn = st[n];
        acc -= (double)cos_rev(q * (tn - st[z * L2 + y * L + (x + 1) % L]));
        acc -= (double)cos_rev(q * (tn - st[z * L2 + ((y + 1) % L) * L + x]));
        acc -= (double)cos_rev(q * (tn - st[((z + 1) % L) * L2 + y * L + x]));
    }
    const double tot = block_sum<256>(acc, s_red);
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.x * gridDim.y + chain] = tot;   // layout [part][chain]
}

}  // namespace

int64_t lat3_blocks(int64_t D, int64_t H, int64_t W, int lb_d, int lb_h, int lb_w)
{
    return ((D + lb_d - 1) / lb_d) * ((H + lb_h - 1) / lb_h) * ((W + lb_w - 1) / lb_w);
}

hipError_t launch_block_stats3(const float* t, const uint8_t* mask, int64_t D, int64_t H, int64_t W, int lb_d,
                               int lb_h, int lb_w, double two_pi_q, double J, double* S, int* N, double* Ts, int* No,
                               hipStream_t s)
{
    const int nbx = (int)((W + lb_w - 1) / lb_w), nby = (int)((H + lb_h - 1) / lb_h);
    const int64_t B = lat3_blocks(D, H, W, lb_d, lb_h, lb_w);
    const double q = (double)(float)(two_pi_q / (2.0 * kPi));        // (2 pi q, q an FP32 value)
    if ((int64_t)lb_d * lb_h * lb_w >= 4096)
        hipLaunchKernelGGL(k_block_stats3<1024>, dim3((unsigned)B), dim3(1024), 0, s, t, mask, D, H, W, lb_d, lb_h, lb_w,
                           nbx, nby, q, J, S, N, Ts, No);
    else
        hipLaunchKernelGGL(k_block_stats3<256>, dim3((unsigned)B), dim3(256), 0, s, t, mask, D, H, W, lb_d, lb_h, lb_w, nbx,
                           nby, q, J, S, N, Ts, No);
    return hipGetLastError();
}

int lat3_zseg(int64_t D, int64_t H, int64_t W, int R)
{
    const int64_t per = ((W + kB3 - 1) / kB3) * ((H + 1) / 2) * ((R + 63) / 64);
    auto planes = [&](int64_t n) { return (int)(((D + n - 1) / n + 3) / 4 * 4); };
    int64_t n = (D + kZSeg3 - 1) / kZSeg3;
        // at least 16384 waves (3072 run at once: the last round is then a small part), but 8 planes: a segment's first
    // two planes are loaded in vain (160^3, R = 128: 1.44 ms per sweep with 9600 waves, 1.40 with 16000)
    while (per * n < 16384 && planes(n) > 8) ++n;
    return planes(n);
}

hipError_t launch_cells3(const uint8_t* mask, int64_t D, int64_t H, int64_t W, int nbands, uint32_t* cells,
                         hipStream_t s)
{
    const int64_t rows = D * H;
    hipLaunchKernelGGL(k_cells3, dim3((unsigned)((rows * nbands + 255) / 256)), dim3(256), 0, s, mask, rows, (int)W,
                       nbands, cells);
    return hipGetLastError();
}

hipError_t launch_sweep3(const Lat3Args& a, const uint32_t* cells, const TBand* tb, float* state, long long* epart,
                         hipStream_t s)
{
    const int64_t N = (int64_t)a.nrows * a.nbands * a.nzseg * (a.Rp / 64);
    if (N <= 0) return hipSuccess;
    const dim3 grid((unsigned)N);
    const bool al = a.lb_w % kB3 == 0 || a.nbx == 1;
#define MPR_S3(CO, EN, AL) \
    hipLaunchKernelGGL((k_sweep3<CO, EN, AL>), grid, dim3(64), 0, s, a, cells, tb, state, epart)
    if (a.colour == 0) {                         // the energy is that of the colour-1 sites
        if (al) MPR_S3(0, false, true);
        else MPR_S3(0, false, false);
    } else if (epart) {
        if (al) MPR_S3(1, true, true);
        else MPR_S3(1, true, false);
    } else {
        if (al) MPR_S3(1, false, true);
        else MPR_S3(1, false, false);
    }
#undef MPR_S3
    return hipGetLastError();
}

hipError_t launch_ref3_half(float* state, const float* Tgrid, int nT, int L, uint32_t sweep, int colour, float q,
                            float delta_e, uint32_t key0, uint32_t key1, double two_pi_q, hipStream_t s)
{
    const int64_t np = (int64_t)L * L * ((L + 3) / 4);
    hipLaunchKernelGGL(k_ref3_half, dim3((unsigned)((np + 255) / 256), (unsigned)nT), dim3(256), 0, s, state, Tgrid, L,
                       sweep, colour, q, delta_e, key0, key1, two_pi_q);
    return hipGetLastError();
}

int ref3_energy_parts(int L)
{
    const int64_t n = (int64_t)L * L * L;
    const int64_t p = (n + 4095) / 4096;
    return (int)(p < 1 ? 1 : (p > 128 ? 128 : p));
}

hipError_t launch_ref3_energy(const float* state, int L, int nT, float q, double* partial, int nparts, hipStream_t s)
{
    hipLaunchKernelGGL(k_ref3_energy, dim3((unsigned)nparts, (unsigned)nT), dim3(256), 0, s, state, L, q, partial);
    return hipGetLastError();
}

}  // namespace mpr
