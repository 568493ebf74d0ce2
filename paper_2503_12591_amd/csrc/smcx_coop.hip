// Cooperative sweep kernels: G lanes share a trial.
//
// One lane per link cell leaves the chip idle where a mini-step has few link
// cells: a trial is a chain of about 120 dependent LDS reads and adds, and with
// fewer trials than the chip has lanes the sweep's time is that chain times the
// mini-steps.  Here half of a trial's G lanes count the active site's
// neighbours and half its partner's, each lane a few of them, all reads in
// flight at once; the packed counts meet by cross-lane adds, the terms of the
// integer dE are spread over the lanes again, and every lane of the group
// comes to the same decision.  The random numbers of G coming mini-steps are
// drawn at once, one per lane.  The decisions are those of the one-lane
// kernels, bit for bit: the same integer sum, the same tests, the same log.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "smcx_device.h"
#include "smcx_internal.h"
#include "smcx_launch.h"

namespace smcx {

// ---------------------------------------------------------------------------
// The neighbours of a site split over H lanes.  In a basis-planar window the
// neighbour at half-unit vector v of a basis-b site lies at
//   site + A(v) + delta(b, type(v)),
// A(v) its offset from a basis-0 site, type(v) the parity class of v (= the
// basis it leads to from basis 0): each odd component of v carries into the
// next conventional cell exactly when the site's own coordinate is odd.  So a
// site needs one base per type and a lane's A(v) hold for every basis.
// Slots: up to H neighbours of one shell and type, one per lane.
// ---------------------------------------------------------------------------
struct CoopSlot {
    int shell, type, n;
};
template <int H>
struct CoopSlots {
    int n;
    CoopSlot s[kMaxSumZ + 8];
    int32_t vec[kMaxSumZ + 8][H];  // (dx + 8) | (dy + 8) << 8 | (dz + 8) << 16 from a basis-0 site
};

template <int LAT, int H>
constexpr CoopSlots<H> make_coop_slots()
{
    const Geometry G = kGeom[LAT];
    CoopSlots<H> P{};
    P.n = 0;
    for (int s = 0; s < kMaxShells; ++s)
        for (int t = 0; t < G.m; ++t) {
            int fill = 0;
            for (int n = 0; n < G.Z[s]; ++n) {
                const Nb nb = nb_of(G, 0, G.v[s][n][0], G.v[s][n][1], G.v[s][n][2]);
                if (nb.bt != t) continue;
                if (fill == 0) {
                    P.s[P.n].shell = s;
                    P.s[P.n].type = t;
                }
                const int32_t w = (nb.dx + 8) | (nb.dy + 8) << 8 | (nb.dz + 8) << 16;
                // lanes past the slot's last neighbour read it again and add nothing
                for (int j = fill; j < H; ++j) P.vec[P.n][j] = w;
                P.s[P.n].n = ++fill;
                if (fill == H) {
                    ++P.n;
                    fill = 0;
                }
            }
            if (fill > 0) ++P.n;
        }
    return P;
}

// The slots of H = 1 (one neighbour each) in the order of the window rows they
// lie in.
struct CoopRows {
    int slot[kMaxSumZ + 8];
    bool first[kMaxSumZ + 8];  // the first of its row
};
template <int LAT>
constexpr CoopRows make_coop_rows(int n)
{
    const CoopSlots<1> P = make_coop_slots<LAT, 1>();
    CoopRows R{};
    auto key = [&P](int i) { return P.s[i].type << 16 | (P.vec[i][0] >> 8); };
    for (int i = 0; i < n; ++i) {
        int k = i;  // insertion by row, in place
        while (k > 0 && key(R.slot[k - 1]) > key(i)) {
            R.slot[k] = R.slot[k - 1];
            --k;
        }
        R.slot[k] = i;
    }
    for (int k = 0; k < n; ++k) R.first[k] = k == 0 || key(R.slot[k - 1]) != key(R.slot[k]);
    return R;
}

template <int LAT, int H>
__device__ const CoopSlots<H> kCoopSlots = make_coop_slots<LAT, H>();

constexpr int coop_slots_of(const CoopSlot* s, int n, int S)
{
    int c = 0;
    for (int i = 0; i < n; ++i) c += s[i].shell < S ? 1 : 0;
    return c;
}

// Sum over the G lanes of a group (every lane gets it); all of them active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp(uint64_t v)
{
    return (uint64_t)dpp<CTRL>((uint32_t)(v >> 32)) << 32 | dpp<CTRL>((uint32_t)v);
}
// cross-lane steps: within a quad xor 1 and xor 2; then lane i with 7 - i of
// its 8 lanes and 15 - i of its 16 (their quads / halves already hold sums)
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141, kMirror16 = 0x140;

template <int G, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    v += dpp<kXor1>(v);
    if constexpr (G >= 4) v += dpp<kXor2>(v);
    if constexpr (G >= 8) v += dpp<kMirror8>(v);
    if constexpr (G >= 16) v += dpp<kMirror16>(v);
    return v;
}

// A value of the group's other half (the same in all lanes of a half).
template <int G>
__device__ __forceinline__ uint32_t other_half(uint32_t v)
{
    if constexpr (G == 2) return dpp<kXor1>(v);
    else if constexpr (G == 4) return dpp<kXor2>(v);
    else if constexpr (G == 8) return dpp<kMirror8>(v);
    else return dpp<kMirror16>(v);
}

// One coming trial as drawn by one lane of the group: the two sites as packed
// words and the random words.  A site word holds the window byte (18 bits),
// whether the trial takes place (bit 18), the site's basis (19-20) and for
// each axis (21-26, two bits, signed) in which direction the window holds an
// image of it, one period away.
struct CoopDraw {
    uint32_t a, b;
    uint32_t w1, w2;
};
constexpr uint32_t kSiteMask = (1u << 18) - 1, kSiteActive = 1u << 18;

// Image direction of coordinate c on an axis of L cells whose halo the window
// holds: +1 within the halo's width of the low face, -1 of the high face.
__device__ __forceinline__ uint32_t image_code(int c, int L) { return c < kHalo ? 1u : (c >= L - kHalo ? 3u : 0u); }

template <int LAT, int E, int SS, int G>
struct Coop {
    using EN = Enc<E>;
    using CT = typename EN::T;
    static constexpr Geometry GM = kGeom[LAT];
    static constexpr int m = GM.m, Z1 = GM.Z[0], H = G / 2;
    static constexpr CoopSlots<H> SL = make_coop_slots<LAT, H>();
    static constexpr int NS = coop_slots_of(SL.s, SL.n, SS ? SS : kMaxShells);
    // terms of dE: SW shells by TW species at a time over the lanes (shells
    // first: a lane's shell is one pick for all its species' fields)
    static constexpr int SP = SS == 1 ? 1 : (SS == 2 ? 2 : 4), SW = G < SP ? G : SP, TW = G / SW;

    int j, side, jj;      // lane in the group, 0: active site / 1: partner, lane in the half
    int LP, PL, CP;       // window pitches: row, plane, basis column
    int off[H > 1 ? NS : 1];  // this lane's neighbour offsets (H = 1: formed in neighbours())
    CT one;               // a neighbour's count: +1 for the active site, -1 for its partner

    __device__ __forceinline__ void init()
    {
        j = threadIdx.x % G;
        side = j / H;
        jj = j % H;
        one = side ? (CT)0 - (CT)1 : (CT)1;
    }

    __device__ __forceinline__ void set_pitches(int lp, int pl, int cp)
    {
        LP = lp;
        PL = pl;
        CP = cp;
        if constexpr (H > 1) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int32_t v = kCoopSlots<LAT, H>.vec[i][jj];
                off[i] = ((v >> 16) - 8) * PL + (((v >> 8) & 0xff) - 8) * LP + ((v & 0xff) - 8) + SL.s[i].type * CP;
            }
        }
    }

    // Read the lane's share of the neighbours of its site (base: one per type).
    __device__ __forceinline__ void neighbours(const uint8_t* win, const int (&base)[m], int S, uint32_t (&v)[NS]) const
    {
        if constexpr (H > 1) {
#pragma unroll
            for (int i = 0; i < NS; ++i)
                if (SL.s[i].shell < S) v[i] = win[base[SL.s[i].type] + off[i]];
        } else {
            // every lane has the same vectors: the window rows they lie in
            // (type, dy, dz) get an address each, x goes into the offset
            // field of the reads
            int row = 0;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                constexpr CoopRows RO = make_coop_rows<LAT>(NS);
                const int i = RO.slot[k];
                const int32_t w = SL.vec[i][0];
                if (RO.first[k]) {
                    row = base[SL.s[i].type] + (((w >> 16) - 8) * PL + (((w >> 8) & 0xff) - 8) * LP + SL.s[i].type * CP - 2);
                    asm("" : "+v"(row));
                }
                if (SL.s[i].shell < S) v[i] = win[row + ((w & 0xff) - 6)];
            }
        }
    }

    // The same draw from lane i of the group, i fixed at compile time, for
    // groups within a quad.
    template <int I>
    __device__ __forceinline__ CoopDraw from_quad_lane(const CoopDraw& d) const
    {
        static_assert(G <= 4 && I < G, "a quad's lanes");
        constexpr int c = G == 4 ? I * 0x55 : (I | I << 2 | (2 + I) << 4 | (2 + I) << 6);
        CoopDraw o;
        o.a = dpp<c>(d.a);
        o.b = dpp<c>(d.b);
        o.w1 = dpp<c>(d.w1);
        o.w2 = dpp<c>(d.w2);
        return o;
    }

    // The same from lane i of the group (every lane of the wave calls this).
    __device__ __forceinline__ CoopDraw from_lane(const CoopDraw& d, int i) const
    {
        const int src = ((int)(threadIdx.x & 63) & ~(G - 1)) + i;
        CoopDraw o;
        o.a = (uint32_t)__shfl((int)d.a, src, 64);
        o.b = (uint32_t)__shfl((int)d.b, src, 64);
        o.w1 = (uint32_t)__shfl((int)d.w1, src, 64);
        o.w2 = (uint32_t)__shfl((int)d.w2, src, 64);
        return o;
    }

    // One trial; every lane of the group takes part.  Returns bit 0:
    // accepted, bit 1: near-tie, the same in all lanes, the swap written to
    // the window.  on_tie(accepted) logs a near-tie.
    template <typename OnTie>
    __device__ __forceinline__ int trial(uint8_t* win, const CoopDraw& d, double beta, int K, int S, int Lx, int Ly,
                                         int Lz, const int32_t* Q, float qscale, float qeps, const double* D,
                                         OnTie on_tie) const
    {
        const uint32_t me = side ? d.b : d.a;
        const int site = (int)(me & kSiteMask);
        int base[m];
        base[0] = site;
        if constexpr (LAT == SMCX_BCC) {
            base[1] = site + (me & (1u << 19) ? 1 + LP + PL - 2 * CP : 0);
        } else {
            // basis 1 is odd in x and y, 2 in x and z, 3 in y and z
            const uint32_t c = (me >> 19) & 3;
            const int fx = c == 1 || c == 2 ? 1 : 0, fy = c & 1 ? LP - 2 * CP : 0, fz = c & 2 ? PL - 4 * CP : 0;
            base[1] = site + fx + fy;
            base[2] = site + fx + fz;
            base[3] = site + fy + fz;
        }
        // the lane's site first, then its neighbours: the exchange of the
        // species and the table reads that need them go out while the
        // neighbours are still on their way
        const int own = win[site];
        uint32_t v[NS];
        neighbours(win, base, S, v);
        __builtin_amdgcn_sched_barrier(0);
        const int oth = (int)other_half<G>((uint32_t)own);
        const int p8 = side ? oth : own, q8 = side ? own : oth;
        const int pair = species_pair<E>(p8, q8, K);
        const int tj = TW > 1 ? j % TW : 0, sj = j / TW;
        constexpr int NT = (EN::KT + TW - 1) / TW, NSH = (kMaxShells + SW - 1) / SW;
        const int32_t* Qp = qtab_row<E>(Q, pair, S);
        const int32_t qbias = Qp[S * EN::KT];
        int32_t qv[NSH][NT];
#pragma unroll
        for (int a = 0; a < NSH; ++a)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int s = a * SW + sj, tt = t * TW + tj;
                qv[a][t] = 0;
                if (a * SW < S) {
                    const bool in = ((a + 1) * SW <= S || s < S) && ((t + 1) * TW <= EN::KT || tt < EN::KT);
                    const int32_t x = Qp[in ? s * EN::KT + tt : 0];
                    qv[a][t] = in ? x : 0;
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        CT acc[kMaxShells];
#pragma unroll
        for (int s = 0; s < kMaxShells; ++s) acc[s] = 0;
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (SL.s[i].shell < S) acc[SL.s[i].shell] += (SL.s[i].n == H || jj < SL.s[i].n ? one : (CT)0) << v[i];
        // counts of the active site minus the partner's, summed over the
        // group modulo 2^32 (or 2^64), then the field bias and the excluded
        // a-b bond: every field is non-negative, as in trial_finish
        CT dsh[kMaxShells];
#pragma unroll
        for (int s = 0; s < kMaxShells; ++s) {
            dsh[s] = 0;
            if (s < S) dsh[s] = group_sum<G, CT>(acc[s]) + EN::bias;
        }
        dsh[0] += ((CT)1 << p8) - ((CT)1 << q8);
        uint32_t part = j == 0 ? 0u - (uint32_t)qbias : 0u;
#pragma unroll
        for (int a = 0; a < NSH; ++a) {
            if (a * SW >= S) continue;
            // this lane's shell, picked among registers (the empty asm keeps
            // the compiler from indexing an array in memory instead)
            CT w = dsh[a * SW];
#pragma unroll
            for (int k = 1; k < SW; ++k) {
                CT x = dsh[a * SW + k];
                asm("" : "+v"(x));
                w = sj >= k ? x : w;
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
                part += (uint32_t)__mul24((int)((w >> ((EN::F * (t * TW + tj)) & (8 * sizeof(CT) - 1))) & EN::mask), qv[a][t]);
        }
        const uint32_t qacc = group_sum<G, uint32_t>(part);
        int f = 0;
        if (p8 != q8) {
            f = metropolis<E>(qacc, qscale, qeps, D, pair, dsh[0], dsh[1], dsh[2], dsh[3], K, S, beta, d.w1, d.w2);
            if (f & 2) on_tie(f & 1);
        }
        if (f & 1) {
            // the lane's site takes the other's species; its images are
            // spread over the half's lanes
            const int cx = (int)(me << 9) >> 30, cy = (int)(me << 7) >> 30, cz = (int)(me << 5) >> 30;
            const int sx = __mul24(cx, Lx), sy = __mul24(cy, Ly * LP), sz = __mul24(cz, Lz * PL);
            const int have = (cx & 1) | (cy & 1) << 1 | (cz & 1) << 2;
            if constexpr (H == 8) {
                if ((jj & have) == jj) win[site + (jj & 1 ? sx : 0) + (jj & 2 ? sy : 0) + (jj & 4 ? sz : 0)] = (uint8_t)oth;
            } else {
                if (jj == 0) win[site] = (uint8_t)oth;
                if (have)
#pragma unroll
                    for (int i0 = 0; i0 < 8; i0 += H) {
                        const int im = i0 + jj;
                        if (im != 0 && (im & have) == im)
                            win[site + (im & 1 ? sx : 0) + (im & 2 ? sy : 0) + (im & 4 ? sz : 0)] = (uint8_t)oth;
                    }
            }
        }
        return f;
    }
};

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Block barrier between mini-steps; a workgroup of one wave only needs its LDS
// accesses kept in order.
__device__ __forceinline__ void step_barrier(bool waves)
{
    if (waves) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// Resident sweeps: a workgroup holds one whole replica in LDS (basis-planar
// rows, 2-cell periodic halo on every axis) for all sweeps and mini-steps of a
// call, reading it from the natural layout once and writing it back once.
// Mini-steps are ordered by workgroup barriers only.  Needs every edge >= 4
// (a site then has at most one image per axis and no partner has images in
// other shells) and the replica within the LDS.
// Small replicas are bound by the trial's chain (LDS reads, cross-lane adds,
// the table reads, the write, the barrier: 0.55 us per mini-step at 8 link
// cells, 16 lanes each), large ones by the CU's LDS and VALU issue (2.9 us at
// 512 link cells, 2 lanes each).  Against tile windows staged anew for every
// offset, one lane per trial: BCC 8^3 588 -> 67 us per sweep, FCC 18x13x11
// 3150 -> 390 us; against row launches 256 BCC 32^3 replicas 570 -> 370 us.
// ---------------------------------------------------------------------------
constexpr int kResidentBlock = 1024;

template <int LAT, int E, int SS, int G>
__global__ __launch_bounds__(kResidentBlock) void k_resident(SweepArgs A)
{
    using CO = Coop<LAT, E, SS, G>;
    constexpr int m = CO::m, F = Enc<E>::F;
    extern __shared__ __align__(16) uint8_t smem[];
    const int r = blockIdx.x;
    const RepDev& rep = rep_of(A, r);
    const int K = A.K, S = SS ? SS : A.S;
    const int Lx = scalar(rep.L[0]), Ly = scalar(rep.L[1]), Lz = scalar(rep.L[2]);
    const int CP = Lx + 2 * kHalo, LP = m * CP, WY = Ly + 2 * kHalo, WZ = Lz + 2 * kHalo, PL = LP * WY;
    int32_t* Q = (int32_t*)smem;
    int32_t* pdt = (int32_t*)(smem + A.lds_pd);
    int32_t* org = (int32_t*)(smem + A.lds_offb);
    uint8_t* win = smem + A.lds_win;
    const int nQ = qtab_entries(K, S);
    for (int i = threadIdx.x; i < nQ; i += blockDim.x) Q[i] = A.Qtab[i];
    for (int i = threadIdx.x; i < m * CO::Z1; i += blockDim.x) pdt[i] = ((const int32_t*)A.pdisp)[i];
    const int ncx = scalar(rep.nc[0]), ncy = scalar(rep.nc[1]), ncz = scalar(rep.nc[2]), ncell = ncx * ncy * ncz;
    for (int i = threadIdx.x; i < ncx + ncy + ncz + 3; i += blockDim.x) org[i] = A.origins[rep.cs_off + i];
    const float qscale = __int_as_float(ld_const(A.Qtab, nQ)), qeps = __int_as_float(ld_const(A.Qtab, nQ + 1));
    uint8_t* occ = A.occ + rep.occ_off;
    // natural cells (m bytes each) -> window columns, halo cells wrapped
    using Cell = typename std::conditional<m == 4, uint32_t, uint16_t>::type;
    const bool aligned = ((uintptr_t)occ % m) == 0;
    for (int c = threadIdx.x; c < CP * WY * WZ; c += blockDim.x) {
        const int wx = c % CP, wr = c / CP, wy = wr % WY, wz = wr / WY;
        int x = wx - kHalo, y = wy - kHalo, z = wz - kHalo;
        x += x < 0 ? Lx : (x >= Lx ? -Lx : 0);
        y += y < 0 ? Ly : (y >= Ly ? -Ly : 0);
        z += z < 0 ? Lz : (z >= Lz ? -Lz : 0);
        const uint8_t* src = occ + (int64_t)m * (x + Lx * (y + Ly * z));
        uint32_t cell = 0;
        if (aligned) {
            cell = *(const Cell*)src;
        } else {
#pragma unroll
            for (int b = 0; b < m; ++b) cell |= (uint32_t)src[b] << (8 * b);
        }
        uint8_t* dst = win + wr * LP + wx;
#pragma unroll
        for (int b = 0; b < m; ++b) dst[b * CP] = (uint8_t)(((cell >> (8 * b)) & 0xff) * F);
    }
    __syncthreads();
    CO co;
    co.init();
    co.set_pitches(LP, PL, CP);
    const int ngrp = blockDim.x / G, grp = threadIdx.x / G;
    const bool single = ncell <= ngrp, waves = blockDim.x > 64;
    // mini-steps drawn together: G when a group keeps its cell, else the
    // mini-steps between two barriers
    const int nbat = single ? G : A.nb;
    const int npass = scalar(single ? 1 : (ncell + ngrp - 1) / ngrp);
    const int Mx = scalar(rep.M[0]), My = scalar(rep.M[1]), MxM = Mx * m, MxyM = MxM * My;
    const int tau_end = min(A.tau_end, scalar(rep.nA));
    const uint32_t first = A.sweep_counter ? *A.sweep_counter : A.first_sweep;
    const int32_t *oy_ = org + ncx + 1, *oz_ = oy_ + ncy + 1;
    // quotients of mini-steps and cells (both far below 2^22, so the float
    // quotient of x + 1/2 rounds down to the right integer)
    auto quot = [](int x, float inv) { return (int)(((float)x + 0.5f) * inv); };
    const float i_xyM = 1.0f / (float)MxyM, i_xM = 1.0f / (float)MxM, i_ncx = 1.0f / (float)ncx, i_ncy = 1.0f / (float)ncy;
    int x0, y0, z0, ex, ey, ez;
    bool have;
    auto take_cell = [&](int cell) {
        have = cell < ncell;
        const int cc = have ? cell : 0;
        const int cr = quot(cc, i_ncx), cx = cc - cr * ncx, cz = quot(cr, i_ncy), cy = cr - cz * ncy;
        x0 = org[cx];
        ex = org[cx + 1] - x0;
        y0 = oy_[cy];
        ey = oy_[cy + 1] - y0;
        z0 = oz_[cz];
        ez = oz_[cz + 1] - z0;
    };
    // the site of mini-step tau in this group's cell; false when the cell sits it out
    auto site_of = [&](int tau, int& x, int& y, int& z, int& b) {
        const int oz = quot(tau, i_xyM), tr = tau - oz * MxyM, oy = quot(tr, i_xM), t2 = tr - oy * MxM, ox = t2 / m;
        b = t2 % m;
        x = x0 + ox;
        y = y0 + oy;
        z = z0 + oz;
        return have && ox < ex && oy < ey && oz < ez;
    };
    take_cell(grp);
    Stats st;
    for (int js = 0; js < A.n_sweeps; ++js) {
        const uint32_t t = first + (uint32_t)js;
        const double beta = ld_const(A.beta, (int64_t)js * A.beta_stride + r);
        for (int t0 = A.tau_begin / A.nb * A.nb; t0 < tau_end; t0 += nbat) {
            for (int pass = 0; pass < npass; ++pass) {
                if (npass > 1) take_cell(pass * ngrp + grp);
                CoopDraw mine;
                {
                    // lane i draws for mini-step t0 + i
                    const int tau = t0 + (single ? co.j : co.j % nbat);
                    int x, y, z, b;
                    const bool has = site_of(tau, x, y, z, b) && tau >= A.tau_begin && tau < tau_end;
                    uint32_t w0, w3;
                    philox4x32_10((uint32_t)(b + m * (x + Lx * (y + Ly * z))), 0u, t, (uint32_t)r, (uint32_t)A.seed,
                                  (uint32_t)(A.seed >> 32), w0, mine.w1, mine.w2, w3);
                    (void)w3;
                    const int pd = pdt[b * CO::Z1 + (int)__umulhi(w0, (uint32_t)CO::Z1)];
                    const int dx = (int8_t)pd, dy = (int8_t)(pd >> 8), dz = (int8_t)(pd >> 16), bt = pd >> 24;
                    const int la = (z + kHalo) * PL + (y + kHalo) * LP + x + kHalo + b * CP;
                    const int lb = la + dz * PL + dy * LP + dx + (bt - b) * CP;
                    // a cell that sits the mini-step out: its offset may lie past
                    // the lattice, and the byte there must not reach into the flags
                    mine.a = ((uint32_t)la & kSiteMask) | (has ? kSiteActive : 0u) | (uint32_t)b << 19 |
                             image_code(x, Lx) << 21 | image_code(y, Ly) << 23 | image_code(z, Lz) << 25;
                    mine.b = (uint32_t)lb | (uint32_t)bt << 19 | image_code(x + dx, Lx) << 21 |
                             image_code(y + dy, Ly) << 23 | image_code(z + dz, Lz) << 25;
                }
                auto step = [&](const CoopDraw& d, int i) {
                    if (d.a & kSiteActive) {
                        const int f = co.trial(win, d, beta, K, S, Lx, Ly, Lz, Q, qscale, qeps, A.Dtab, [&](int acc) {
                            if (co.j != 0) return;
                            int x, y, z, b;
                            (void)site_of(t0 + i, x, y, z, b);
                            log_tie(A, r, t, b + m * (x + Lx * (y + Ly * z)), acc);
                        });
                        ++st.att;
                        st.acc += f & 1;
                        st.tie += f >> 1;
                    }
                    // a group's later mini-steps read what this one wrote
                    if (single && (A.nb == 1 || (i + 1) % m == 0)) step_barrier(waves);
                };
                if constexpr (G <= 4) {
                    step(co.template from_quad_lane<0>(mine), 0);
                    if (nbat > 1) step(co.template from_quad_lane<1>(mine), 1);
                    if constexpr (G == 4) {
                        if (nbat > 2) step(co.template from_quad_lane<2>(mine), 2);
                        if (nbat > 3) step(co.template from_quad_lane<3>(mine), 3);
                    }
                } else {
                    CoopDraw next = co.from_lane(mine, 0);
                    for (int i = 0; i < nbat; ++i) {
                        const CoopDraw d = next;
                        next = co.from_lane(mine, min(i + 1, nbat - 1));
                        step(d, i);
                    }
                }
            }
            if (npass > 1) __syncthreads();
        }
        // one workgroup counts every trial of the call: the 32-bit sums go out
        // before 2^30 of them (a sweep tries each of at most 160 K sites once)
        if ((js & 4095) == 4095 || js + 1 == A.n_sweeps) {
            if (co.j != 0) st = Stats();  // the group's lanes counted alike
            __syncthreads();
            flush_stats_block(A, r, st);
        }
    }
    for (int c = threadIdx.x; c < Lx * Ly * Lz; c += blockDim.x) {
        const int x = c % Lx, cr = c / Lx, y = cr % Ly, z = cr / Ly;
        const uint8_t* src = win + ((z + kHalo) * WY + (y + kHalo)) * LP + x + kHalo;
        uint8_t* dst = occ + (int64_t)m * c;
        uint32_t cell = 0;
#pragma unroll
        for (int b = 0; b < m; ++b) cell |= (uint32_t)species_of(src[b * CP], F) << (8 * b);
        if (aligned) {
            *(Cell*)dst = (Cell)cell;
        } else {
#pragma unroll
            for (int b = 0; b < m; ++b) dst[b] = (uint8_t)(cell >> (8 * b));
        }
    }
}

// ---------------------------------------------------------------------------
// Row windows with G lanes per trial: the schedule, windows and write-back of
// k_rows (one launch per (o_y, o_z) group, whole rows of link cells per
// workgroup), for launches with too few link cells to fill the chip.  Bound by
// latency: of the 13 us of a BCC 64^3 launch (8 mini-steps, 16 lanes per
// trial; 24 us with one lane) 2.8 are an empty launch, 4.8 the chain of
// argument, table and window reads and the write-back, 0.54 each mini-step.
// ---------------------------------------------------------------------------
template <int LAT, int E, int SS, int G>
__global__ __launch_bounds__(kMaxCoopRowBlock) void k_rows_coop(SweepArgs A)
{
    using CO = Coop<LAT, E, SS, G>;
    using Geo = GeoRow<SS>;
    constexpr int m = CO::m;
    extern __shared__ __align__(16) uint8_t smem[];
    const int K = A.K, S = SS ? SS : A.S;
    int32_t* Q = (int32_t*)smem;
    int32_t* pdt = (int32_t*)(smem + A.lds_pd);
    uint8_t* win = smem + A.lds_win;
    const int nQ = qtab_entries(K, S);
    for (int i = threadIdx.x; i < nQ; i += blockDim.x) Q[i] = A.Qtab[i];
    for (int i = threadIdx.x; i < m * CO::Z1; i += blockDim.x) pdt[i] = ((const int32_t*)A.pdisp)[i];
    const float qscale = __int_as_float(ld_const(A.Qtab, nQ)), qeps = __int_as_float(ld_const(A.Qtab, nQ + 1));
    const int64_t total = ld_const(A.tile_off, A.R);  // row groups of all replicas
    const int64_t W = gridDim.x / 8;
    const int64_t chunk = (total + 7) / 8;
    const int64_t lo = (blockIdx.x % 8) * chunk;
    const int64_t hi = min(lo + chunk, total);
    CO co;
    co.init();
    const int T0 = A.T[0], T1 = A.T[1], T2 = A.T[2];
    const int l = threadIdx.x / G;
    const int lx = l % T0, ly = (l / T0) % T1, lz = l / (T0 * T1);
    const bool waves = blockDim.x > 64;
    const uint32_t t = A.sweep_counter ? *A.sweep_counter + A.first_sweep : A.first_sweep;
    Stats st;
    int r_stats = -1;
    __syncthreads();  // the tables are in place
    for (int64_t i = lo + blockIdx.x / 8; i < hi; i += W) {
        int a = 0, z = A.R - 1;  // last replica with tile_off[r] <= i
        while (a < z) {
            const int mid = (a + z + 1) >> 1;
            if (ld_const(A.tile_off, mid) <= i) a = mid; else z = mid - 1;
        }
        int r = a;
        int64_t grp = i - ld_const(A.tile_off, a);
        uniform(r, grp);
        const RepDev& rep = rep_of(A, r);
        const int Mx = scalar(rep.M[0]), My = scalar(rep.M[1]);
        int g0 = A.g, gn = A.nb;
        if (A.gq >= 0) {
            // this replica's q-th (o_y, o_z) group, every offset o_x and basis site
            if (A.gq >= My * rep.M[2]) continue;
            gn = m * Mx;
            g0 = A.gq * gn;
        }
        if (g0 >= rep.nA) continue;
        const int rest = g0 / m / Mx, oy = rest % My, oz = rest / My;
        const int gy = (int)grp % rep.rg[0], gz = (int)grp / rep.rg[0];
        TileGeom tg;
        tg.c0[0] = 0;
        tg.c1[0] = rep.nc[0];
        tg.c0[1] = gy * T1;
        tg.c1[1] = min(tg.c0[1] + T1, rep.nc[1]);
        tg.c0[2] = gz * T2;
        tg.c1[2] = min(tg.c0[2] + T2, rep.nc[2]);
        if (oy >= rep.emin[1] || oz >= rep.emin[2]) {
            // uneven partitions: row groups without a cell row active at
            // these offsets are skipped before staging
            bool any_y = false, any_z = false;
            for (int c = tg.c0[1]; c < tg.c1[1]; ++c)
                any_y |= cell_origin<Geo>(A, rep, 1, c + 1) - cell_origin<Geo>(A, rep, 1, c) > oy;
            for (int c = tg.c0[2]; c < tg.c1[2]; ++c)
                any_z |= cell_origin<Geo>(A, rep, 2, c + 1) - cell_origin<Geo>(A, rep, 2, c) > oz;
            if (!(any_y && any_z)) continue;
        }
        tg.w0[0] = -kHalo;
        tg.n[0] = rep.L[0] + 2 * kHalo;
        tg.gx0 = 0;
        const int oo[3] = {0, oy, oz};
#pragma unroll
        for (int ax = 1; ax < 3; ++ax) {
            tg.w0[ax] = cell_origin<Geo>(A, rep, ax, tg.c0[ax]) + oo[ax] - kHalo;
            const int w1 = min(cell_origin<Geo>(A, rep, ax, tg.c1[ax] - 1) + oo[ax] + kHalo + 1, rep.L[ax] + kHalo);
            tg.n[ax] = w1 - tg.w0[ax];
        }
        if (tg.n[1] <= 0 || tg.n[2] <= 0) continue;
        lds_barrier();  // every lane is done with the previous window
        stage_async<LAT, Geo>(A, rep, tg, A.ws + rep.pad_off, win);
        // this group's cell and first draws while the loads fly
        const int Lx = scalar(rep.L[0]), Ly = scalar(rep.L[1]);
        const int LP = A.LP, PL = LP * A.WY, CP = scalar(rep.cp);
        co.set_pitches(LP, PL, CP);
        const int cx = lx, cy = tg.c0[1] + ly, cz = tg.c0[2] + lz;
        const bool row_in = lz < T2 && cy < tg.c1[1] && cz < tg.c1[2];
        const bool in = row_in && cx < tg.c1[0];
        int x0 = 0, ex = 0, y = 0, z0 = 0;
        bool row_yz = false;
        if (row_in) {
            const int y0 = cell_origin<Geo>(A, rep, 1, cy), ey = cell_origin<Geo>(A, rep, 1, cy + 1) - y0;
            const int zc = cell_origin<Geo>(A, rep, 2, cz), ez = cell_origin<Geo>(A, rep, 2, cz + 1) - zc;
            // the cell row has active sites at (o_y, o_z)
            row_yz = oy < ey && oz < ez;
            y = y0 + oy;
            z0 = zc + oz;
        }
        if (in) {
            x0 = cell_origin<Geo>(A, rep, 0, cx);
            ex = row_yz ? cell_origin<Geo>(A, rep, 0, cx + 1) - x0 : 0;
        }
        const int64_t yz_site = (int64_t)m * Lx * ((int64_t)y + (int64_t)Ly * z0);
        const int row_byte0 = ((z0 - tg.w0[2]) * A.WY + (y - tg.w0[1])) * LP + kHalo;
        const double beta = ld_const(A.beta, r);
        const int tau1 = g0 + gn, ox0 = (g0 / m) % Mx;
        // lane i draws for mini-step tau + i
        auto draw = [&](int tau) {
            const int tt = tau + co.j, b = tt % m, ox = ox0 + (tt / m - g0 / m), x = x0 + ox;
            const bool has = ox < ex && tt < tau1;
            const int64_t site = yz_site + (b + m * x);
            CoopDraw d;
            uint32_t w0, w3;
            philox4x32_10((uint32_t)site, (uint32_t)((uint64_t)site >> 32), t, (uint32_t)r, (uint32_t)A.seed,
                          (uint32_t)(A.seed >> 32), w0, d.w1, d.w2, w3);
            (void)w3;
            const int pd = pdt[b * CO::Z1 + (int)__umulhi(w0, (uint32_t)CO::Z1)];
            const int dx = (int8_t)pd, dy = (int8_t)(pd >> 8), dz = (int8_t)(pd >> 16), bt = pd >> 24;
            const int la = row_byte0 + x + b * CP, lb = la + dz * PL + dy * LP + dx + (bt - b) * CP;
            // the window holds images along x only
            d.a = (uint32_t)(has ? la : 0) | (has ? kSiteActive : 0u) | (uint32_t)b << 19 | image_code(x, Lx) << 21;
            d.b = (uint32_t)(has ? lb : 0) | (uint32_t)bt << 19 | image_code(x + dx, Lx) << 21;
            return d;
        };
        CoopDraw mine = draw(g0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (r != r_stats) {
            if (co.j != 0) st = Stats();
            flush_stats_block(A, r_stats, st);
            r_stats = r;
        }
        for (int tau = g0; tau < tau1; tau += G) {
            if (tau != g0) mine = draw(tau);
            const int n = min(G, tau1 - tau);
            auto step = [&](const CoopDraw& d, int k) {
                if (d.a & kSiteActive) {
                    const int f = co.trial(win, d, beta, K, S, Lx, 0, 0, Q, qscale, qeps, A.Dtab, [&](int acc) {
                        if (co.j != 0) return;
                        const int tt = tau + k;
                        log_tie(A, r, t, yz_site + (tt % m + m * (x0 + ox0 + (tt / m - g0 / m))), acc);
                    });
                    ++st.att;
                    st.acc += f & 1;
                    st.tie += f >> 1;
                }
                // the next offset's trials read what this one wrote
                if ((tau + k + 1) % m == 0) step_barrier(waves);
            };
            if constexpr (G <= 4) {
                step(co.template from_quad_lane<0>(mine), 0);
                if (n > 1) step(co.template from_quad_lane<1>(mine), 1);
                if constexpr (G == 4) {
                    if (n > 2) step(co.template from_quad_lane<2>(mine), 2);
                    if (n > 3) step(co.template from_quad_lane<3>(mine), 3);
                }
            } else {
                CoopDraw next = co.from_lane(mine, 0);
                for (int k = 0; k < n; ++k) {
                    const CoopDraw d = next;
                    next = co.from_lane(mine, min(k + 1, n - 1));
                    step(d, k);
                }
            }
        }
        __syncthreads();  // every trial's window writes are visible
        if (row_yz)
            rows_writeback<LAT, Geo>(A, rep, tg, lx * G + co.j, T0 * G, y, z0, A.ws + rep.pad_off, win);
    }
    if (co.j != 0) st = Stats();
    flush_stats_block(A, r_stats, st);
}

// Kernels with a compile-time shell count for 32-bit counters (up to 6
// species), a runtime one for 64-bit counters.
template <bool ROWS, int LAT, int E, int SS, int G>
static const void* coop_kernel_s()
{
    if constexpr (ROWS) return (const void*)k_rows_coop<LAT, E, SS, G>;
    else return (const void*)k_resident<LAT, E, SS, G>;
}

template <bool ROWS, int LAT, int E, int G>
static const void* coop_kernel_e(int S)
{
    return S == 1   ? coop_kernel_s<ROWS, LAT, E, 1, G>()
           : S == 2 ? coop_kernel_s<ROWS, LAT, E, 2, G>()
           : S == 3 ? coop_kernel_s<ROWS, LAT, E, 3, G>()
                    : coop_kernel_s<ROWS, LAT, E, 4, G>();
}

template <bool ROWS, int LAT, int G>
static const void* coop_kernel_l(int K, int S)
{
    return K <= 4   ? coop_kernel_e<ROWS, LAT, 1, G>(S)
           : K == 5 ? coop_kernel_e<ROWS, LAT, 3, G>(S)
           : K == 6 ? coop_kernel_e<ROWS, LAT, 4, G>(S)
                    : coop_kernel_s<ROWS, LAT, 2, 0, G>();
}

template <bool ROWS>
static const void* coop_kernel(int lattice, int K, int S, int lanes)
{
    if (lattice == SMCX_BCC)
        return lanes == 16 ? coop_kernel_l<ROWS, SMCX_BCC, 16>(K, S)
                           : (lanes == 8 ? coop_kernel_l<ROWS, SMCX_BCC, 8>(K, S)
                                         : (lanes == 4 ? coop_kernel_l<ROWS, SMCX_BCC, 4>(K, S)
                                                       : coop_kernel_l<ROWS, SMCX_BCC, 2>(K, S)));
    return lanes == 16 ? coop_kernel_l<ROWS, SMCX_FCC, 16>(K, S)
                       : (lanes == 8 ? coop_kernel_l<ROWS, SMCX_FCC, 8>(K, S) : coop_kernel_l<ROWS, SMCX_FCC, 4>(K, S));
}

const void* resident_kernel(int lattice, int K, int S, int lanes) { return coop_kernel<false>(lattice, K, S, lanes); }
const void* row_coop_kernel(int lattice, int K, int S, int lanes) { return coop_kernel<true>(lattice, K, S, lanes); }

}  // namespace smcx
