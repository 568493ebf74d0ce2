// gfx950 kernels of libsmcx: link-cell parallel swap Metropolis sweeps with a
// multi-shell EPI energy over row and tile windows (sweeps with several lanes
// per trial, pair counts, the qSRO model and local energies have files of their
// own), packing, energies, replica exchange, and helpers.
//
// Trial (one lane per link cell of a tile):
//   1. Philox4x32-10 on counter (site, sweep, replica) gives the partner
//      direction k and the uniform u (Methods, "Random number generator"
//      bullet: one draw per trial);
//   2. the tile window around the active sites is staged from the padded
//      HBM copy into LDS with 16-byte loads, species stored pre-shifted
//      (F * sigma) so that a neighbour costs one LDS byte read and one
//      shift-add into a packed per-shell counter (F = 8 or 6 bits per species);
//   3. dE = sum_s sum_t (n_a - n_b)[s][t] * (V_s[q][t] - V_s[p][t]) in binary64
//      from the integer counters, s and t ascending, the a-b bond excluded
//      (Methods, "The EPI and qSRO model": the energy change of a pair model
//      is twice the change of the two local energies);
//   4. Metropolis test (Supplementary, acceptance equation), near-ties within
//      1e-12 logged; accepted swaps write two bytes (and their halo images)
//      straight to HBM.
// The trials of one mini-step are independent (Results, LIZ / LIZ+
// argument), so a mini-step is one grid-wide wave of independent lanes and
// mini-steps are ordered by launch order or by workgroup barriers.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "smcx_internal.h"
#include "smcx_device.h"
#include "smcx_launch.h"

namespace smcx {

// Padded copies of a replica: rows of conventional cells with a 2-cell
// periodic halo on every axis.  Interleaved rows hold the m basis sites of a
// cell side by side (byte m * (x + H) + b); basis-planar rows hold one column
// per basis site (byte b * cp + x + H), so that neighbouring link cells' sites
// of one basis are 4 bytes apart and a wave's LDS reads of them fall into
// distinct banks.
template <bool PLANAR>
__device__ __forceinline__ int row_byte(const RepDev& rep, int m, int x, int b)
{
    return PLANAR ? b * rep.cp + x + kHalo : m * (x + kHalo) + b;
}

// Write one species value to a site and to every periodic image of it that
// lies inside the padded copy.
template <bool PLANAR>
__device__ __forceinline__ void store_site(uint8_t* pad, const RepDev& rep, int m, int x, int y, int z,
                                           int b, uint8_t v)
{
    const int prow = PLANAR ? rep.prowp : rep.prow;
    if (x >= kHalo && x < rep.L[0] - kHalo && y >= kHalo && y < rep.L[1] - kHalo && z >= kHalo &&
        z < rep.L[2] - kHalo) {
        // away from the faces a site has no other image
        pad[((int64_t)(z + kHalo) * rep.prows + (y + kHalo)) * prow + row_byte<PLANAR>(rep, m, x, b)] = v;
        return;
    }
    int xs[3], ys[3], zs[3];
    int nx = 0, ny = 0, nz = 0;
    xs[nx++] = x;
    if (x < kHalo) xs[nx++] = x + rep.L[0];
    if (x >= rep.L[0] - kHalo) xs[nx++] = x - rep.L[0];
    ys[ny++] = y;
    if (y < kHalo) ys[ny++] = y + rep.L[1];
    if (y >= rep.L[1] - kHalo) ys[ny++] = y - rep.L[1];
    zs[nz++] = z;
    if (z < kHalo) zs[nz++] = z + rep.L[2];
    if (z >= rep.L[2] - kHalo) zs[nz++] = z - rep.L[2];
    for (int iz = 0; iz < nz; ++iz)
        for (int iy = 0; iy < ny; ++iy) {
            uint8_t* row = pad + ((int64_t)(zs[iz] + kHalo) * rep.prows + (ys[iy] + kHalo)) * prow;
            for (int ix = 0; ix < nx; ++ix) row[row_byte<PLANAR>(rep, m, xs[ix], b)] = v;
        }
}

// Smallest cell offset on each axis and smallest basis index over the
// neighbours (all shells) of a basis-b site.
constexpr Nb min_components(const Geometry& G, int b)
{
    Nb r{0, 0, 0, b};
    for (int s = 0; s < kMaxShells; ++s)
        for (int n = 0; n < G.Z[s]; ++n) {
            const Nb nb = nb_of(G, b, G.v[s][n][0], G.v[s][n][1], G.v[s][n][2]);
            r.dx = nb.dx < r.dx ? nb.dx : r.dx;
            r.dy = nb.dy < r.dy ? nb.dy : r.dy;
            r.dz = nb.dz < r.dz ? nb.dz : r.dz;
            r.bt = nb.bt < r.bt ? nb.bt : r.bt;
        }
    return r;
}

// Both sites of a BCC trial (active site of basis B at `ba`, its partner of
// the other basis at `bb`): packed neighbour counters, A[s] and Bc[s] get 1 <<
// (F * species) per neighbour of shell s.  The reads are rebased at the most
// negative offset (a window's neighbours lie within two conventional cells on
// every axis), so that with compile-time pitches every offset is a non-negative
// constant in the LDS instruction; they are software-pipelined in chunks of up to CHUNK neighbours of
// one (site, shell): the reads of chunk g + 1 are issued before chunk g's
// counter adds (scheduling barriers keep that order), so LDS latency
// overlaps the adds.  Row windows (compile-time pitches in the benchmark's
// preset) take chunks of 4: 954 us per 800^3 launch against 984 for whole
// (site, shell) groups, 965 for chunks of 8, 960 for chunks of 4 with two in
// flight, 972 with the order left to the compiler.  Tile windows keep whole
// groups: with chunks of 4 their runtime-pitch address arithmetic is cut
// into the same small pieces, and the batched tile sweeps of the ladder ran
// 11 % slower.
struct PairChunk {
    int site, shell, n0, n1;  // neighbours n0 .. n1 - 1 of shell `shell` of site 0 (active) or 1 (partner)
};
struct PairChunks {
    int n;
    PairChunk c[2 * kMaxShells * kMaxZ];
};
constexpr PairChunks make_pair_chunks(const Geometry& G, int S, int chunk)
{
    PairChunks P{};
    P.n = 0;
    for (int site = 0; site < 2; ++site)
        for (int s = 0; s < S; ++s)
            for (int n0 = 0; n0 < G.Z[s]; n0 += chunk) {
                PairChunk c{};
                c.site = site;
                c.shell = s;
                c.n0 = n0;
                c.n1 = n0 + chunk < G.Z[s] ? n0 + chunk : G.Z[s];
                P.c[P.n++] = c;
            }
    return P;
}

template <int LAT, int B, bool PLANAR, typename CT, int CHUNK>
__device__ __forceinline__ void count_pair(const uint8_t* win, int ba, int bb, int LP, int PL, int CP, int S,
                                           CT (&A)[kMaxShells], CT (&Bc)[kMaxShells])
{
    constexpr Geometry G = kGeom[LAT];
    constexpr int BB = 1 - B;
    const int XS = PLANAR ? 1 : G.m, BS = PLANAR ? CP : 1;
    constexpr Nb mna = min_components(G, B), mnb = min_components(G, BB);
    const int loa = mna.dz * PL + mna.dy * LP + XS * mna.dx + BS * (mna.bt - B);
    const int lob = mnb.dz * PL + mnb.dy * LP + XS * mnb.dx + BS * (mnb.bt - BB);
    int ra = ba + loa, rb = bb + lob;
    asm("" : "+v"(ra), "+v"(rb));
    const uint8_t* wa = win + ra;
    const uint8_t* wb = win + rb;
    // every chunk of the largest shell count; chunks of shells >= S are skipped
    constexpr PairChunks PC = make_pair_chunks(G, kMaxShells, CHUNK);
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s) {
        A[s] = 0;
        Bc[s] = 0;
    }
    uint32_t buf[2][CHUNK];
    auto load = [&](const int g, uint32_t(&v)[CHUNK]) {
        const PairChunk& c = PC.c[g];
        const int bs = c.site == 0 ? B : BB;
        if (c.shell < S) {
#pragma unroll
            for (int n = c.n0; n < c.n1; ++n) {
                const Nb nb = nb_of(G, bs, G.v[c.shell][n][0], G.v[c.shell][n][1], G.v[c.shell][n][2]);
                const int off = nb.dz * PL + nb.dy * LP + XS * nb.dx + BS * (nb.bt - bs);
                v[n - c.n0] = c.site == 0 ? wa[off - loa] : wb[off - lob];
            }
        }
    };
    auto add = [&](const int g, const uint32_t(&v)[CHUNK]) {
        const PairChunk& c = PC.c[g];
        if (c.shell < S) {
            CT acc = c.site == 0 ? A[c.shell] : Bc[c.shell];
            const int Z = c.n1 - c.n0, Z4 = Z & ~3;
#pragma unroll
            for (int n = 0; n < Z4; n += 4) acc = shl1_add4(v[n], v[n + 1], v[n + 2], v[n + 3], acc);
            if (Z - Z4 >= 2) {
                acc = shl1_add2(v[Z4], v[Z4 + 1], acc);
                if (Z - Z4 == 3) acc = shl1_add(v[Z4 + 2], acc);
            } else if (Z - Z4 == 1) {
                acc = shl1_add(v[Z4], acc);
            }
            if (c.site == 0) A[c.shell] = acc;
            else Bc[c.shell] = acc;
        }
    };
    load(0, buf[0]);
#pragma unroll
    for (int g = 0; g < PC.n; ++g) {
        if (g + 1 < PC.n) load(g + 1, buf[(g + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        add(g, buf[g & 1]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Packed neighbour counters of one FCC site, given the window byte `base[t]`
// that neighbour vectors of parity class t count from (a class is the basis
// they lead to from basis 0; each odd component carries into the next cell
// exactly when the site's own coordinate is odd, so a site of any basis needs
// one base per class and compile-time displacements from there).  A shell's
// vectors go by the window rows they lie in: one address per row, x in the
// reads' offset fields.  Bound by VALU issue and LDS reads; against a table of
// 16-bit offsets per (basis, partner, vector) in LDS, which cost an address
// read per neighbour: FCC 200^3 (5 species, 4 shells) 1694 -> 1265 us per
// sweep, 400^3 8089 -> 6950, 300x310x290 (4 species) 7234 -> 6415.
struct ShellRows {
    int n[kMaxZ];        // vectors of the shell in order of their rows
    bool first[kMaxZ];   // the first of its row
};
constexpr ShellRows make_shell_rows(const Geometry& G, int s)
{
    ShellRows R{};
    auto key = [&G, s](int i) {
        const Nb nb = nb_of(G, 0, G.v[s][i][0], G.v[s][i][1], G.v[s][i][2]);
        return (nb.bt * 8 + nb.dz + 4) * 8 + nb.dy + 4;
    };
    for (int i = 0; i < G.Z[s]; ++i) {
        int k = i;
        while (k > 0 && key(R.n[k - 1]) > key(i)) {
            R.n[k] = R.n[k - 1];
            --k;
        }
        R.n[k] = i;
    }
    for (int k = 0; k < G.Z[s]; ++k) R.first[k] = k == 0 || key(R.n[k - 1]) != key(R.n[k]);
    return R;
}

// Base per class of an FCC site of basis c at window byte `site`; X, LP, PL,
// BS: window steps of a cell along x, y and z and of a basis site.
__device__ __forceinline__ void class_bases(int site, int c, int X, int LP, int PL, int BS, int (&base)[4])
{
    // class 1 is odd in x and y, 2 in x and z, 3 in y and z
    const int fx = c == 1 || c == 2 ? X : 0, fy = c & 1 ? LP - 2 * BS : 0, fz = c & 2 ? PL - 4 * BS : 0;
    base[0] = site;
    base[1] = site + fx + fy;
    base[2] = site + fx + fz;
    base[3] = site + fy + fz;
}

template <bool PLANAR, typename CT>
__device__ __forceinline__ void count_classes(const uint8_t* win, const int (&base)[4], int LP, int PL, int BS, int S,
                                              CT (&A)[kMaxShells])
{
    constexpr Geometry G = kGeom[SMCX_FCC];
    constexpr int X = PLANAR ? 1 : G.m;
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s) {
        CT acc = 0;
        if (s < S) {
            constexpr ShellRows RW[kMaxShells] = {make_shell_rows(G, 0), make_shell_rows(G, 1), make_shell_rows(G, 2),
                                                  make_shell_rows(G, 3)};
            uint32_t v[kMaxZ];
            int row = 0;
#pragma unroll
            for (int k = 0; k < G.Z[s]; ++k) {
                const int* d = G.v[s][RW[s].n[k]];
                const Nb nb = nb_of(G, 0, d[0], d[1], d[2]);
                if (RW[s].first[k]) {
                    row = base[nb.bt] + (nb.dz * PL + nb.dy * LP + nb.bt * BS - 2 * X);
                    asm("" : "+v"(row));
                }
                v[k] = win[row + X * (nb.dx + 2)];
            }
            static_assert(G.Z[0] % 2 == 0 && G.Z[1] % 2 == 0 && G.Z[2] % 2 == 0 && G.Z[3] % 2 == 0, "pairs");
            const int Z4 = G.Z[s] & ~3;
#pragma unroll
            for (int n = 0; n < Z4; n += 4) acc = shl1_add4(v[n], v[n + 1], v[n + 2], v[n + 3], acc);
            if (G.Z[s] & 2) acc = shl1_add2(v[Z4], v[Z4 + 1], acc);
        }
        A[s] = acc;
    }
}

template <int PI>
struct GeoFix {
    static constexpr Preset P = kPresets[PI];
    static_assert(preset_ok(P), "tile start must be 16-byte aligned");
    static constexpr bool fixed = true;
    static constexpr bool rows = false;
    static constexpr bool own_cp = false;
    static constexpr bool may_alias = true;
    static constexpr int ELL = P.ell;
    static constexpr int kLP = preset_LP(P), kWY = preset_WY(P), kWZ = preset_WZ(P);
    static constexpr int kBLOCK = (P.tx * P.ty * P.tz + 63) / 64 * 64;
    __device__ static constexpr int T(const SweepArgs&, int a) { return a == 0 ? P.tx : (a == 1 ? P.ty : P.tz); }
    __device__ static constexpr int LP(const SweepArgs&) { return preset_LP(P); }
    __device__ static constexpr int WY(const SweepArgs&) { return preset_WY(P); }
    __device__ static constexpr int WZ(const SweepArgs&) { return preset_WZ(P); }
    __device__ static constexpr int block(const SweepArgs&) { return (P.tx * P.ty * P.tz + 63) / 64 * 64; }
    __device__ static constexpr int K(const SweepArgs&) { return P.K; }
    __device__ static constexpr int S(const SweepArgs&) { return P.S; }
    __device__ static int CP(const RepDev& rep) { return rep.cp; }  // tile windows are interleaved
};

// Row windows of a compile-time preset.
template <int PI>
struct GeoRowFix : GeoRt {
    static constexpr RowPreset P = kRowPresets[PI];
    static constexpr bool rows = true;
    static constexpr bool may_alias = false;  // chosen only for lattices without partner images
    __device__ static constexpr int T(const SweepArgs&, int a) { return a == 0 ? P.rt0 : (a == 1 ? P.rt1 : P.rt2); }
    __device__ static constexpr int LP(const SweepArgs&) { return P.LP; }
    __device__ static constexpr int WY(const SweepArgs&) { return P.WY; }
    __device__ static constexpr int WZ(const SweepArgs&) { return P.WZ; }
    __device__ static constexpr int K(const SweepArgs&) { return P.K; }
    __device__ static constexpr int S(const SweepArgs&) { return P.S; }
    __device__ static constexpr int CP(const RepDev&) { return P.cp; }
};

// Window of one tile for mini-step offsets o, identical in every thread.
// Returns false when no cell of the tile has these offsets.
template <int LAT, class Geo>
__device__ __forceinline__ bool tile_geometry(const SweepArgs& A, const RepDev& rep, int64_t tile,
                                              const int (&o)[3], TileGeom& tg)
{
    constexpr int m = kGeom[LAT].m;
    // tiles per replica stay below 2^31 (cells per replica do), so 32-bit division
    const int tl = (int)tile;
    const int tx = tl % rep.ntile[0];
    const int trest = tl / rep.ntile[0];
    const int ty = trest % rep.ntile[1];
    const int tz = trest / rep.ntile[1];
    tg.c0[0] = tx * Geo::T(A, 0);
    tg.c0[1] = ty * Geo::T(A, 1);
    tg.c0[2] = tz * Geo::T(A, 2);
    bool any = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        tg.c1[a] = min(tg.c0[a] + Geo::T(A, a), rep.nc[a]);
        tg.w0[a] = cell_origin<Geo>(A, rep, a, tg.c0[a]) + o[a] - kHalo;
        const int w1 = min(cell_origin<Geo>(A, rep, a, tg.c1[a] - 1) + o[a] + kHalo + 1, rep.L[a] + kHalo);
        tg.n[a] = w1 - tg.w0[a];
        any &= tg.n[a] > 0;
        if constexpr (!Geo::fixed) {
            // some cell of the tile must be longer than the offset (uneven partitions)
            bool has = false;
            for (int c = tg.c0[a]; c < tg.c1[a]; ++c)
                has |= cell_origin<Geo>(A, rep, a, c + 1) - cell_origin<Geo>(A, rep, a, c) > o[a];
            any &= has;
        }
    }
    tg.gx0 = (m * (tg.w0[0] + kHalo)) & ~15;
    return any;
}

// Per-thread staging plan of a compile-time window: thread t stages window
// slots t + i * BLOCK; soff[i] is the slot's byte offset from the window's
// first staged byte in the padded copy (plane and row pitches of a replica).
template <int LAT, class Geo>
struct StagePlan {
    static constexpr int LPc = Geo::kLP / 16;
    static constexpr int WY = Geo::kWY;
    static constexpr int WZ = Geo::kWZ;
    static constexpr int NSLOT = WZ * WY * LPc;
    static constexpr int BLOCK = Geo::kBLOCK;
    static constexpr int NP = (NSLOT + BLOCK - 1) / BLOCK;
    int soff[NP];
    int rep = -1;

    __device__ __forceinline__ void prepare(const RepDev& rp, int r)
    {
        if (r == rep) return;
        rep = r;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int slot = threadIdx.x + i * BLOCK;
            const int R = slot / LPc, col = slot - R * LPc;
            const int wz = R / WY, wy = R - wz * WY;
            soff[i] = (wz * rp.prows + wy) * rp.prow + 16 * col;
        }
    }

    // every slot of a full window lies inside the padded copy
    __device__ __forceinline__ void stage_full(const uint8_t* first, uint8_t* buf) const
    {
        const int wave64 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (i * BLOCK + wave64 < NSLOT && threadIdx.x + i * BLOCK < NSLOT)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(first + soff[i]),
                                                 (__attribute__((address_space(3))) void*)(buf + 16 * (i * BLOCK + wave64)),
                                                 16, 0, 0);
        }
    }
};

// A trial is split at the point where it stops reading the tile window:
// trial_read draws the random numbers and forms the packed neighbour counts
// from LDS, trial_finish turns them into dE, takes the Metropolis decision
// and writes the swap.  Between the two the window buffer may be refilled.
template <int E>
struct LaneState {
    using CT = typename Enc<E>::T;
    int active = 0;
    int p8 = 0, q8 = 0, k = 0, b = 0;
    CT Ca[kMaxShells], Cb[kMaxShells];
    uint32_t w1 = 0, w2 = 0;
    int ax = 0, ay = 0, az = 0;
    int la = 0, lb = 0;  // window bytes of the two sites
    int64_t ia = 0;
};

template <int LAT, int E, int B, class Geo>
__device__ __forceinline__ void trial_read(const SweepArgs& A, const RepDev& rep, const Lds& T, const uint8_t* win,
                                           const TileGeom& tg, int r, uint32_t t, int ax, int ay, int az,
                                           LaneState<E>& L, int64_t yz = 0)
{
    using CT = typename Enc<E>::T;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m;
    constexpr int Z1 = G.Z[0];
    const int LP = Geo::LP(A), WY = Geo::WY(A), PL = LP * WY;
    const int S = Geo::S(A);
    constexpr bool PLANAR = Geo::rows;
    const int la = ((az - tg.w0[2]) * WY + (ay - tg.w0[1])) * LP +
                   (PLANAR ? B * Geo::CP(rep) + ax + kHalo : m * (ax + kHalo) + B) - tg.gx0;
    // site index b + m (x + L0 (y + L1 z)); row kernels pass yz = m L0 (y + L1 z),
    // fixed for a row group, so a trial adds only b + m x
    int64_t ia;
    if constexpr (Geo::rows)
        ia = yz + (B + m * ax);
    else
        ia = B + (int64_t)m * (ax + (int64_t)rep.L[0] * (ay + (int64_t)rep.L[1] * az));
    uint32_t w0, w1, w2, w3;
    philox4x32_10((uint32_t)ia, (uint32_t)((uint64_t)ia >> 32), t, (uint32_t)r, (uint32_t)A.seed,
                  (uint32_t)(A.seed >> 32), w0, w1, w2, w3);
    (void)w3;
    const int k = (int)__umulhi(w0, (uint32_t)Z1);
    const int p8 = win[la];
    int offb, bt = 1 - B;  // the partner's window offset and basis
    if constexpr (Geo::own_cp || LAT == SMCX_FCC) {
        // from its cell displacement (row windows: and this replica's column
        // pitch, as replicas may differ in width)
        const int d = *(const int32_t*)(T.pd + (B * Z1 + k) * 4);
        bt = d >> 24;
        offb = (int)(int8_t)(d >> 16) * PL + (int)(int8_t)(d >> 8) * LP + (int)(int8_t)d * (PLANAR ? 1 : m) +
               (bt - B) * (PLANAR ? Geo::CP(rep) : 1);
    } else {
        offb = T.offB[B * Z1 + k];
    }
    const int q8 = win[la + offb];
    L.active = 1;
    L.p8 = p8;
    L.q8 = q8;
    L.k = k;
    L.b = B;
    L.w1 = w1;
    L.w2 = w2;
    L.ax = ax;
    L.ay = ay;
    L.az = az;
    L.ia = ia;
    L.la = la;
    L.lb = la + offb;
    if (p8 == q8) return;
    if constexpr (LAT == SMCX_BCC) {
        // the partner of a BCC site always sits on the other sublattice
        count_pair<LAT, B, PLANAR, CT, Geo::rows ? 4 : kMaxZ>(win, la, la + offb, LP, PL, Geo::CP(rep), S, L.Ca, L.Cb);
    } else {
        constexpr int X = PLANAR ? 1 : m;
        const int BS = PLANAR ? Geo::CP(rep) : 1;
        int base[4];
        class_bases(la, B, X, LP, PL, BS, base);
        count_classes<PLANAR, CT>(win, base, LP, PL, BS, S, L.Ca);
        class_bases(la + offb, bt, X, LP, PL, BS, base);
        count_classes<PLANAR, CT>(win, base, LP, PL, BS, S, L.Cb);
    }
}

// Returns flags: bit0 active, bit1 accepted, bit2 near-tie (0 for an idle lane).
template <int LAT, int E, class Geo>
__device__ __forceinline__ int trial_finish(const SweepArgs& A, const RepDev& rep, uint8_t* pad, const Lds& T,
                                            uint8_t* win, int r, uint32_t t, double beta, const LaneState<E>& L)
{
    using EN = Enc<E>;
    using CT = typename EN::T;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m;
    constexpr int Z1 = G.Z[0];
    if (!L.active) return 0;
    if (L.p8 == L.q8) return 1;
    const int K = Geo::K(A), S = Geo::S(A);
    const int p8 = L.p8, q8 = L.q8, k = L.k;
    // the per-shell count differences, fields biased by `half`
    CT dsh[kMaxShells];
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s) {
        // images of the partner inside shell s (1, 0, 0, 0 unless an edge is 2)
        const CT mu = Geo::may_alias && rep.alias ? (CT)rep.mult[s][k] : (CT)(s == 0 ? 1 : 0);
        dsh[s] = s < S ? L.Ca[s] + EN::bias - L.Cb[s] + (mu << p8) - (mu << q8) : (CT)0;
    }
    // Screen: dE in integers.  With every D[s][t][p][q] rounded to a multiple
    // of qscale, Qtab holds each shell's D_t - D_last (24-bit signed; a shell's
    // count differences c_t sum to zero, so the last species needs no term), so
    // sum_t (c_t + half) Q - bias, bias = half sum Q, is sum_t c_t D_t of the
    // rounded D exactly (modulo 2^32, and it fits in 32 bits), within qeps /
    // qscale units of the binary64 dE.  It settles the decision whenever that
    // uncertainty cannot change it; otherwise the binary64 sum and test below
    // decide, as they always would.
    // Every table read is issued before the first product, so the trial waits
    // for the LDS once; a pair's terms lie side by side at fixed offsets.
    // Against tables [s][t][p][q] with one term more per shell and, but for
    // two alloys, shell counts known only at run time, us per sweep: FCC 200^3 of
    // 6 species 1930 -> 925 (2 shells; 64-bit counters before), 250x200x220 of
    // 3 species and 3 shells 2175 -> 1490, BCC 250x260x270 of 3 species and 3
    // shells 1397 -> 920, of 4 species and 4 shells 1172 -> 1030.
    constexpr int KT = EN::KT;
    const int pair = species_pair<E>(p8, q8, K);
    const int32_t* Qp = qtab_row<E>(T.Q, pair, S);
    int32_t qv[kMaxShells][KT];
    const int32_t qbias = Qp[S * KT];
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s)
#pragma unroll
        for (int tt = 0; tt < KT; ++tt) qv[s][tt] = s < S ? Qp[s * KT + tt] : 0;
    __builtin_amdgcn_sched_barrier(0);
    uint32_t qacc = 0u - (uint32_t)qbias;
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s) {
        if (s < S) {
#pragma unroll
            for (int tt = 0; tt < KT; ++tt)
                qacc += (uint32_t)__mul24((int)((dsh[s] >> (EN::F * tt)) & EN::mask), qv[s][tt]);
        }
    }
    static_assert(kMaxShells == 4, "four shell counters");
    const int f = metropolis<E>(qacc, T.qscale, T.qeps, A.Dtab, pair, dsh[0], dsh[1], dsh[2], dsh[3], K, S, beta,
                                L.w1, L.w2);
    const bool acc = (f & 1) != 0, tie = (f & 2) != 0;
    if (tie) log_tie(A, r, t, L.ia, acc);
    if (acc) {
        const int8_t* pd = T.pd + (L.b * Z1 + k) * 4;
        int bx = L.ax + pd[0], by = L.ay + pd[1], bz = L.az + pd[2];
        const int bb = pd[3];
        const int ubx = bx;  // partner x before the periodic wrap (its column in a row window)
        bx += bx < 0 ? rep.L[0] : (bx >= rep.L[0] ? -rep.L[0] : 0);
        by += by < 0 ? rep.L[1] : (by >= rep.L[1] ? -rep.L[1] : 0);
        bz += bz < 0 ? rep.L[2] : (bz >= rep.L[2] ? -rep.L[2] : 0);
        // the padded copy holds F * species, like the window; the window copy
        // serves the next basis site's trial of this lane
        // (row windows reach HBM in one copy of their changed rows per group)
        if constexpr (!Geo::rows) {
            store_site<false>(pad, rep, m, L.ax, L.ay, L.az, L.b, (uint8_t)q8);
            store_site<false>(pad, rep, m, bx, by, bz, bb, (uint8_t)p8);
        }
        win[L.la] = (uint8_t)q8;
        win[L.lb] = (uint8_t)p8;
        if constexpr (Geo::rows) {
            // row windows span x in [-H, L + H): sites within H of an x face appear twice
            const int Lx = rep.L[0], sh = Lx;  // basis-planar rows: x step 1
            if (L.ax < kHalo) win[L.la + sh] = (uint8_t)q8;
            if (L.ax >= Lx - kHalo) win[L.la - sh] = (uint8_t)q8;
            if (ubx < kHalo) win[L.lb + sh] = (uint8_t)p8;
            if (ubx >= Lx - kHalo) win[L.lb - sh] = (uint8_t)p8;
        }
    }
    return 1 | (acc ? 2 : 0) | (tie ? 4 : 0);
}

template <int LAT, int E, class Geo>
__device__ __forceinline__ void read_dispatch(int b, const SweepArgs& A, const RepDev& rep, const Lds& T,
                                              const uint8_t* win, const TileGeom& tg, int r, uint32_t t, int ax,
                                              int ay, int az, LaneState<E>& L)
{
    if constexpr (LAT == SMCX_BCC) {
        if (b == 0) trial_read<LAT, E, 0, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L);
        else trial_read<LAT, E, 1, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L);
    } else {
        switch (b) {
        case 0: trial_read<LAT, E, 0, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L); break;
        case 1: trial_read<LAT, E, 1, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L); break;
        case 2: trial_read<LAT, E, 2, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L); break;
        default: trial_read<LAT, E, 3, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L); break;
        }
    }
}

// First half of the trials of one staged tile (one lane per link cell):
// lanes outside the tile or whose cell is shorter than an offset stay idle.
template <int LAT, int E, class Geo>
__device__ __forceinline__ void tile_read(const SweepArgs& A, const RepDev& rep, int r, const TileGeom& tg, int b,
                                          const int (&o)[3], uint32_t t, const Lds& T, const uint8_t* win,
                                          LaneState<E>& L)
{
    L.active = 0;
    const int l = threadIdx.x;
    const int lx = l % Geo::T(A, 0);
    const int ly = (l / Geo::T(A, 0)) % Geo::T(A, 1);
    const int lz = l / (Geo::T(A, 0) * Geo::T(A, 1));
    const int cx = tg.c0[0] + lx, cy = tg.c0[1] + ly, cz = tg.c0[2] + lz;
    if (!(lz < Geo::T(A, 2) && cx < tg.c1[0] && cy < tg.c1[1] && cz < tg.c1[2])) return;
    const int ax = cell_origin<Geo>(A, rep, 0, cx) + o[0];
    const int ay = cell_origin<Geo>(A, rep, 1, cy) + o[1];
    const int az = cell_origin<Geo>(A, rep, 2, cz) + o[2];
    if constexpr (!Geo::fixed) {
        if (!(ax < cell_origin<Geo>(A, rep, 0, cx + 1) && ay < cell_origin<Geo>(A, rep, 1, cy + 1) &&
              az < cell_origin<Geo>(A, rep, 2, cz + 1)))
            return;
    }
    read_dispatch<LAT, E, Geo>(b, A, rep, T, win, tg, r, t, ax, ay, az, L);
}

template <int LAT, int E, class Geo>
__device__ __forceinline__ void tile_finish(const SweepArgs& A, const RepDev& rep, int r, uint32_t t, double beta,
                                            const Lds& T, uint8_t* win, const LaneState<E>& L, Stats& st)
{
    const int f = trial_finish<LAT, E, Geo>(A, rep, A.ws + rep.pad_off, T, win, r, t, beta, L);
    st.att += f & 1;
    st.acc += (f >> 1) & 1;
    st.tie += (f >> 2) & 1;
}

// Trials of basis sites b0 .. b0 + nb - 1 at the same offsets o, each lane in
// its own link cell.  One window serves them all: a lane's trial at b + 1
// reads within two conventional cells of its site, which no other cell's
// trial at b writes (the sites of two cells stay at least three cells apart
// on some axis), so the lane's own accepted swap, written back into the
// window, is the only change it can see.  (Needs every edge >= 4, so that no
// periodic image of a written site lies in that reach.)
template <int LAT, int E, class Geo>
__device__ __forceinline__ void tile_trials(const SweepArgs& A, const RepDev& rep, int r, const TileGeom& tg,
                                            int b0, int nb, const int (&o)[3], uint32_t t, double beta,
                                            const Lds& T, uint8_t* win, Stats& st)
{
    for (int j = 0; j < nb; ++j) {
        LaneState<E> L;
        tile_read<LAT, E, Geo>(A, rep, r, tg, b0 + j, o, t, T, win, L);
        tile_finish<LAT, E, Geo>(A, rep, r, t, beta, T, win, L, st);
    }
}

// Tiles first, first + step, ... (< end) of a logical tile space for mini-step
// tau of sweep t.  With two window buffers the next tile's window streams into
// LDS while the current tile's trials run; with one, each window is staged in
// turn (half the LDS, so more workgroups per CU hide the latency instead).
// tile_of(i, r, tile) maps a logical index to (replica, tile of that replica);
// beta_of(r) gives the replica's inverse temperature.  Every thread calls this
// with the same arguments.
template <int LAT, int E, class Geo, int NBUF, typename TileOf, typename BetaOf>
__device__ void run_tiles(const SweepArgs& A, int64_t first, int64_t end, int64_t step, int tau, int nb, uint32_t t,
                          const Lds& T, uint8_t* win0, uint8_t* win1, TileOf tile_of, BetaOf beta_of, Stats& st,
                          int& r_stats)
{
    constexpr int m = kGeom[LAT].m;
    if (first >= end) return;
    auto offsets = [&](const RepDev& rep, int (&o)[3], int& b) {
        b = tau % m;
        const int rest = tau / m;
        o[0] = rest % rep.M[0];
        o[1] = (rest / rep.M[0]) % rep.M[1];
        o[2] = rest / (rep.M[0] * rep.M[1]);
    };
    if constexpr (NBUF == 1) {
        struct NoPlan {};
        [[maybe_unused]] std::conditional_t<Geo::fixed, StagePlan<LAT, Geo>, NoPlan> plan;
        for (int64_t i = first; i < end; i += step) {
            int r;
            int64_t tile;
            tile_of(i, r, tile);
            uniform(r, tile);
            const RepDev& rep = rep_of(A, r);
            if (tau >= rep.nA) continue;  // uniform across the block
            int o[3], b;
            offsets(rep, o, b);
            TileGeom tg;
            if (!tile_geometry<LAT, Geo>(A, rep, tile, o, tg)) continue;
            lds_barrier();  // every lane is done with the window of the previous tile
            const uint8_t* pad = A.ws + rep.pad_off;
            if constexpr (Geo::fixed) {
                constexpr int m = kGeom[LAT].m;
                using SP = decltype(plan);
                const int gx1 = (m * (tg.w0[0] + tg.n[0] + kHalo) + 15) & ~15;
                if (((gx1 - tg.gx0) >> 4) == SP::LPc && tg.n[1] == SP::WY && tg.n[2] == SP::WZ) {
                    plan.prepare(rep, r);
                    plan.stage_full(pad + ((int64_t)(tg.w0[2] + kHalo) * rep.prows + (tg.w0[1] + kHalo)) * rep.prow +
                                        tg.gx0,
                                    win0);
                } else {
                    stage_async<LAT, Geo>(A, rep, tg, pad, win0);
                }
            } else {
                stage_async<LAT, Geo>(A, rep, tg, pad, win0);
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (r != r_stats) {
                flush_stats(A, r_stats, st);
                r_stats = r;
            }
            tile_trials<LAT, E, Geo>(A, rep, r, tg, b, nb, o, t, beta_of(r), T, win0, st);
        }
        return;
    }
    int r = 0, rn = 0;
    int64_t tile = 0, tilen = 0;
    tile_of(first, r, tile);
    uniform(r, tile);
    int o[3], b;
    TileGeom tg;
    bool have;
    constexpr bool dbl = true;
    {
        const RepDev& rep = rep_of(A, r);
        offsets(rep, o, b);
        have = tau < rep.nA && tile_geometry<LAT, Geo>(A, rep, tile, o, tg);
        if (have && dbl) stage_async<LAT, Geo>(A, rep, tg, A.ws + rep.pad_off, win0);
    }
    int k = 0;
    for (int64_t i = first; i < end; i += step, ++k) {
        const int64_t inext = i + step;
        int on[3] = {0, 0, 0}, bn = 0;
        TileGeom tgn;
        bool haven = false;
        if (inext < end) {
            tile_of(inext, rn, tilen);
            uniform(rn, tilen);
            const RepDev& repn = rep_of(A, rn);
            offsets(repn, on, bn);
            haven = tau < repn.nA && tile_geometry<LAT, Geo>(A, repn, tilen, on, tgn);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();  // double buffering: window of tile i landed; both: lanes done with the buffer
        uint8_t* cur = win0;
        if (dbl) {
            cur = (k & 1) ? win1 : win0;
            if (haven) stage_async<LAT, Geo>(A, rep_of(A, rn), tgn, A.ws + rep_of(A, rn).pad_off, (k & 1) ? win0 : win1);
        } else if (have) {
            stage_async<LAT, Geo>(A, rep_of(A, r), tg, A.ws + rep_of(A, r).pad_off, win0);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        if (have) {
            if (r != r_stats) {
                flush_stats(A, r_stats, st);
                r_stats = r;
            }
            tile_trials<LAT, E, Geo>(A, rep_of(A, r), r, tg, b, nb, o, t, beta_of(r), T, cur, st);
        }
        r = rn;
        tile = tilen;
        tg = tgn;
        have = haven;
        o[0] = on[0];
        o[1] = on[1];
        o[2] = on[2];
        b = bn;
    }
}

// ---------------------------------------------------------------------------
// Stream mode: one launch per mini-step g.  The logical tiles of all replicas
// (or of one replica in plain mode) are split into 8 contiguous chunks, one
// per XCD (hardware workgroup i runs on XCD i % 8); the workgroups of an XCD
// walk their chunk together with stride W, so neighbouring tiles -- which
// share halo rows -- are in flight on the same L2 at the same time.
// ---------------------------------------------------------------------------
template <int LAT, int E, class Geo, int NBUF>
__global__ __launch_bounds__(kBlock) void k_ministep(SweepArgs A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    load_tables<LAT>(A, smem);
    const Lds T = lds_ptrs(A, smem);
    const int64_t total = A.only_rep >= 0 ? A.reps[A.only_rep].ntiles : A.tile_off[A.R];
    const int xcd = blockIdx.x % 8;
    const int64_t W = gridDim.x / 8;
    const int64_t chunk = (total + 7) / 8;
    const int64_t lo = xcd * chunk;
    const int64_t hi = min(lo + chunk, total);
    auto tile_of = [&](int64_t i, int& r, int64_t& tile) {
        if (A.only_rep >= 0) {
            r = A.only_rep;
            tile = i;
            return;
        }
        int a = 0, z = A.R - 1;  // last replica with tile_off[r] <= i
        while (a < z) {
            const int mid = (a + z + 1) >> 1;
            if (ld_const(A.tile_off, mid) <= i) a = mid; else z = mid - 1;
        }
        r = a;
        tile = i - ld_const(A.tile_off, a);
    };
    auto beta_of = [&](int r) { return ld_const(A.beta, r); };
    Stats st;
    int r_stats = -1;
    // a captured sweep reads its sweep index from the device counter
    const uint32_t t = A.sweep_counter ? *A.sweep_counter + A.first_sweep : A.first_sweep;
    run_tiles<LAT, E, Geo, NBUF>(A, lo + blockIdx.x / 8, hi, W, A.g, A.nb, t, T, smem + A.lds_win,
                           smem + A.lds_win + A.win_bytes, tile_of, beta_of, st, r_stats);
    flush_stats(A, r_stats, st);
}

// ---------------------------------------------------------------------------
// Row mode: one launch per group of mini-steps sharing the offsets (o_y, o_z)
// -- every o_x and basis site, M_x * m mini-steps.  A workgroup owns whole
// x-rows of link cells (T[1] x T[2] rows of every cell along x) and stages
// their window once: full padded x-rows, y and z within two cells of the
// active rows.  Within the group a trial depends only on trials of the same
// row (cells in other rows stay beyond the reach on y or z, since o_y and o_z
// are fixed), and there only on earlier offsets o_x; a workgroup barrier after
// each o_x orders them.  Accepted swaps go to HBM, to the window and to the
// window's x-images, so every later trial of the group reads them from LDS.
// A launch covers mini-steps g .. g + nb - 1 of one group.  MAXB: the largest
// workgroup the instantiation serves (1024 caps registers at 4 waves/SIMD).
// ---------------------------------------------------------------------------
// Trials of basis sites b0 .. b1 - 1 at one site of a lane's link cell, one
// code path per basis site (no merge of the sites' lane states).
template <int LAT, int E, class Geo, int B>
__device__ __forceinline__ void row_trials(int b0, int b1, const SweepArgs& A, const RepDev& rep, const Lds& T,
                                           uint8_t* win, const TileGeom& tg, int r, uint32_t t, double beta, int ax,
                                           int ay, int az, int64_t yz, Stats& st)
{
    if constexpr (B < kGeom[LAT].m) {
        if (B >= b0 && B < b1) {
            LaneState<E> L;
            trial_read<LAT, E, B, Geo>(A, rep, T, win, tg, r, t, ax, ay, az, L, yz);
            tile_finish<LAT, E, Geo>(A, rep, r, t, beta, T, win, L, st);
        }
        row_trials<LAT, E, Geo, B + 1>(b0, b1, A, rep, T, win, tg, r, t, beta, ax, ay, az, yz, st);
    }
}

template <int LAT, int E, class Geo, int MAXB>
__global__ __launch_bounds__(MAXB) void k_rows(SweepArgs A)
{
    constexpr int m = kGeom[LAT].m;
    extern __shared__ __align__(16) uint8_t smem[];
    load_tables<LAT>(A, smem);
    const Lds T = lds_ptrs(A, smem);
    uint8_t* win = smem + A.lds_win;
    const int64_t total = ld_const(A.tile_off, A.R);  // row groups of all replicas
    const int xcd = blockIdx.x % 8;
    const int64_t W = gridDim.x / 8;
    const int64_t chunk = (total + 7) / 8;
    const int64_t lo = xcd * chunk;
    const int64_t hi = min(lo + chunk, total);
    const int l = threadIdx.x;
    const int T0 = Geo::T(A, 0), T1 = Geo::T(A, 1), T2 = Geo::T(A, 2);
    const int lx = l % T0, ly = (l / T0) % T1, lz = l / (T0 * T1);
    const uint32_t t = A.sweep_counter ? *A.sweep_counter + A.first_sweep : A.first_sweep;
    Stats st;
    int r_stats = -1;
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
        int g0 = A.g, gn = A.nb;
        if (A.gq >= 0) {
            // this replica's q-th (o_y, o_z) group, every offset o_x and basis site
            if (A.gq >= rep.M[1] * rep.M[2]) continue;
            gn = m * rep.M[0];
            g0 = A.gq * gn;
        }
        if (g0 >= rep.nA) continue;
        const int b0 = g0 % m, rest = g0 / m;
        const int ox0 = rest % rep.M[0];
        const int oy = (rest / rep.M[0]) % rep.M[1], oz = rest / (rep.M[0] * rep.M[1]);
        const int gy = (int)(grp % rep.rg[0]), gz = (int)(grp / rep.rg[0]);
        TileGeom tg;
        tg.c0[0] = 0;
        tg.c1[0] = rep.nc[0];
        tg.c0[1] = gy * T1;
        tg.c1[1] = min(tg.c0[1] + T1, rep.nc[1]);
        tg.c0[2] = gz * T2;
        tg.c1[2] = min(tg.c0[2] + T2, rep.nc[2]);
        if (oy >= rep.emin[1] || oz >= rep.emin[2]) {
            // uneven partitions: offsets past the shorter cells leave some row
            // groups without an active cell row; skip them before staging
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
        // this lane's cell while the loads fly
        const int cx = lx, cy = tg.c0[1] + ly, cz = tg.c0[2] + lz;
        const bool row_in = lz < T2 && cy < tg.c1[1] && cz < tg.c1[2];
        const bool in = row_in && cx < tg.c1[0];
        int x0 = 0, ex = 0, y0 = 0, ey = 0, z0 = 0, ez = 0;
        if (row_in) {
            y0 = cell_origin<Geo>(A, rep, 1, cy);
            ey = cell_origin<Geo>(A, rep, 1, cy + 1) - y0;
            z0 = cell_origin<Geo>(A, rep, 2, cz);
            ez = cell_origin<Geo>(A, rep, 2, cz + 1) - z0;
        }
        if (in) {
            x0 = cell_origin<Geo>(A, rep, 0, cx);
            ex = cell_origin<Geo>(A, rep, 0, cx + 1) - x0;
        }
        // the cell row has active sites at (o_y, o_z)
        const bool row_yz = row_in && oy < ey && oz < ez;
        const bool yz = in && row_yz;
        const double beta = ld_const(A.beta, r);
        const int64_t yz_site = (int64_t)m * rep.L[0] * ((int64_t)(y0 + oy) + (int64_t)rep.L[1] * (z0 + oz));
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (r != r_stats) {
            flush_stats_block(A, r_stats, st);
            r_stats = r;
        }
        int tau = g0, b = b0, ox = ox0;
        const int tau1 = g0 + gn;
        while (true) {
            const int nbb = min(m - b, tau1 - tau);
            if (yz && ox < ex)
                row_trials<LAT, E, Geo, 0>(b, b + nbb, A, rep, T, win, tg, r, t, beta, x0 + ox, y0 + oy, z0 + oz, yz_site, st);
            tau += nbb;
            if (tau >= tau1) break;
            b = 0;
            ++ox;
            __syncthreads();  // the next offset's trials read what this one wrote
        }
        __syncthreads();  // every trial's window writes are visible
        if (row_yz) rows_writeback<LAT, Geo>(A, rep, tg, lx, T0, y0 + oy, z0 + oz, A.ws + rep.pad_off, win);
    }
    flush_stats_block(A, r_stats, st);
}

// ---------------------------------------------------------------------------
// Persistent mode: one workgroup per replica runs every sweep and mini-step;
// block barriers order the mini-steps (all writes of a replica come from its
// own workgroup, and a barrier makes them visible to its later loads).
// ---------------------------------------------------------------------------
template <int LAT, int E, class Geo>
__global__ __launch_bounds__(kBlock) void k_persistent(SweepArgs A)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int r = blockIdx.x;
    const RepDev& rep = rep_of(A, r);
    load_tables<LAT>(A, smem);
    const Lds T = lds_ptrs(A, smem);
    const uint32_t first = A.sweep_counter ? *A.sweep_counter : A.first_sweep;
    auto tile_of = [&](int64_t i, int& rr, int64_t& tile) {
        rr = r;
        tile = i;
    };
    Stats st;
    int r_stats = r;
    const int tau_end = min(A.tau_end, rep.nA);
    for (int js = 0; js < A.n_sweeps; ++js) {
        const uint32_t t = first + (uint32_t)js;
        const double beta = ld_const(A.beta, (int64_t)js * A.beta_stride + r);
        auto beta_of = [&](int) { return beta; };
        for (int tau = A.tau_begin; tau < tau_end;) {
            // mini-steps of consecutive basis sites at one offset share a window
            const int nb = min(A.nb - tau % A.nb, tau_end - tau);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();  // the previous mini-step's writes are visible to every wave
            run_tiles<LAT, E, Geo, 1>(A, 0, rep.ntiles, 1, tau, nb, t, T, smem + A.lds_win,
                                   smem + A.lds_win + A.win_bytes, tile_of, beta_of, st, r_stats);
            tau += nb;
        }
        // the 32-bit sums of a wave go out before 2^30 trials of the workgroup (a
        // sweep tries every site once)
        if ((js & 63) == 63 || rep.N > 1 << 24 || js + 1 == A.n_sweeps) flush_stats(A, r, st);
    }
}

__global__ void k_advance_counter(uint32_t* counter, uint32_t n)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *counter += n;
}

// Natural layout <-> padded copy.
//
// Basis-planar rows: a thread takes 16 padded bytes of every basis column of a
// row, cells x0 = 16 j - H .. x0 + 15, which lie next to each other in the
// natural row (16 M bytes, at any alignment): M wide loads, a byte transpose
// in registers, M wide stores, the other way round to unpack.  Chunks that
// reach past a face go byte by byte.  Bound by memory: BCC 800^3 packs in
// 641 us and unpacks in 454 us (2.1 GB each); word loads at a
// 32-byte stride, a fifth of whose lines are used at a time, took 1110 and
// 780 us.
constexpr int kPackCells = 16;

// d[4 i .. 4 i + 3], i < M: 16 cells of M bytes; c[b][0 .. 3]: 16 bytes of column b.
template <int M>
__device__ __forceinline__ void to_columns(const uint32_t (&d)[4 * M], uint32_t (&c)[M][4])
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (M == 2) {
            c[0][w] = __builtin_amdgcn_perm(d[2 * w + 1], d[2 * w], 0x06040200u);
            c[1][w] = __builtin_amdgcn_perm(d[2 * w + 1], d[2 * w], 0x07050301u);
        } else {
            const uint32_t *q = d + 4 * w;  // four cells
            const uint32_t t0 = __builtin_amdgcn_perm(q[1], q[0], 0x05010400u), t1 = __builtin_amdgcn_perm(q[3], q[2], 0x05010400u);
            const uint32_t t2 = __builtin_amdgcn_perm(q[1], q[0], 0x07030602u), t3 = __builtin_amdgcn_perm(q[3], q[2], 0x07030602u);
            c[0][w] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
            c[1][w] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
            c[2][w] = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
            c[3][w] = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
        }
    }
}
template <int M>
__device__ __forceinline__ void to_cells(const uint32_t (&c)[M][4], uint32_t (&d)[4 * M])
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (M == 2) {
            d[2 * w] = __builtin_amdgcn_perm(c[1][w], c[0][w], 0x05010400u);
            d[2 * w + 1] = __builtin_amdgcn_perm(c[1][w], c[0][w], 0x07030602u);
        } else {
            const uint32_t t0 = __builtin_amdgcn_perm(c[1][w], c[0][w], 0x05010400u), t1 = __builtin_amdgcn_perm(c[3][w], c[2][w], 0x05010400u);
            const uint32_t t2 = __builtin_amdgcn_perm(c[1][w], c[0][w], 0x07030602u), t3 = __builtin_amdgcn_perm(c[3][w], c[2][w], 0x07030602u);
            d[4 * w] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
            d[4 * w + 1] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
            d[4 * w + 2] = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
            d[4 * w + 3] = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
        }
    }
}

template <int M, bool PLANAR>
__global__ __launch_bounds__(kBlock) void k_pack(const uint8_t* occ, uint8_t* ws, const RepDev* reps, int r, int F)
{
    const RepDev& rep = rep_at(reps, r < 0 ? (int)blockIdx.y : r);  // r < 0: one replica per grid row
    uint8_t* pad = ws + rep.pad_off;
    const uint8_t* o = occ + rep.occ_off;
    const int L0 = rep.L[0], L1 = rep.L[1], L2 = rep.L[2];
    const int nrow = rep.prows * (L2 + 2 * kHalo);
    // padded row -> the natural row at its wrapped y, z
    auto source = [&](int row) {
        const int zp = row / rep.prows, yp = row - zp * rep.prows;
        int y = yp - kHalo, z = zp - kHalo;
        y += y < 0 ? L1 : (y >= L1 ? -L1 : 0);
        z += z < 0 ? L2 : (z >= L2 ? -L2 : 0);
        return o + (int64_t)M * L0 * (y + (int64_t)L1 * z);
    };
    if constexpr (PLANAR) {
        const int nblk = rep.cp >> 4;
        const int64_t total = (int64_t)nrow * nblk;
        for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
            const int row = total < (1ll << 31) ? (int)((uint32_t)i / (uint32_t)nblk) : (int)(i / nblk);
            const int j = (int)(i - (int64_t)row * nblk), x0 = kPackCells * j - kHalo;
            const uint8_t* src = source(row);
            uint32_t d[4 * M], c[M][4];
            if (x0 >= 0 && x0 + kPackCells <= L0) {
                __builtin_memcpy(d, src + M * x0, 16 * M);
                to_columns<M>(d, c);
            } else {
#pragma unroll
                for (int b = 0; b < M; ++b)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        c[b][w] = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            int x = x0 + 4 * w + k;  // bytes past the halo stay 0
                            if (x < L0 + kHalo) {
                                x += x < 0 ? L0 : (x >= L0 ? -L0 : 0);
                                c[b][w] |= (uint32_t)src[M * x + b] << (8 * k);
                            }
                        }
                    }
            }
            uint8_t* dst = pad + (int64_t)row * rep.prowp + 16 * j;
#pragma unroll
            for (int b = 0; b < M; ++b) {
                uint4 v;  // F * species < 256: no carry crosses a byte
                v.x = c[b][0] * (uint32_t)F;
                v.y = c[b][1] * (uint32_t)F;
                v.z = c[b][2] * (uint32_t)F;
                v.w = c[b][3] * (uint32_t)F;
                *(uint4*)(dst + b * rep.cp) = v;
            }
        }
    } else {
        // interleaved rows: a workgroup per row, a thread one word of it at a
        // time; bytes past the row's M (L0 + 2H) sites stay 0
        const int words = rep.prow >> 2;
        for (int row = blockIdx.x; row < nrow; row += gridDim.x) {
            const uint8_t* src = source(row);
            uint32_t* dst = (uint32_t*)(pad + (int64_t)row * rep.prow);
            for (int w = threadIdx.x; w < words; w += blockDim.x) {
                uint32_t v = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = 4 * w + i, b = j % M;
                    int x = j / M - kHalo;
                    if (x < L0 + kHalo) {
                        x += x < 0 ? L0 : (x >= L0 ? -L0 : 0);
                        v |= (uint32_t)(src[M * x + b] * F) << (8 * i);
                    }
                }
                dst[w] = v;
            }
        }
    }
}

// Four species from their stored form F * species: v / 6 = ((v / 2) 11) / 32
// for v in 0, 6, .. 30, and no product leaves its byte.
__device__ __forceinline__ uint32_t species_of4(uint32_t v, int F)
{
    return F == 8 ? (v >> 3) & 0x1F1F1F1Fu : ((((v >> 1) & 0x0F0F0F0Fu) * 11u) >> 5) & 0x07070707u;
}

template <int M, bool PLANAR>
__global__ __launch_bounds__(kBlock) void k_unpack(uint8_t* occ, const uint8_t* ws, const RepDev* reps, int r, int F,
                                                   int64_t* slots, int parts, int64_t* stats)
{
    const int ri = r < 0 ? (int)blockIdx.y : r;  // r < 0: one replica per grid row
    if (parts > 0 && blockIdx.x == 0 && threadIdx.x < 64) {
        // the sweep launches' counter slots (at most 64), added up and cleared
        for (int k = 0; k < 3; ++k) {
            int64_t* s = slots + ((int64_t)ri * parts + threadIdx.x) * kStatStride + k;
            int64_t v = 0;
            if ((int)threadIdx.x < parts) {
                v = *s;
                *s = 0;
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
            // atomic: handles on other streams may count into the same words
            if (threadIdx.x == 0 && v) atomicAdd((unsigned long long*)&stats[3 * (int64_t)ri + k], (unsigned long long)v);
        }
    }
    const RepDev& rep = rep_at(reps, ri);
    const uint8_t* pad = ws + rep.pad_off;
    uint8_t* o = occ + rep.occ_off;
    const int L0 = rep.L[0], L1 = rep.L[1], L2 = rep.L[2];
    if constexpr (PLANAR) {
        const int nblk = (L0 + kHalo + kPackCells - 1) / kPackCells;  // chunks with an interior cell
        const int64_t total = (int64_t)L1 * L2 * nblk;
        for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
            const int row = total < (1ll << 31) ? (int)((uint32_t)i / (uint32_t)nblk) : (int)(i / nblk);
            const int j = (int)(i - (int64_t)row * nblk), x0 = kPackCells * j - kHalo;
            const int z = row / L1, y = row - z * L1;
            const uint8_t* src = pad + ((int64_t)(z + kHalo) * rep.prows + (y + kHalo)) * rep.prowp + 16 * j;
            uint8_t* dst = o + (int64_t)M * ((int64_t)L0 * row + x0);
            uint32_t c[M][4], d[4 * M];
#pragma unroll
            for (int b = 0; b < M; ++b) {
                const uint4 v = *(const uint4*)(src + b * rep.cp);
                c[b][0] = species_of4(v.x, F);
                c[b][1] = species_of4(v.y, F);
                c[b][2] = species_of4(v.z, F);
                c[b][3] = species_of4(v.w, F);
            }
            to_cells<M>(c, d);
            if (x0 >= 0 && x0 + kPackCells <= L0) {
                __builtin_memcpy(dst, d, 16 * M);
            } else {
#pragma unroll
                for (int k = 0; k < kPackCells * M; ++k)
                    if (x0 + k / M >= 0 && x0 + k / M < L0) dst[k] = (uint8_t)(d[k >> 2] >> (8 * (k & 3)));
            }
        }
    } else {
        // interleaved rows: a workgroup per natural row, a thread per site byte
        const int n = M * L0;
        for (int row = blockIdx.x; row < L1 * L2; row += gridDim.x) {
            const int z = row / L1, y = row - z * L1;
            const uint8_t* src = pad + ((int64_t)(z + kHalo) * rep.prows + (y + kHalo)) * rep.prow;
            uint8_t* dst = o + (int64_t)n * row;
            for (int j = threadIdx.x; j < n; j += blockDim.x) dst[j] = (uint8_t)species_of(src[M * kHalo + j], F);
        }
    }
}

// Species check of n sites: 16 at a time between the first and the last byte
// of an aligned 16.  Bound by HBM: an init of BCC 800^3 (1.02 GB) takes 280 us,
// 1100 byte by byte.
__global__ void k_validate(const uint8_t* occ, int64_t n, int K, int32_t* bad)
{
    const int64_t head = min((int64_t)(-(uintptr_t)occ & 15), n), n16 = (n - head) >> 4, tail = head + 16 * n16;
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    const uint32_t addK = (uint32_t)(128 - K) * 0x01010101u;
    uint32_t over = 0;
    const uint4* v = (const uint4*)(occ + head);
    for (int64_t i = i0; i < n16; i += step) {
        const uint4 d = v[i];
        over |= (((d.x & 0x7f7f7f7fu) + addK) | d.x) | (((d.y & 0x7f7f7f7fu) + addK) | d.y) |
                (((d.z & 0x7f7f7f7fu) + addK) | d.z) | (((d.w & 0x7f7f7f7fu) + addK) | d.w);
    }
    int found = (over & 0x80808080u) != 0;
    if (i0 < 16) {
        if (i0 < head) found |= occ[i0] >= K;
        if (tail + i0 < n) found |= occ[tail + i0] >= K;
    }
    if (__ballot(found) && (threadIdx.x & 63) == 0) atomicOr(bad, 1);
}

__global__ void k_fill_i64(int64_t* p, int64_t n, int64_t v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Kernel resolution: (lattice, counter encoding, window preset) -> kernels.
// Stream kernels exist for the runtime geometry and every preset of the
// lattice; persistent kernels use the runtime geometry only.
// ---------------------------------------------------------------------------
// f with the counter encoding of K species as an integral constant
template <typename F>
static const void* with_encoding(int K, F f)
{
    if (K <= 4) return f(std::integral_constant<int, 1>{});
    if (K == 5) return f(std::integral_constant<int, 3>{});
    if (K == 6) return f(std::integral_constant<int, 4>{});
    return f(std::integral_constant<int, 2>{});
}

// Preset PI for counters of encoding E, where its species count has that
// encoding (others are never asked for).
template <int LAT, int E, int PI>
static const void* preset_kernel()
{
    constexpr Preset q = kPresets[PI];
    constexpr int e = q.K <= 4 ? 1 : (q.K == 5 ? 3 : (q.K == 6 ? 4 : 2));
    if constexpr (q.lattice == LAT && e == E) return (const void*)k_ministep<LAT, E, GeoFix<PI>, 1>;
    else return nullptr;
}

template <int LAT, int E>
static const void* stream_kernel(int preset, int nbuf)
{
    static_assert(kNumPresets == 4, "presets by number");
    switch (preset) {
    case 0: return preset_kernel<LAT, E, 0>();
    case 1: return preset_kernel<LAT, E, 1>();
    case 2: return preset_kernel<LAT, E, 2>();
    case 3: return preset_kernel<LAT, E, 3>();
    default: break;
    }
    if (nbuf == 2) return (const void*)k_ministep<LAT, E, GeoRt, 2>;
    return (const void*)k_ministep<LAT, E, GeoRt, 1>;
}

template <int LAT, int E>
static const void* persistent_kernel()
{
    return (const void*)k_persistent<LAT, E, GeoRt>;
}

// Row kernels: a compile-time shell count for 32-bit counters (up to 6
// species; with a runtime one the 2-shell BCC lattice of 795^3 cells took 2.2x
// as long), a runtime one for 64-bit counters.
template <int LAT, int E, int MAXB>
static const void* row_kernel_e(int S)
{
    if constexpr (E != 2) {
        if (S == 1) return (const void*)k_rows<LAT, E, GeoRow<1>, MAXB>;
        if (S == 2) return (const void*)k_rows<LAT, E, GeoRow<2>, MAXB>;
        if (S == 3) return (const void*)k_rows<LAT, E, GeoRow<3>, MAXB>;
        return (const void*)k_rows<LAT, E, GeoRow<4>, MAXB>;
    } else {
        return (const void*)k_rows<LAT, E, GeoRow<0>, MAXB>;
    }
}

template <int MAXB>
static const void* row_kernel_b(int lattice, int K, int S)
{
    return with_encoding(K, [&](auto e) {
        constexpr int E = decltype(e)::value;
        return lattice == SMCX_BCC ? row_kernel_e<SMCX_BCC, E, MAXB>(S) : row_kernel_e<SMCX_FCC, E, MAXB>(S);
    });
}

// The row kernel of compile-time row preset PI or a later one.
template <int PI>
static const void* row_preset_kernel(int preset)
{
    if constexpr (PI < kNumRowPresets) {
        if (preset == PI) {
            constexpr RowPreset q = kRowPresets[PI];
            static_assert(q.K <= 4, "row presets use 8-bit fields");
            constexpr int B = (q.rt0 * q.rt1 * q.rt2 + 63) / 64 * 64;
            return (const void*)k_rows<q.lattice, 1, GeoRowFix<PI>, (B <= kBlock ? kBlock : kMaxRowBlock)>;
        }
        return row_preset_kernel<PI + 1>(preset);
    } else {
        return nullptr;
    }
}

const void* row_kernel(int lattice, int K, int S, int block, int preset)
{
    if (preset >= 0) return row_preset_kernel<0>(preset);
    return block <= kBlock ? row_kernel_b<kBlock>(lattice, K, S) : row_kernel_b<kMaxRowBlock>(lattice, K, S);
}

const void* sweep_kernel(int lattice, int K, bool persistent, int preset, int nbuf)
{
    return with_encoding(K, [&](auto e) {
        constexpr int E = decltype(e)::value;
        if (persistent) return lattice == SMCX_BCC ? persistent_kernel<SMCX_BCC, E>() : persistent_kernel<SMCX_FCC, E>();
        return lattice == SMCX_BCC ? stream_kernel<SMCX_BCC, E>(preset, nbuf) : stream_kernel<SMCX_FCC, E>(preset, nbuf);
    });
}

hipError_t launch_sweep(const void* kernel, dim3 grid, int block, size_t lds, hipStream_t st, const SweepArgs& a)
{
    if (!kernel) return hipErrorInvalidDeviceFunction;
    SweepArgs copy = a;
    void* args[] = {&copy};
    return hipLaunchKernel(kernel, grid, dim3(block), args, lds, st);
}

hipError_t set_sweep_lds_limit(const void* kernel, size_t lds)
{
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

hipError_t sweep_occupancy(const void* kernel, int block, size_t lds, int* blocks_per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, kernel, block, lds);
}

hipError_t launch_pack(int lattice, int K, bool unpack, bool planar, uint8_t* occ, uint8_t* ws,
                       const RepDev* reps, int r, int64_t nrows, int row16, int nrep, int64_t* slots, int parts,
                       int64_t* stats, hipStream_t st)
{
    // replica r, or with r < 0 a grid row per replica (nrep of them); nrows
    // rows and row16 chunks of 16 cells per row of the largest replica
    int64_t nb = planar ? (nrows * row16 + kBlock - 1) / kBlock : (r < 0 ? (nrows + 7) / 8 : nrows);
    nb = std::max<int64_t>(1, std::min<int64_t>(nb, planar ? 1 << 20 : 65536));
    if (r < 0 && (nrep < 1 || nrep > 65535)) return hipErrorInvalidValue;
    const dim3 g((unsigned)nb, r < 0 ? (unsigned)nrep : 1u), b(kBlock);
    const int F = field_bits_of(K);
    auto go = [&](auto mt, auto pt) {
        constexpr int M = decltype(mt)::value;
        constexpr bool PL = decltype(pt)::value;
        if (unpack) hipLaunchKernelGGL((k_unpack<M, PL>), g, b, 0, st, occ, ws, reps, r, F, slots, parts, stats);
        else hipLaunchKernelGGL((k_pack<M, PL>), g, b, 0, st, occ, ws, reps, r, F);
    };
    using T2 = std::integral_constant<int, 2>;
    using T4 = std::integral_constant<int, 4>;
    using Y = std::true_type;
    using N = std::false_type;
    if (lattice == SMCX_BCC) {
        if (planar) go(T2{}, Y{}); else go(T2{}, N{});
    } else {
        if (planar) go(T4{}, Y{}); else go(T4{}, N{});
    }
    return hipGetLastError();
}

hipError_t launch_validate(const uint8_t* occ, int64_t n, int K, int32_t* bad, hipStream_t st)
{
    const int64_t nb = std::max<int64_t>(1, std::min<int64_t>((n / 16 + kBlock - 1) / kBlock, 8192));
    hipLaunchKernelGGL(k_validate, dim3((unsigned)nb), dim3(kBlock), 0, st, occ, n, K, bad);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Replica exchange.  k_energy: E_r = 1/2 sum_{s,k,l} C_r[s][k][l] V[s][k][l],
// accumulated s, k, l ascending in binary64 (the order fixes the rounding, the
// same as the host-side energy): a wave per replica forms the products, one
// lane adds them up (a thread per replica, loading term by term, took 7 to 12
// us where this takes 3 to 5).  k_exchange:
// one round of trades between neighbouring temperature slots (i, i + 1),
// i = round mod 2, round mod 2 + 2, ...: with a = rep_at[i], b = rep_at[i+1]
// and x = (beta_slot[i] - beta_slot[i+1]) (E_a - E_b), the trade is taken
// when x >= 0, else when u < exp(x) (u from Philox on counter
// (i, 0, round, 0xffffffff), which no trial uses); near-ties
// (|u - exp(x)| < 1e-12) go to the tie log as {-1, round, i, decision}.
// One workgroup: every pair of the round has its own thread, so the pairs'
// slots, stats and trades never collide.  Then every replica's new beta is
// written to each of the n_rows rows the next sweeps read.  rep_at entries
// outside [0, R) leave their pair (and their replica's beta) untouched.
// ---------------------------------------------------------------------------
constexpr int kMaxTerms = kMaxShells * kMaxK * kMaxK;

__global__ __launch_bounds__(64) void k_energy(const int64_t* C, const double* V, int R, int SKK, double* E)
{
    __shared__ double p[kMaxTerms];
    for (int r = blockIdx.x; r < R; r += gridDim.x) {
        const int64_t* c = C + (int64_t)r * SKK;
        double acc = 0.0;
        for (int i0 = 0; i0 < SKK; i0 += kMaxTerms) {
            const int n = min(kMaxTerms, SKK - i0);
            for (int i = threadIdx.x; i < n; i += 64) p[i] = (double)c[i0 + i] * V[i0 + i];
            __syncthreads();
            if (threadIdx.x == 0) acc = sum_in_order<1>(acc, p, n);
            __syncthreads();
        }
        if (threadIdx.x == 0) E[r] = 0.5 * acc;
    }
}

__global__ __launch_bounds__(kBlock) void k_exchange(const double* E, const double* beta_slot, int32_t* rep_at, int R,
                                                     uint64_t seed, uint32_t round, double* beta_rows, int n_rows,
                                                     int64_t* xstats, smcx_tie* ties, int32_t tie_cap,
                                                     int32_t* tie_count)
{
    for (int i = (int)(round & 1u) + 2 * (int)threadIdx.x; i + 1 < R; i += 2 * (int)blockDim.x) {
        const int a = rep_at[i], b = rep_at[i + 1];
        if (a < 0 || a >= R || b < 0 || b >= R) continue;
        const double x = (beta_slot[i] - beta_slot[i + 1]) * (E[a] - E[b]);
        bool acc = true, tie = false;
        if (!(x >= 0.0)) {
            uint32_t w0, w1, w2, w3;
            philox4x32_10((uint32_t)i, 0u, round, 0xffffffffu, (uint32_t)seed, (uint32_t)(seed >> 32), w0, w1, w2,
                          w3);
            (void)w0;
            (void)w3;
            const double P = exp(x);
            const double u = (double)(((uint64_t)w1 << 21) | (uint64_t)(w2 >> 11)) * 0x1p-53;
            acc = u < P;
            tie = fabs(u - P) < 1e-12;
        }
        if (tie) {
            const int slot = atomicAdd(tie_count, 1);
            if (slot < tie_cap) {
                smcx_tie e;
                e.replica = -1;
                e.sweep = round;
                e.site = i;
                e.decision = acc ? 1 : 0;
                e.pad = 0;
                ties[slot] = e;
            }
        }
        xstats[2 * i] += 1;
        if (acc) {
            xstats[2 * i + 1] += 1;
            rep_at[i] = b;
            rep_at[i + 1] = a;
        }
    }
    __syncthreads();  // every trade of the round is in rep_at
    for (int j = threadIdx.x; j < R; j += blockDim.x) {
        const int r = rep_at[j];
        if (r < 0 || r >= R) continue;
        const double bj = beta_slot[j];
        for (int row = 0; row < n_rows; ++row) beta_rows[(int64_t)row * R + r] = bj;
    }
}

// Heat capacity per site (units of k_B) of every (step, replica) from its
// recorded energies E[s][j][r], j < n_rec: c = (beta beta) v / N with
// m = (sum_j E) / n_rec and v = (sum_j (E - m)^2) / n_rec, j ascending in
// binary64 (the canonical fluctuation formula); beta = beta_steps[s][r].
__global__ void k_heat_capacity(const double* E, const double* beta_steps, const RepDev* reps, int n_steps,
                                int n_rec, int R, double* cv)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n_steps * R) return;
    const int64_t s = i / R;
    const int r = (int)(i - s * R);
    const double* e = E + s * n_rec * R + r;
    double m = 0.0;
    for (int j = 0; j < n_rec; ++j) m = m + e[(int64_t)j * R];
    m = m / (double)n_rec;
    double v = 0.0;
    for (int j = 0; j < n_rec; ++j) {
        const double d = e[(int64_t)j * R] - m;
        v = v + d * d;
    }
    v = v / (double)n_rec;
    const double b = beta_steps[i];
    cv[i] = b * b * v / (double)reps[r].N;
}

hipError_t launch_heat_capacity(const double* E, const double* beta_steps, const RepDev* reps, int n_steps, int n_rec,
                                int R, double* cv, hipStream_t st)
{
    const int64_t n = (int64_t)n_steps * R;
    hipLaunchKernelGGL(k_heat_capacity, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, E, beta_steps,
                       reps, n_steps, n_rec, R, cv);
    return hipGetLastError();
}

hipError_t launch_energy(const int64_t* C, const double* V, int R, int SKK, double* E, hipStream_t st)
{
    hipLaunchKernelGGL(k_energy, dim3((unsigned)std::min(R, 1 << 20)), dim3(64), 0, st, C, V, R, SKK, E);
    return hipGetLastError();
}

// Gradient of sum_b g_b E_b with respect to V for E_b = 1/2 <C_b, V>:
// grad[i] = 1/2 sum_b g_b C_b[i], b ascending in binary64.  The order makes
// the adds a chain of B, so the work is to keep it fed: a workgroup takes 8
// entries i, its 1024 threads form the products of 1024 configurations, and 8
// lanes add them up while the next loads are on their way (one thread per
// entry, loading as it went, took 984 us for 4096 configurations; this
// 37).
constexpr int kGradEntries = 8, kGradBlock = 1024, kGradTile = 1024, kGradPer = kGradTile * kGradEntries / kGradBlock;

__global__ __launch_bounds__(kGradBlock) void k_energy_grad(const int64_t* C, const double* g, int B, int SKK, double* grad)
{
    __shared__ double p[kGradTile * kGradEntries];  // [configuration][entry]
    const int e = threadIdx.x % kGradEntries, b0 = threadIdx.x / kGradEntries, i = blockIdx.x * kGradEntries + e;
    constexpr int step = kGradBlock / kGradEntries;
    double v[kGradPer];
    auto load = [&](int64_t first) {
#pragma unroll
        for (int k = 0; k < kGradPer; ++k) {
            const int64_t b = first + b0 + k * step;
            v[k] = b < B && i < SKK ? g[b] * (double)C[b * SKK + i] : 0.0;
        }
    };
    double acc = 0.0;
    load(0);
    for (int64_t first = 0; first < B; first += kGradTile) {
        __syncthreads();  // the tile before is added up
#pragma unroll
        for (int k = 0; k < kGradPer; ++k) p[(b0 + k * step) * kGradEntries + e] = v[k];
        __syncthreads();
        if (first + kGradTile < B) load(first + kGradTile);
        if (threadIdx.x < kGradEntries)
            acc = sum_in_order<kGradEntries>(acc, p + threadIdx.x, (int)min((int64_t)kGradTile, B - first));
    }
    const int o = blockIdx.x * kGradEntries + threadIdx.x;
    if (threadIdx.x < kGradEntries && o < SKK) grad[o] = 0.5 * acc;
}

hipError_t launch_energy_grad(const int64_t* C, const double* g, int B, int SKK, double* grad, hipStream_t st)
{
    hipLaunchKernelGGL(k_energy_grad, dim3((unsigned)((SKK + kGradEntries - 1) / kGradEntries)), dim3(kGradBlock), 0, st, C,
                       g, B, SKK, grad);
    return hipGetLastError();
}

hipError_t launch_exchange(const double* E, const double* beta_slot, int32_t* rep_at, int R, uint64_t seed,
                           uint32_t round, double* beta_rows, int n_rows, int64_t* xstats, smcx_tie* ties,
                           int32_t tie_cap, int32_t* tie_count, hipStream_t st)
{
    hipLaunchKernelGGL(k_exchange, dim3(1), dim3(kBlock), 0, st, E, beta_slot, rep_at, R, seed, round, beta_rows,
                       n_rows, xstats, ties, tie_cap, tie_count);
    return hipGetLastError();
}

hipError_t launch_fill_i64(int64_t* p, int64_t n, int64_t v, hipStream_t st)
{
    int64_t nb = (n + kBlock - 1) / kBlock;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_fill_i64, dim3((unsigned)nb), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_advance_counter(uint32_t* counter, uint32_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_advance_counter, dim3(1), dim3(64), 0, st, counter, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Static workspace for smcx_lattice_init_static: a file-scope device array, so
// that a caller that cannot allocate device memory still gets a workspace.
// Every device holds its own copy at its own address, resolved here once per
// device (that device current) with hipGetSymbolAddress; host code passes
// that address on, never the array's name, which in host code is only a
// stand-in for the symbol.
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[kStaticWorkspaceBytes];

hipError_t static_workspace(void** ptr)
{
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

}  // namespace smcx
