// Local energies of sites and clusters of low-energy sites.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "smcx_device.h"
#include "smcx_internal.h"
#include "smcx_launch.h"

namespace smcx {

// ---------------------------------------------------------------------------
// Local energies: e_i = 1/2 sum_s sum_t n_i[s][t] V_s[sigma_i][t] (s, t
// ascending, binary64), n_i[s][t] the shell-s neighbours of species t with
// periodic images.
//
// A workgroup stages TX x (256 / TX) x TZ cells and a 2-cell halo in LDS, as F
// * species; a lane walks a column of TZ cells.  A neighbour is one LDS byte at
// a compile-time offset and one shift-add into F-bit fields.  Bound by VALU
// issue and, with it, the windows per CU: BCC 250x199x221 (4 species, 4
// shells) takes 160 us with 32 x 8 x 8 cells, 174 with 64 x 4 x 8, 195 with
// 64 x 4 x 16 (and a table of the products n V, which costs more LDS than it
// saves), 206 with three operations per neighbour; FCC 120x110x100 (5 species)
// 65 us, 138 with every neighbour from global memory.
// ---------------------------------------------------------------------------
template <int LAT, int E, int TX, int TZ>
__global__ __launch_bounds__(kBlock) void k_local_energy(const uint8_t* occ, int L0, int L1, int L2, int K, int S,
                                                         const double* V, double* e)
{
    using EN = Enc<E>;
    using CT = typename EN::T;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m, F = EN::F;
    constexpr int TY = kBlock / TX;
    constexpr int WX = TX + 2 * kHalo, WY = TY + 2 * kHalo, WZ = TZ + 2 * kHalo;
    constexpr int LP = WX * m, PL = LP * WY;
    using Cell = typename std::conditional<m == 4, uint32_t, uint16_t>::type;
    __shared__ __align__(16) uint8_t win[PL * WZ];
    __shared__ double Vs[kMaxShells * EN::KP * EN::KP];
    const int KK = K * K;
    for (int i = threadIdx.x; i < S * KK; i += kBlock) Vs[i] = V[i];
    const int ntx = (L0 + TX - 1) / TX, nty = (L1 + TY - 1) / TY, ntz = (L2 + TZ - 1) / TZ;
    const int64_t ntiles = (int64_t)ntx * nty * ntz;
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    auto wrap = [](int v, int L) {
        v += v < 0 ? L : 0;
        v -= v >= L ? L : 0;
        return v >= L ? v % L : v;  // only lattices narrower than a tile wrap twice
    };
    for (int64_t ti = blockIdx.x; ti < ntiles; ti += gridDim.x) {
        const int tx = (int)(ti % ntx);
        const int64_t tr = ti / ntx;
        const int ty = (int)(tr % nty), tz = (int)(tr / nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
        __syncthreads();  // every lane is done with the previous tile (and Vs is in place)
        for (int c = threadIdx.x; c < WX * WY * WZ; c += kBlock) {
            const int wx = c % WX, wr = c / WX, wy = wr % WY, wz = wr / WY;
            const int x = wrap(x0 + wx - kHalo, L0), y = wrap(y0 + wy - kHalo, L1), z = wrap(z0 + wz - kHalo, L2);
            Cell v;
            __builtin_memcpy(&v, occ + (int64_t)m * (x + (int64_t)L0 * (y + (int64_t)L1 * z)), m);
            *(Cell*)(win + m * c) = (Cell)(v * (uint32_t)F);
        }
        __syncthreads();
        if (x0 + lx >= L0 || y0 + ly >= L1) continue;
        for (int lz = 0; lz < TZ && z0 + lz < L2; ++lz) {
            const int64_t cell = (x0 + lx) + (int64_t)L0 * ((y0 + ly) + (int64_t)L1 * (z0 + lz));
            double out[m];
#pragma unroll
            for (int b = 0; b < m; ++b) {
                const int base = ((lz + kHalo) * WY + (ly + kHalo)) * LP + (lx + kHalo) * m + b;
                const int p = min(species_of(win[base], F), K - 1);  // checked < K at init
                CT h[kMaxShells];
#pragma unroll
                for (int s = 0; s < kMaxShells; ++s) {
                    h[s] = 0;
                    if (s < S) {
                        uint32_t v[kMaxZ];
#pragma unroll
                        for (int n = 0; n < G.Z[s]; ++n) {
                            const Nb nb = nb_of(G, b, G.v[s][n][0], G.v[s][n][1], G.v[s][n][2]);
                            v[n] = win[base + nb.dz * PL + nb.dy * LP + m * nb.dx + (nb.bt - b)];
                        }
#pragma unroll
                        for (int n = 0; n < G.Z[s]; ++n) h[s] = shl1_add(v[n], h[s]);
                    }
                }
                double en = 0.0;
                const double* row = Vs + p * K;
#pragma unroll
                for (int s = 0; s < kMaxShells; ++s)
                    if (s < S) {
                        int left = G.Z[s];  // a species whose field has no room for it is what the others leave
#pragma unroll
                        for (int t = 0; t < EN::KP; ++t) {
                            const bool whole = F * (t + 1) <= 8 * (int)sizeof(CT);
                            const int c = whole ? (int)((h[s] >> (whole ? F * t : 0)) & EN::mask) : left;
                            left -= c;
                            if (t < K) en = en + (double)c * row[s * KK + t];
                        }
                    }
                out[b] = 0.5 * en;
            }
            __builtin_memcpy(e + m * cell, out, sizeof(out));
        }
    }
}

// The same for lattices of few sites and 5 or more species, a thread per cell
// and every neighbour from memory: no window to stage first, and one cell's
// chain instead of a column's.  us, tiles in brackets: FCC 9^3 of 8 species and
// 4 shells 11.8 (30.5), 48^3 19.0 (32.4), BCC 64^3 17.2 (20.1), of 5 species and 2
// shells 7.7 (11.6), 16^3 4.4 (10.3).  Rows of 17 to 20 cells, a third of whose
// two tiles would be empty, take it at every size (FCC 20x20x2000 of 8 species
// 82 (104)).
template <int LAT, int B>
__device__ __forceinline__ void local_energy_cell(const uint8_t* occ, int c, int x, int y, int z, int L0, int L1, int L2,
                                                  int K, int S, const double* Vs, double* e)
{
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m;
    if constexpr (B < m) {
        uint64_t acc[kMaxShells];
#pragma unroll
        for (int s = 0; s < kMaxShells; ++s) {
            uint64_t a = 0;
            if (s < S) {
#pragma unroll
                for (int n = 0; n < G.Z[s]; ++n) {
                    const Nb nb = nb_of(G, B, G.v[s][n][0], G.v[s][n][1], G.v[s][n][2]);
                    int xx = x + nb.dx, yy = y + nb.dy, zz = z + nb.dz;
                    xx += xx < 0 ? L0 : (xx >= L0 ? -L0 : 0);
                    yy += yy < 0 ? L1 : (yy >= L1 ? -L1 : 0);
                    zz += zz < 0 ? L2 : (zz >= L2 ? -L2 : 0);
                    const uint32_t t = occ[nb.bt + m * (xx + L0 * (yy + L1 * zz))] & 7u;  // species < K <= 8
                    a += (uint64_t)1 << (8 * t);
                }
            }
            acc[s] = a;
        }
        const int p = min((int)occ[B + m * c], K - 1);  // checked < K at init
        double en = 0.0;
#pragma unroll
        for (int s = 0; s < kMaxShells; ++s)
            if (s < S)
                for (int t = 0; t < K; ++t)
                    en = en + (double)(int)((acc[s] >> (8 * t)) & 0xff) * Vs[(s * K + p) * K + t];
        e[B + m * c] = 0.5 * en;
        local_energy_cell<LAT, B + 1>(occ, c, x, y, z, L0, L1, L2, K, S, Vs, e);
    }
}

template <int LAT>
__global__ __launch_bounds__(kBlock) void k_local_energy_cells(const uint8_t* occ, int L0, int L1, int L2, int K, int S,
                                                               const double* V, double* e)
{
    __shared__ double Vs[kMaxShells * kMaxK * kMaxK];
    for (int i = threadIdx.x; i < S * K * K; i += kBlock) Vs[i] = V[i];
    __syncthreads();
    const int ncell = L0 * L1 * L2;
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < ncell; c += gridDim.x * kBlock) {
        const int cr = c / L0, x = c - cr * L0, z = cr / L1, y = cr - z * L1;
        local_energy_cell<LAT, 0>(occ, c, x, y, z, L0, L1, L2, K, S, Vs, e);
    }
}

template <int LAT, int E>
static void local_energy_go(const uint8_t* occ, const int32_t* L, int K, int S, const double* V, double* e, hipStream_t st)
{
    // shallower tiles for lattices that would leave CUs idle (the shallowest
    // where a lane's chain is longest, past 4 species: FCC 64^3 of 5 species and 2
    // shells 11.8 us against 17.2, BCC 80^3 11.8 against 13.5; at twice the sites
    // the staging costs as much); narrow ones for narrow lattices
    const int64_t ncell = (int64_t)L[0] * L[1] * L[2], sites = kGeom[LAT].m * ncell;
    if (E != 1 && (sites <= 1 << 19 || (L[0] > 16 && L[0] <= 20))) {
        hipLaunchKernelGGL(k_local_energy_cells<LAT>, dim3((unsigned)((ncell + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, occ,
                           L[0], L[1], L[2], K, S, V, e);
        return;
    }
    auto tiles = [&](int TX, int TZ) {
        const int TY = kBlock / TX;
        return (int64_t)((L[0] + TX - 1) / TX) * ((L[1] + TY - 1) / TY) * ((L[2] + TZ - 1) / TZ);
    };
    auto go = [&](auto tx, auto tz) {
        constexpr int TX = decltype(tx)::value, TZ = decltype(tz)::value;
        const unsigned g = (unsigned)std::min<int64_t>(tiles(TX, TZ), 1 << 20);
        hipLaunchKernelGGL((k_local_energy<LAT, E, TX, TZ>), dim3(g), dim3(kBlock), 0, st, occ, L[0], L[1], L[2], K, S, V, e);
    };
    using std::integral_constant;
    if (L[0] <= 20) go(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    else if (E != 1 && sites <= 3 << 19) go(integral_constant<int, 32>{}, integral_constant<int, 2>{});
    else if (tiles(32, 8) < 2048) go(integral_constant<int, 32>{}, integral_constant<int, 4>{});
    else go(integral_constant<int, 32>{}, integral_constant<int, 8>{});
}

hipError_t launch_local_energy(int lattice, const uint8_t* occ, const int32_t* L, int K, int S, const double* V,
                               double* e, hipStream_t st)
{
    auto go = [&](auto lat) {
        constexpr int LAT = decltype(lat)::value;
        if (K <= 4) local_energy_go<LAT, 1>(occ, L, K, S, V, e, st);
        else if (K == 5) local_energy_go<LAT, 3>(occ, L, K, S, V, e, st);
        else if (K == 6) local_energy_go<LAT, 4>(occ, L, K, S, V, e, st);
        else local_energy_go<LAT, 2>(occ, L, K, S, V, e, st);
    };
    if (lattice == SMCX_BCC) go(std::integral_constant<int, SMCX_BCC>{});
    else go(std::integral_constant<int, SMCX_FCC>{});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Clusters: site i is marked when e_i <= threshold; marked nearest neighbours
// join, and a cluster's label is its smallest site.  Union-find in which a
// parent is never larger than its child: a union hooks the larger of two roots
// under the smaller (compare-and-swap), so the smallest site of a cluster is
// its final root, whatever the order of the unions; a failed hook goes on from
// the value the swap returned and a find only descends, so both loops end.
//
// Most bonds lie inside a tile of 4096 sites: k_cluster_tiles marks, joins and
// counts a tile's sites in LDS, and leaves every site pointing at the smallest
// site of its piece and that site holding the piece's size.  k_cluster_merge
// joins the pieces over the bonds that leave their tile (one bond in eight) in
// global memory, where every access to a parent is an agent-scope atomic (the
// L2 of one XCD does not see another's plain stores).  k_cluster_label points
// every site at its root and moves the pieces' sizes there.  With all unions
// in global memory and an atomic per site and wave, BCC 250x199x221 with a
// sixth of the sites marked took 60 + 632 + 315 us; now 209 + 127 + 77 (where they form one large cluster,
// 5.6 ms, now 0.9).
// ---------------------------------------------------------------------------
template <int SCOPE>
__device__ __forceinline__ int32_t par_load(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, SCOPE);
}

// Root of x; entries on the way are pointed at their grandparents (while
// trees still merge any ancestor will do).
template <int SCOPE>
__device__ __forceinline__ int32_t cluster_find(int32_t* parent, int32_t x)
{
    while (true) {
        const int32_t p = par_load<SCOPE>(parent + x);
        if (p == x) return x;
        const int32_t gp = par_load<SCOPE>(parent + p);
        if (gp != p) __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, SCOPE);
        x = gp;
    }
}

template <int SCOPE>
__device__ __forceinline__ void cluster_union(int32_t* parent, int32_t a, int32_t b)
{
    while (true) {
        a = cluster_find<SCOPE>(parent, a);
        b = cluster_find<SCOPE>(parent, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        int32_t expected = a;  // hook root a under the smaller root b
        if (__hip_atomic_compare_exchange_strong(parent + a, &expected, b, __ATOMIC_RELAXED, __ATOMIC_RELAXED, SCOPE)) return;
        a = expected;  // a was no longer a root: go on from its parent (< a)
    }
}

// Tiles of whole cells; sites are numbered in a tile in the order they have in
// the lattice, so the smallest site of a piece is the same by either number.
template <int LAT>
struct ClusterTile {
    static constexpr int m = kGeom[LAT].m;
    static constexpr int TX = LAT == SMCX_BCC ? 32 : 16, TY = 8, TZ = 8, SITES = TX * TY * TZ * m;
};

// One direction of every nearest-neighbour bond.
constexpr bool bond_once(const int (&v)[3]) { return v[2] > 0 || (v[2] == 0 && (v[1] > 0 || (v[1] == 0 && v[0] > 0))); }

template <int LAT>
__global__ __launch_bounds__(kBlock) void k_cluster_tiles(const double* e, int L0, int L1, int L2, double threshold,
                                                          int32_t* label, int32_t* size)
{
    using T = ClusterTile<LAT>;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m, SC = __HIP_MEMORY_SCOPE_WORKGROUP;
    __shared__ int32_t parent[T::SITES], count[T::SITES];
    __shared__ uint16_t marked[T::SITES];  // the tile's marked sites, in any order
    __shared__ int nmarked;
    if (threadIdx.x == 0) nmarked = 0;
    __syncthreads();
    const int ntx = (L0 + T::TX - 1) / T::TX, nty = (L1 + T::TY - 1) / T::TY;
    const int tx = blockIdx.x % ntx, tr = blockIdx.x / ntx, ty = tr % nty, tz = tr / nty;
    const int x0 = tx * T::TX, y0 = ty * T::TY, z0 = tz * T::TZ;
    const int nx = min(T::TX, L0 - x0), ny = min(T::TY, L1 - y0), nz = min(T::TZ, L2 - z0);
    constexpr int ROW = T::TX * m;
    auto site = [&](int li) {  // lattice site of tile site li, or -1 outside the lattice
        const int b = li % m, lx = li / m % T::TX, ly = li / ROW % T::TY, lz = li / (ROW * T::TY);
        return lx < nx && ly < ny && lz < nz ? b + m * ((x0 + lx) + L0 * ((y0 + ly) + L1 * (z0 + lz))) : -1;
    };
    // A sixth of the sites marked, say, leaves five lanes in six idle in every
    // later loop: the marked ones are listed and the loops run over the list.
    const int lane = threadIdx.x & 63;
    constexpr int PER = T::SITES / kBlock;
    double ev[PER];  // all loads on their way before the first is looked at
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = site(threadIdx.x + k * kBlock);
        ev[k] = i >= 0 ? e[i] : __builtin_nan("");
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int li = threadIdx.x + k * kBlock;
        const bool in = ev[k] <= threshold;
        parent[li] = in ? li : -1;
        count[li] = 0;
        const uint64_t mask = __ballot(in);
        int at = 0;
        if (lane == 0 && mask) at = atomicAdd(&nmarked, __popcll(mask));
        at = __builtin_amdgcn_readfirstlane(at);
        if (in) marked[at + __popcll(mask & ((1ull << lane) - 1))] = (uint16_t)li;
    }
    __syncthreads();
    const int nm = nmarked;
    // Neighbour n of tile site li inside the tile, or -1.
    auto neighbour = [&](int li, const int (&v)[3]) {
        const int b = li % m, lx = li / m % T::TX, ly = li / ROW % T::TY, lz = li / (ROW * T::TY);
        const int bx = m == 2 ? b : (b == 1 || b == 2), by = m == 2 ? b : b & 1, bz = m == 2 ? b : b >> 1;
        const Nb nb = nb_of(G, 0, v[0], v[1], v[2]);
        const int xx = lx + nb.dx + (v[0] & 1 & bx), yy = ly + nb.dy + (v[1] & 1 & by), zz = lz + nb.dz + (v[2] & 1 & bz);
        const bool in = xx >= 0 && xx < nx && yy >= 0 && yy < ny && zz >= 0 && zz < nz;
        return in ? (nb.bt ^ b) + m * (xx + T::TX * (yy + T::TY * zz)) : -1;
    };
    // A site's first bond to a smaller marked site needs no union: it points
    // there (a forest, as parents are smaller).  Its other bonds to smaller
    // sites are noted and joined afterwards.
    for (int k = threadIdx.x; k < nm; k += kBlock) {
        const int li = marked[k];
        int first = li, rest = 0;
#pragma unroll
        for (int n = 0; n < G.Z[0]; ++n) {
            const int lj = neighbour(li, G.v[0][n]);
            if (lj < 0 || lj >= li || parent[lj] < 0) continue;  // marks (>= 0) never change
            if (first == li) first = lj;
            else rest |= 1 << n;
        }
        parent[li] = first;
        count[li] = rest;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nm; k += kBlock) {
        const int li = marked[k];
        const int rest = count[li];
        count[li] = 0;
#pragma unroll
        for (int n = 0; n < G.Z[0]; ++n)
            if (rest >> n & 1) cluster_union<SC>(parent, li, neighbour(li, G.v[0][n]));
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nm; k += kBlock) {
        const int li = marked[k];
        int32_t p = parent[li];
        while (parent[p] != p) p = parent[p];  // the trees are final
        atomicAdd(&count[p], 1);
        if (p != li) parent[li] = p;  // an ancestor, for whoever passes by
    }
    __syncthreads();
#pragma unroll 4
    for (int li = threadIdx.x; li < T::SITES; li += kBlock) {
        const int i = site(li);
        if (i < 0) continue;
        const int p = parent[li];
        label[i] = p < 0 ? -1 : site(p);
        size[i] = count[li];
    }
}

template <int LAT>
__global__ __launch_bounds__(kBlock) void k_cluster_merge(int32_t* label, int L0, int L1, int L2)
{
    using T = ClusterTile<LAT>;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m;
    const int ncell = L0 * L1 * L2;
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < ncell; c += gridDim.x * kBlock) {
        const int cr = c / L0, x = c - cr * L0, z = cr / L1, y = cr - z * L1;
        // the tile's cells around this one; a cell clear of its faces has no bond that leaves
        const int lx = x % T::TX, ly = y % T::TY, lz = z % T::TZ;
        const int nx = min(T::TX, L0 - (x - lx)), ny = min(T::TY, L1 - (y - ly)), nz = min(T::TZ, L2 - (z - lz));
        if (lx > 0 && lx < nx - 1 && ly > 0 && ly < ny - 1 && lz < nz - 1) continue;
        int32_t own[m];  // marks never change: plain loads will do
        __builtin_memcpy(own, label + m * c, sizeof(own));
        constexpr int NB = G.Z[0] / 2;
#pragma unroll
        for (int b = 0; b < m; ++b) {
            if (own[b] < 0) continue;
            int32_t far[NB];  // the sites over the faces, all on their way at once
            int k = 0;
#pragma unroll
            for (int n = 0; n < G.Z[0]; ++n) {
                if (!bond_once(G.v[0][n])) continue;
                const Nb nb = nb_of(G, b, G.v[0][n][0], G.v[0][n][1], G.v[0][n][2]);
                const int ux = lx + nb.dx, uy = ly + nb.dy, uz = lz + nb.dz;
                int xx = x + nb.dx, yy = y + nb.dy, zz = z + nb.dz;
                xx += xx < 0 ? L0 : (xx >= L0 ? -L0 : 0);
                yy += yy < 0 ? L1 : (yy >= L1 ? -L1 : 0);
                zz += zz < 0 ? L2 : (zz >= L2 ? -L2 : 0);
                const bool inside = ux >= 0 && ux < nx && uy >= 0 && uy < ny && uz >= 0 && uz < nz;  // joined in the tile
                far[k] = -1;
                if (!inside) far[k] = label[nb.bt + m * (xx + L0 * (yy + L1 * zz))];
                ++k;
            }
            // an entry is an ancestor of its site: as good a place to start
#pragma unroll
            for (int n = 0; n < NB; ++n)
                if (far[n] >= 0) cluster_union<__HIP_MEMORY_SCOPE_AGENT>(label, own[b], far[n]);
        }
    }
}

// The trees no longer merge (an out-of-date entry is still an ancestor): every
// site takes its root, a piece's first site (the one with a size) hands its
// size over.
constexpr int kLabelBlock = 1024;

__global__ __launch_bounds__(kLabelBlock) void k_cluster_label(int32_t* label, int N, int32_t* size, int64_t* n_clusters)
{
    __shared__ int total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    int roots = 0;
    constexpr int U = 4;  // sites of a thread whose loads are on their way together
    const int64_t step = (int64_t)gridDim.x * kLabelBlock;
    for (int64_t i0 = blockIdx.x * (int64_t)kLabelBlock + threadIdx.x; i0 < N; i0 += U * step) {
        int32_t p[U], r[U], n[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = i0 + u * step < N ? label[i0 + u * step] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            r[u] = p[u] >= 0 ? label[p[u]] : -1;
            n[u] = p[u] >= 0 ? size[i0 + u * step] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (p[u] < 0) continue;
            const int i = (int)(i0 + u * step);
            int32_t q = p[u];
            while (r[u] != q) {
                q = r[u];
                r[u] = label[q];
            }
            if (q == i) {
                ++roots;
                continue;
            }
            if (q != p[u]) label[i] = q;
            if (n[u] > 0) {
                atomicAdd(size + q, n[u]);
                size[i] = 0;
            }
        }
    }
    const int w = wave_sum_i(roots);
    if ((threadIdx.x & 63) == 0 && w) atomicAdd(&total, w);
    __syncthreads();
    if (threadIdx.x == 0 && total) atomicAdd((unsigned long long*)n_clusters, (unsigned long long)total);
}

hipError_t launch_clusters(int lattice, const double* e, const int32_t* L, double threshold, int32_t* label,
                           int32_t* size, int64_t* n_clusters, hipStream_t st)
{
    const int m = lattice == SMCX_BCC ? 2 : 4;
    const int64_t ncell = (int64_t)L[0] * L[1] * L[2];
    const int N = (int)(m * ncell);
    const unsigned nbc = (unsigned)std::min<int64_t>((ncell + kBlock - 1) / kBlock, 1 << 20);
    // two label workgroups per CU: each ends with one atomic on the cluster count
    const unsigned nbl = (unsigned)std::min<int64_t>(((int64_t)N + kLabelBlock - 1) / kLabelBlock, 512);
    hipError_t err = launch_fill_i64(n_clusters, 1, 0, st);
    if (err != hipSuccess) return err;
    auto go = [&](auto lat) {
        constexpr int LAT = decltype(lat)::value;
        using T = ClusterTile<LAT>;
        const int64_t tiles = (int64_t)((L[0] + T::TX - 1) / T::TX) * ((L[1] + T::TY - 1) / T::TY) * ((L[2] + T::TZ - 1) / T::TZ);
        hipLaunchKernelGGL(k_cluster_tiles<LAT>, dim3((unsigned)tiles), dim3(kBlock), 0, st, e, L[0], L[1], L[2], threshold,
                           label, size);
        hipLaunchKernelGGL(k_cluster_merge<LAT>, dim3(nbc), dim3(kBlock), 0, st, label, L[0], L[1], L[2]);
    };
    if (lattice == SMCX_BCC) go(std::integral_constant<int, SMCX_BCC>{});
    else go(std::integral_constant<int, SMCX_FCC>{});
    hipLaunchKernelGGL(k_cluster_label, dim3(nbl), dim3(kLabelBlock), 0, st, label, N, size, n_clusters);
    return hipGetLastError();
}

}  // namespace smcx
