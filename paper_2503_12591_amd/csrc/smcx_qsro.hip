// Sweeps under the nonlinear (quadratic, qSRO) model.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "smcx_device.h"
#include "smcx_internal.h"
#include "smcx_launch.h"

namespace smcx {

// ---------------------------------------------------------------------------
// qSRO model: trials whose energy change needs every local energy of the
// swap's interaction zone.  E_i = sum_m sum_t V_m[p][t] (n_i[m][t] / Z_m)
// + sum_m W_m[p] (n_i[m][p] / Z_m)^2 (p = sigma_i; m, then t, ascending,
// binary64).  A wave takes one trial (the same Philox draw, partner and
// acceptance rule as the pair model); its lanes take the sites of the
// affected set (a, the partner and every shell neighbour of either, in the
// host table's order), recount each one's neighbours before and after the
// swap (the swap applied to the two sites on the fly) and leave
// E_after - E_before in LDS; lane 0 adds the terms in table order, decides
// and writes the swap.  The sites are read from the natural layout; the
// partition keeps every read of a mini-step's trial clear of the other
// trials' writes (interaction-zone rule).
// ---------------------------------------------------------------------------

__device__ __forceinline__ int qsro_site_of(const QsroArgs& A, int x, int y, int z, int32_t d, int m)
{
    // d packs (dx + 8) | (dy + 8) << 8 | (dz + 8) << 16 | basis << 24
    int xx = x + (d & 0xff) - 8, yy = y + ((d >> 8) & 0xff) - 8, zz = z + ((d >> 16) & 0xff) - 8;
    xx += xx < 0 ? A.L0 : (xx >= A.L0 ? -A.L0 : 0);
    yy += yy < 0 ? A.L1 : (yy >= A.L1 ? -A.L1 : 0);
    zz += zz < 0 ? A.L2 : (zz >= A.L2 ? -A.L2 : 0);
    return ((d >> 24) & 3) + m * (xx + A.L0 * (yy + A.L1 * zz));
}

// Tables of a qSRO launch in LDS: V and W, and every fraction n / Z_s
// (n = 0 .. Z_s), each the correctly rounded quotient, so a lookup gives the
// value the division would.
struct QsroTables {
    double V[kMaxShells * 8 * 8];
    double W[kMaxShells * 8];
    double F[kMaxShells * kQsroFrac];
};

// (for workgroups of one wave: the launch's block size is a load from a cache
// line of its own, 0.2 us at the start of every launch)
__device__ __forceinline__ void qsro_tables(const QsroArgs& A, QsroTables& T)
{
    for (int i = threadIdx.x; i < A.S * A.K * A.K; i += 64) T.V[i] = A.V[i];
    for (int i = threadIdx.x; i < A.S * A.K; i += 64) T.W[i] = A.W[i];
    for (int i = threadIdx.x; i < A.S * kQsroFrac; i += 64) {
        const int s = i / kQsroFrac, n = i - s * kQsroFrac;
        T.F[i] = (double)n / (double)A.Z[s];
    }
    __syncthreads();
}

__device__ __forceinline__ double qsro_energy(const QsroArgs& A, const QsroTables& T, int p,
                                              const uint64_t (&n)[kMaxShells])
{
    double acc = 0.0;
    for (int s = 0; s < A.S; ++s)
        for (int t = 0; t < A.K; ++t)
            acc = acc + T.V[(s * A.K + p) * A.K + t] * T.F[s * kQsroFrac + (int)((n[s] >> (8 * t)) & 0xff)];
    for (int s = 0; s < A.S; ++s) {
        const double f = T.F[s * kQsroFrac + (int)((n[s] >> (8 * p)) & 0xff)];
        acc = acc + T.W[s * A.K + p] * (f * f);
    }
    return acc;
}

template <int LAT>
__global__ __launch_bounds__(64) void k_qsro_ministep(QsroArgs A)
{
    constexpr int m = kGeom[LAT].m;
    __shared__ double term[kQsroMaxAff];
    __shared__ QsroTables tab;
    qsro_tables(A, tab);
    const int lane = threadIdx.x;
    const int ncell = A.ncx * A.ncy * A.ncz;
    const int32_t* ox = A.org;
    const int32_t* oy = ox + A.ncx + 1;
    const int32_t* oz = oy + A.ncy + 1;
    int att = 0, nacc = 0, ntie = 0;
    for (int c = blockIdx.x; c < ncell; c += gridDim.x) {
        const int cx = c % A.ncx, cy = (c / A.ncx) % A.ncy, cz = c / (A.ncx * A.ncy);
        if (A.o0 >= ox[cx + 1] - ox[cx] || A.o1 >= oy[cy + 1] - oy[cy] || A.o2 >= oz[cz + 1] - oz[cz]) continue;
        const int x = ox[cx] + A.o0, y = oy[cy] + A.o1, z = oz[cz] + A.o2;
        const int a = A.b + m * (x + A.L0 * (y + A.L1 * z));
        uint32_t w0, w1, w2, w3;
        philox4x32_10((uint32_t)a, 0u, A.sweep, A.replica, (uint32_t)A.seed, (uint32_t)(A.seed >> 32), w0, w1, w2, w3);
        (void)w3;
        const int k = (int)__umulhi(w0, (uint32_t)A.Z1);
        const int bsite = qsro_site_of(A, x, y, z, A.nbr[A.b * A.sumZ + k], m);
        const int p = A.occ[a], q = A.occ[bsite];
        ++att;
        if (p == q) continue;
        const int32_t* list = A.aff + (int64_t)(A.b * A.Z1 + k) * (1 + A.naff_max);
        const int naff = list[0];
        for (int i = lane; i < naff; i += 64) {
            const int j = qsro_site_of(A, x, y, z, list[1 + i], m);
            const int jb = j % m, jc = j / m;
            const int jx = jc % A.L0, jy = (jc / A.L0) % A.L1, jz = jc / (A.L0 * A.L1);
            const int sj = A.occ[j];
            const int sj2 = j == a ? q : (j == bsite ? p : sj);
            uint64_t nb[kMaxShells], na[kMaxShells];
            const int32_t* nl = A.nbr + jb * A.sumZ;
            int off = 0;
            for (int s = 0; s < kMaxShells; ++s) {
                uint64_t cb = 0, ca = 0;
                if (s < A.S) {
                    for (int n = 0; n < A.Z[s]; ++n) {
                        const int xs = qsro_site_of(A, jx, jy, jz, nl[off + n], m);
                        const int v = A.occ[xs];
                        const int v2 = xs == a ? q : (xs == bsite ? p : v);
                        cb += (uint64_t)1 << (8 * (v & 7));
                        ca += (uint64_t)1 << (8 * (v2 & 7));
                    }
                    off += A.Z[s];
                }
                nb[s] = cb;
                na[s] = ca;
            }
            term[i] = qsro_energy(A, tab, min(sj2, A.K - 1), na) - qsro_energy(A, tab, min(sj, A.K - 1), nb);
        }
        __syncthreads();
        if (lane == 0) {
            double dE = 0.0;
            for (int i = 0; i < naff; ++i) dE = dE + term[i];
            bool acc = true, tie = false;
            if (!(dE <= 0.0)) {
                const double P = exp(-(A.beta * dE));
                const double u = (double)(((uint64_t)w1 << 21) | (uint64_t)(w2 >> 11)) * 0x1p-53;
                acc = u < P;
                tie = fabs(u - P) < 1e-12;
            }
            if (tie) {
                ++ntie;
                const int slot = atomicAdd(A.tie_count, 1);
                if (slot < A.tie_cap) {
                    smcx_tie e;
                    e.replica = (int32_t)A.replica;
                    e.sweep = A.sweep;
                    e.site = a;
                    e.decision = acc ? 1 : 0;
                    e.pad = 0;
                    A.ties[slot] = e;
                }
            }
            if (acc) {
                ++nacc;
                A.occ[a] = (uint8_t)q;
                A.occ[bsite] = (uint8_t)p;
            }
        }
        __syncthreads();  // the terms are free again
    }
    if (lane == 0) {
        // this workgroup's own counter slot (no other workgroup of the
        // launch writes it; launches on one stream follow each other), so no
        // atomics: thousands of atomics on one address would serialise
        int64_t* slot = A.slots + 3 * (int64_t)blockIdx.x;
        slot[0] += att;
        slot[1] += nacc;
        slot[2] += ntie;
    }
}

// ---------------------------------------------------------------------------
// The trials of every basis site of a cell at one offset, neighbourhood
// staged: the wave first copies the box of (2 reach + 1)^3 cells around the
// active cell (periodic, one load per cell of m bytes) into LDS, then makes
// the m trials in turn.  The active site moves by at most one half-unit per
// axis between them, so other cells' swaps stay outside what they read as long
// as 2 e - 1 > 2 + 2 c_max for every cell edge e, which the interaction-zone
// rule already gives (2 e > 2 + 2 c_max, both sides even).  Each lattice site
// appears once in the box because every edge is at least 2 reach + 1 cells;
// bytes that no trial of this cell reads may be written by other waves
// meanwhile, which is harmless.
//
// A lane takes an affected site (an entry of the host's table, which also
// says in which of its shells the active site and the partner lie): all its
// neighbours are read at fixed offsets at once (one base per parity class, as
// the window bytes of a neighbour vector differ between basis sites only by
// its carries), the counts after the swap are the counts before with those
// one or two neighbours moved, and both energies are sums of products looked
// up in LDS (V_s[p][t] n / Z_s and W_s[p] (n / Z_s)^2, each rounded as the
// sums round them).  The differences meet in LDS and every lane adds them in
// table order.  Bound by latency: 17.7 us per launch of four trials at FCC 64^3
// (5 species, 2 shells, 4096 cells, a wave each), against 15 us per trial with
// a launch per basis site, loops over neighbour tables and one lane adding.
// ---------------------------------------------------------------------------
constexpr int qsro_reach(int lattice, int S)
{
    const Geometry G = kGeom[lattice];
    auto far = [](const Nb& n) {
        const int x = n.dx < 0 ? -n.dx : n.dx, y = n.dy < 0 ? -n.dy : n.dy, z = n.dz < 0 ? -n.dz : n.dz;
        return x > y ? (x > z ? x : z) : (y > z ? y : z);
    };
    int ra = 0, rn = 0;
    for (int b = 0; b < G.m; ++b)
        for (int s = 0; s < S; ++s)
            for (int n = 0; n < G.Z[s]; ++n) {
                const int* v = G.v[s][n];
                const int f = far(nb_of(G, b, v[0], v[1], v[2]));
                rn = f > rn ? f : rn;
                ra = f > ra ? f : ra;
                for (int k = 0; k < G.Z[0]; ++k) {
                    const int* p = G.v[0][k];
                    const int g = far(nb_of(G, b, p[0] + v[0], p[1] + v[1], p[2] + v[2]));
                    ra = g > ra ? g : ra;
                }
            }
    return ra + rn;
}

constexpr int kQsroWaves = 4;  // waves (cells) per workgroup

template <int LAT, int S, int E>
__global__ __launch_bounds__(64 * kQsroWaves) void k_qsro_cell(QsroArgs A)
{
    using EN = Enc<E>;
    using CT = typename EN::T;  // neighbour counts, F bits per species; the box holds F * species
    constexpr int KP = EN::KP, F = EN::F;
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m, Z1 = G.Z[0], Rch = qsro_reach(LAT, S), W = 2 * Rch + 1, W3 = W * W * W;
    constexpr int LP = W * m, PL = W * W * m, SZ = sum_Z(G, S);
    constexpr int NL = (2 + 2 * SZ + 63) / 64;  // affected sites per lane, at most
    using Cell = typename std::conditional<m == 4, uint32_t, uint16_t>::type;
    extern __shared__ __align__(16) double gtab[];  // products: [S][K][K][n], then [S][K][n], n < kQsroFrac
    __shared__ double term[kQsroWaves][NL * 64];
    __shared__ __align__(16) uint8_t boxes[kQsroWaves][(W3 * m + 15) & ~15];
    const int K = A.K, KF = K * kQsroFrac, SKKF = S * K * KF;
    for (int i = threadIdx.x; i < SKKF + S * KF; i += 64 * kQsroWaves) gtab[i] = A.G[i];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint8_t* box = boxes[wave];
    double* tm = term[wave];
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const int ncell = A.ncx * A.ncy * A.ncz;
    const int32_t* ox = A.org;
    const int32_t* oy = ox + A.ncx + 1;
    const int32_t* oz = oy + A.ncy + 1;
    constexpr int center = ((Rch * W + Rch) * W + Rch) * m;  // byte of basis site 0 of the active cell
    int att = 0, nacc = 0, ntie = 0;
    for (int c = blockIdx.x * kQsroWaves + wave; c < ncell; c += gridDim.x * kQsroWaves) {
        const int cx = c % A.ncx, cy = (c / A.ncx) % A.ncy, cz = c / (A.ncx * A.ncy);
        const int x0 = ld_const(ox, cx), x1 = ld_const(ox, cx + 1), y0 = ld_const(oy, cy), y1 = ld_const(oy, cy + 1),
                  z0 = ld_const(oz, cz), z1 = ld_const(oz, cz + 1);
        if (A.o0 >= x1 - x0 || A.o1 >= y1 - y0 || A.o2 >= z1 - z0) continue;
        const int x = x0 + A.o0, y = y0 + A.o1, z = z0 + A.o2;
        const int cell = x + A.L0 * (y + A.L1 * z);
        fence();  // the previous cell's trials are done with the box
        constexpr int NB = (W3 + 63) / 64;
        Cell st[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int i = lane + 64 * j;
            const int wx = i % W, wy = (i / W) % W, wz = i / (W * W);
            int xx = x + wx - Rch, yy = y + wy - Rch, zz = z + wz - Rch;
            xx += xx < 0 ? A.L0 : (xx >= A.L0 ? -A.L0 : 0);
            yy += yy < 0 ? A.L1 : (yy >= A.L1 ? -A.L1 : 0);
            zz += zz < 0 ? A.L2 : (zz >= A.L2 ? -A.L2 : 0);
            st[j] = 0;
            if (i < W3) st[j] = *(const Cell*)(A.occ + m * (xx + A.L0 * (yy + A.L1 * zz)));
        }
        // lane b draws for basis site b while the box is on its way
        const int db = lane % m;
        uint32_t w0, v1, v2, w3;
        philox4x32_10((uint32_t)(db + m * cell), 0u, A.sweep, A.replica, (uint32_t)A.seed, (uint32_t)(A.seed >> 32), w0, v1,
                      v2, w3);
        (void)w3;
        const int vk = (int)__umulhi(w0, (uint32_t)Z1), vn = A.nbr[db * A.sumZ + vk];
        int naffs[m], sites[m][NL];  // lanes past a list look at the active cell's first site
#pragma unroll
        for (int b = 0; b < m; ++b) {
            const int32_t* list = A.aff + (int64_t)(b * Z1 + __builtin_amdgcn_readlane(vk, b)) * (1 + A.naff_max);
            naffs[b] = ld_const(list, 0);
#pragma unroll
            for (int h = 0; h < NL; ++h) sites[b][h] = lane + 64 * h < naffs[b] ? list[1 + lane + 64 * h] : 0x080808;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (lane + 64 * j < W3) *(Cell*)(box + m * (lane + 64 * j)) = (Cell)(st[j] * (uint32_t)F);
        fence();
#pragma unroll
        for (int b = 0; b < m; ++b) {
            const uint32_t w1 = __builtin_amdgcn_readlane(v1, b), w2 = __builtin_amdgcn_readlane(v2, b);
            const int nd = __builtin_amdgcn_readlane(vn, b);  // partner's displacement
            const int dx = (nd & 0xff) - 8, dy = ((nd >> 8) & 0xff) - 8, dz = ((nd >> 16) & 0xff) - 8, bt = (nd >> 24) & 3;
            const int abyte = center + b, bbyte = center + dz * PL + dy * LP + dx * m + bt;
            const int pF = __builtin_amdgcn_readfirstlane(box[abyte]), qF = __builtin_amdgcn_readfirstlane(box[bbyte]);
            ++att;
            if (pF == qF) continue;
            const CT swap = ((CT)1 << qF) - ((CT)1 << pF);  // a neighbour of species p becomes q
            const int naff = naffs[b];
#pragma unroll
            for (int h = 0; h < NL; ++h) {
                if (64 * h >= naff) continue;
                const int d = sites[b][h], jb = (d >> 24) & 3;
                const int jbyte = center + (((d >> 16) & 0xff) - 8) * PL + (((d >> 8) & 0xff) - 8) * LP + ((d & 0xff) - 8) * m + jb;
                int base[m];
                base[0] = jbyte;
                if constexpr (LAT == SMCX_BCC) {
                    base[1] = jbyte + (jb ? m + LP + PL - 2 : 0);
                } else {
                    const int fx = jb == 1 || jb == 2 ? m : 0, fy = jb & 1 ? LP - 2 : 0, fz = jb & 2 ? PL - 4 : 0;
                    base[1] = jbyte + fx + fy;
                    base[2] = jbyte + fx + fz;
                    base[3] = jbyte + fy + fz;
                }
                const int own = box[jbyte];
                CT before[S], after[S];
                // shells of this site that hold the active site, the partner (0: none)
                const int sa = (d >> 26) & 7, sb = (int)((uint32_t)d >> 29);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    CT n = 0;
#pragma unroll
                    for (int i = 0; i < G.Z[s]; ++i) {
                        const Nb nb = nb_of(G, 0, G.v[s][i][0], G.v[s][i][1], G.v[s][i][2]);
                        const int off = nb.dz * PL + nb.dy * LP + nb.dx * m + nb.bt;
                        n = shl1_add(box[base[nb.bt] + off], n);
                    }
                    before[s] = n;
                    after[s] = n + (sa == s + 1 ? swap : (CT)0) - (sb == s + 1 ? swap : (CT)0);
                }
                const int sj = min(species_of(own, F), K - 1),
                          sj2 = min(species_of(jbyte == abyte ? qF : (jbyte == bbyte ? pF : own), F), K - 1);
                const double *gb = gtab + sj * KF, *ga = gtab + sj2 * KF;
                double eb = 0.0, ea = 0.0;
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int t = 0; t < KP; ++t)
                        if (t < K) {
                            eb = eb + gb[s * K * KF + t * kQsroFrac + (int)((before[s] >> (F * t)) & EN::mask)];
                            ea = ea + ga[s * K * KF + t * kQsroFrac + (int)((after[s] >> (F * t)) & EN::mask)];
                        }
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    eb = eb + gtab[SKKF + s * KF + sj * kQsroFrac + (int)((before[s] >> (F * sj)) & EN::mask)];
                    ea = ea + gtab[SKKF + s * KF + sj2 * kQsroFrac + (int)((after[s] >> (F * sj2)) & EN::mask)];
                }
                if (lane + 64 * h < naff) tm[lane + 64 * h] = ea - eb;
            }
            fence();
            const double dE = sum_in_order<1>(0.0, tm, naff);
            bool acc = true, tie = false;
            if (!(dE <= 0.0)) {
                const double P = exp(-(A.beta * dE));
                const double u = (double)(((uint64_t)w1 << 21) | (uint64_t)(w2 >> 11)) * 0x1p-53;
                acc = u < P;
                tie = fabs(u - P) < 1e-12;
            }
            if (lane == 0) {
                if (tie) {
                    const int slot = atomicAdd(A.tie_count, 1);
                    if (slot < A.tie_cap) {
                        smcx_tie e;
                        e.replica = (int32_t)A.replica;
                        e.sweep = A.sweep;
                        e.site = b + m * cell;
                        e.decision = acc ? 1 : 0;
                        e.pad = 0;
                        A.ties[slot] = e;
                    }
                }
                if (acc) {
                    box[abyte] = (uint8_t)qF;
                    box[bbyte] = (uint8_t)pF;
                    A.occ[b + m * cell] = (uint8_t)species_of(qF, F);
                    A.occ[qsro_site_of(A, x, y, z, nd, m)] = (uint8_t)species_of(pF, F);
                }
            }
            nacc += acc;
            ntie += tie;
            fence();  // the next trial sees the swap; the terms are free again
        }
    }
    if (lane == 0) {
        int64_t* slot = A.slots + 3 * (int64_t)(blockIdx.x * kQsroWaves + wave);
        slot[0] += att;
        slot[1] += nacc;
        slot[2] += ntie;
    }
}

// Sum the workgroups' counter slots into a replica's counters.
__global__ void k_qsro_reduce(const int64_t* slots, int n, int64_t* stats)
{
    int64_t v[3] = {0, 0, 0};
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        for (int c = 0; c < 3; ++c) v[c] += slots[3 * (int64_t)i + c];
    __shared__ int64_t red[3][kBlock];
    for (int c = 0; c < 3; ++c) red[c][threadIdx.x] = v[c];
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int c = 0; c < 3; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int c = 0; c < 3; ++c)
            if (red[c][0]) atomicAdd((unsigned long long*)(stats + c), (unsigned long long)red[c][0]);
}

hipError_t launch_qsro_reduce(const int64_t* slots, int n, int64_t* stats, hipStream_t st)
{
    hipLaunchKernelGGL(k_qsro_reduce, dim3(1), dim3(kBlock), 0, st, slots, n, stats);
    return hipGetLastError();
}

// The staged kernel where its box fits the lattice and cells are aligned.
bool qsro_staged(int lattice, const QsroArgs& A)
{
    const int m = lattice == SMCX_BCC ? 2 : 4, W = 2 * qsro_reach(lattice, A.S) + 1;
    return A.L0 >= W && A.L1 >= W && A.L2 >= W && ((uintptr_t)A.occ % m) == 0;
}

template <int LAT, int S>
static const void* qsro_cell_kernel(int K)
{
    return K <= 4   ? (const void*)k_qsro_cell<LAT, S, 1>
           : K == 5 ? (const void*)k_qsro_cell<LAT, S, 3>
                    : (const void*)k_qsro_cell<LAT, S, 2>;
}

template <int LAT>
static const void* qsro_cell_kernel_s(int S, int K)
{
    return S == 1   ? qsro_cell_kernel<LAT, 1>(K)
           : S == 2 ? qsro_cell_kernel<LAT, 2>(K)
           : S == 3 ? qsro_cell_kernel<LAT, 3>(K)
                    : qsro_cell_kernel<LAT, 4>(K);
}

hipError_t launch_qsro_offset(int lattice, const QsroArgs& A, int grid, hipStream_t st)
{
    const void* kern = lattice == SMCX_BCC ? qsro_cell_kernel_s<SMCX_BCC>(A.S, A.K) : qsro_cell_kernel_s<SMCX_FCC>(A.S, A.K);
    const size_t lds = sizeof(double) * qsro_products(A.K, A.S);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    QsroArgs copy = A;
    void* args[] = {&copy};
    return hipLaunchKernel(kern, dim3((unsigned)((grid + kQsroWaves - 1) / kQsroWaves)), dim3(64 * kQsroWaves), args, lds, st);
}

hipError_t launch_qsro_ministep(int lattice, const QsroArgs& A, int grid, hipStream_t st)
{
    if (lattice == SMCX_BCC) hipLaunchKernelGGL(k_qsro_ministep<SMCX_BCC>, dim3((unsigned)grid), dim3(64), 0, st, A);
    else hipLaunchKernelGGL(k_qsro_ministep<SMCX_FCC>, dim3((unsigned)grid), dim3(64), 0, st, A);
    return hipGetLastError();
}

}  // namespace smcx
