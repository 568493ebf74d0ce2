// Pair counts C[cfg][s][k][l] on the natural layout, 32 sites at a time.
//
// A configuration's species are held as bit planes along x: one word per 32
// cells of a row, basis site and species bit.  For a neighbour direction the
// neighbours of 32 sites are then two words of a neighbouring row shifted
// together, and the pairs of unlike species {k, l} among the 32 bonds are one
// or two logic operations and a population count.  Each site takes one
// direction of every +-d pair (the one with d_z > 0, then d_y, then d_x), so
// these are the undirected pairs U[k][l] = C[k][l] = C[l][k]; like pairs
// follow from the species counts, C[k][k] = Z_s N_k - sum_{l != k} U[k][l].
// All integer, exact.  (Pair numbers n_m^{pp'} of the EPI features, Methods
// "The EPI and qSRO model".)
//
// Against one LDS byte read and shift-add per neighbour, and a histogram per
// site: BCC 800^3 (4 species, 4 shells) 3.63 -> 0.79 ms, 64 x BCC 64^3 198 ->
// 41 us, 4096 x BCC 16^3 271 -> 78 us, FCC 128^3 (5 species) 80 -> 41 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "smcx_internal.h"
#include "smcx_launch.h"

namespace smcx {

namespace {

constexpr int kBitBlock = 512;  // the most threads of a workgroup (512 or 256)

// One direction of every +-d pair.
constexpr bool positive(const int (&v)[3]) { return v[2] > 0 || (v[2] == 0 && (v[1] > 0 || (v[1] == 0 && v[0] > 0))); }

constexpr int planes_of(int KT) { return KT <= 2 ? 1 : (KT <= 4 ? 2 : 3); }

struct BitTile {
    int L[3];
    int W;            // words of a row
    int tw, ty, tz;   // tile: words, rows and planes whose sites are counted
    int nw, ny, nz;   // tiles per axis
    int pitch;        // LDS words per row of cells (odd: rows of one word spread over the banks)
    int tiles;        // nw * ny * nz
};

__device__ __forceinline__ int wrap(int v, int L)
{
    v += v < 0 ? L : 0;
    v -= v >= L ? L : 0;
    return v >= 0 && v < L ? v : ((v % L) + L) % L;  // lattices narrower than the halo wrap twice
}

// v + population count of x (one instruction).
__device__ __forceinline__ uint32_t bcnt(uint32_t x, uint32_t v) { return (uint32_t)__popc(x) + v; }

// Sum over a wave, valid in lane 63.
__device__ __forceinline__ uint32_t wave_total(uint32_t v)
{
#define SMCX_DPP_ADD(ctrl, rm) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rm, 0xf, false)
    SMCX_DPP_ADD(0x111, 0xf);  // row_shr 1, 2, 4, 8: lane 15 of every row of 16
    SMCX_DPP_ADD(0x112, 0xf);
    SMCX_DPP_ADD(0x114, 0xf);
    SMCX_DPP_ADD(0x118, 0xf);
    SMCX_DPP_ADD(0x142, 0xa);  // row_bcast 15: rows 1 and 3 take the row before
    SMCX_DPP_ADD(0x143, 0xc);  // row_bcast 31: rows 2 and 3 take the lower half
#undef SMCX_DPP_ADD
    return v;
}

// The bit planes of up to 32 cells (n of them) from src (m bytes per cell):
// out[b][q] bit i = bit q of the species of cell i, basis b.  `over` gathers
// the high bits of every byte + (128 - K): non-zero there means a species
// that is not below K.
template <int m, int NP>
__device__ __forceinline__ void pack_bits(const uint8_t* src, int n, uint32_t addK, uint32_t (&out)[m][NP], uint32_t& over)
{
#pragma unroll
    for (int b = 0; b < m; ++b)
#pragma unroll
        for (int q = 0; q < NP; ++q) out[b][q] = 0;
    constexpr int CPC = 16 / m;  // cells per 16-byte chunk
#pragma unroll
    for (int c0 = 0; c0 < 32; c0 += CPC) {
        uint32_t d[4] = {0, 0, 0, 0};
        if (c0 + CPC <= n) {
            __builtin_memcpy(d, src + m * c0, 16);
        } else if (c0 < n) {
            for (int i = 0; i < m * (n - c0); ++i) {
                const uint32_t v = (uint32_t)src[m * c0 + i] << (8 * (i & 3));
#pragma unroll
                for (int w = 0; w < 4; ++w) d[w] |= (i >> 2) == w ? v : 0u;
            }
        } else {
            break;
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) over |= ((d[w] & 0x7f7f7f7fu) + addK) | d[w];
        if constexpr (m == 4) {
            // a word per cell: transpose to a word per basis site
            const uint32_t t0 = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u), t1 = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u);
            const uint32_t t2 = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u), t3 = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);
            d[0] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
            d[1] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
            d[2] = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
            d[3] = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int q = 0; q < NP; ++q)
                    out[b][q] |= __builtin_amdgcn_udot4((d[b] >> q) & 0x01010101u, 0x08040201u, 0u, false) << c0;
        } else {
            // a word holds two cells of both basis sites; 8 cells give 8 bits
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                uint32_t v[2] = {0, 0};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t bits = (d[w] >> q) & 0x01010101u;
                    v[0] = __builtin_amdgcn_udot4(bits, (1u << (2 * w)) | (2u << (2 * w)) << 16, v[0], false);
                    v[1] = __builtin_amdgcn_udot4(bits, (1u << (2 * w)) << 8 | (2u << (2 * w)) << 24, v[1], false);
                }
                out[0][q] |= v[0] << c0;
                out[1][q] |= v[1] << c0;
            }
        }
    }
}

// Undirected unlike pairs of 32 bonds: own species bits o, neighbours' n, own
// sites valid; U[pair(k, l)] for k < l, pairs in the order (0,1), (0,2), ...
template <int KT>
struct UnlikePairs {
    static constexpr int NP = planes_of(KT), NU = KT * (KT - 1) / 2;
    static constexpr int at(int k, int l) { return k * (2 * KT - k - 1) / 2 + (l - k - 1); }
    uint32_t M[KT];  // own species masks (KT > 4)

    __device__ __forceinline__ void own(const uint32_t (&o)[NP], uint32_t valid)
    {
        if constexpr (KT > 4) {
#pragma unroll
            for (int k = 0; k < KT; ++k)
                M[k] = (k & 1 ? o[0] : ~o[0]) & (k & 2 ? o[1] : ~o[1]) & (k & 4 ? o[2] : ~o[2]) & valid;
        }
    }

    // Pairs (k, l) from the totals of what add() counts (u[at(k, l)]).
    __device__ static __forceinline__ uint32_t finish(const uint32_t* u, int k, int l)
    {
        uint32_t v = u[at(k, l)];
        if constexpr (KT == 4) {
            if (l == 1) v -= u[at(2, 3)] + u[at(0, 3)] + u[at(1, 2)];
            if (k == 0 && l == 2) v -= u[at(1, 3)] + u[at(0, 3)] + u[at(1, 2)];
        }
        return v;
    }

    __device__ __forceinline__ void add(const uint32_t (&o)[NP], const uint32_t (&n)[NP], uint32_t valid,
                                        uint32_t (&U)[NU]) const
    {
        if constexpr (KT == 2) {
            U[0] = bcnt((o[0] ^ n[0]) & valid, U[0]);
        } else if constexpr (KT <= 4) {
            // A, B: low, high species bit differs; pairs (0,1), (2,3) differ in
            // the low bit only, (0,2), (1,3) in the high one, (0,3), (1,2) in
            // both.  Counted: A and B themselves, (0,3), (1,2), (2,3), (1,3);
            // finish() takes (0,1) and (0,2) from them.
            const uint32_t A = __builtin_amdgcn_bitop3_b32(o[0], n[0], valid, 0x28);  // (a ^ b) & c
            const uint32_t B = __builtin_amdgcn_bitop3_b32(o[1], n[1], valid, 0x28);
            const uint32_t X = o[0] ^ o[1];
            U[at(0, 1)] = bcnt(A, U[at(0, 1)]);
            U[at(0, 2)] = bcnt(B, U[at(0, 2)]);
            U[at(1, 2)] = bcnt(__builtin_amdgcn_bitop3_b32(A, B, X, 0x80), U[at(1, 2)]);  // a & b & c
            if constexpr (KT == 4) {
                U[at(2, 3)] = bcnt(__builtin_amdgcn_bitop3_b32(A, o[1], n[1], 0x80), U[at(2, 3)]);
                U[at(1, 3)] = bcnt(__builtin_amdgcn_bitop3_b32(B, o[0], n[0], 0x80), U[at(1, 3)]);
                U[at(0, 3)] = bcnt(__builtin_amdgcn_bitop3_b32(A, B, X, 0x40), U[at(0, 3)]);  // a & b & ~c
            }
        } else {
            uint32_t N[KT];
#pragma unroll
            for (int k = 0; k < KT; ++k) N[k] = (k & 1 ? n[0] : ~n[0]) & (k & 2 ? n[1] : ~n[1]) & (k & 4 ? n[2] : ~n[2]);
#pragma unroll
            for (int k = 0; k < KT; ++k)
#pragma unroll
                for (int l = k + 1; l < KT; ++l) {
                    const uint32_t t = M[l] & N[k];
                    U[at(k, l)] = bcnt(__builtin_amdgcn_bitop3_b32(M[k], N[l], t, 0xEA), U[at(k, l)]);  // (a & b) | c
                }
        }
    }
};

// The unlike pairs of one word of basis-b sites (b fixed at compile time, or
// uniform over the wave: the shifts and rows are scalars then).
template <int LAT, int KT>
__device__ __forceinline__ void count_word(const uint32_t* cur, int b, int rowy, int rowz, int wpp, int S, uint32_t valid,
                                           uint32_t (&U)[kMaxShells][UnlikePairs<KT>::NU], uint32_t (&N)[KT])
{
    constexpr Geometry G = kGeom[LAT];
    constexpr int NP = planes_of(KT);
    UnlikePairs<KT> P;
    uint32_t o[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) o[q] = cur[(b * NP + q) * wpp];
    P.own(o, valid);
    if constexpr (KT <= 4) {
        // N[1..3]: sites with the low bit, the high bit, both
        N[1] = bcnt(o[0] & valid, N[1]);
        if constexpr (KT > 2) {
            N[2] = bcnt(o[1] & valid, N[2]);
            N[0] = bcnt(o[0] & o[1] & valid, N[0]);
        }
    } else {
#pragma unroll
        for (int k = 1; k < KT; ++k) N[k] = bcnt(P.M[k], N[k]);
    }
    const int bx = G.m == 2 ? b : (b == 1 || b == 2), by = G.m == 2 ? b : b & 1, bz = G.m == 2 ? b : b >> 1;
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s) {
        if (s >= S) continue;
#pragma unroll
        for (int i = 0; i < G.Z[s]; ++i) {
            if (!positive(G.v[s][i])) continue;
            // an odd component carries into the next cell from an odd site
            const Nb nb = nb_of(G, 0, G.v[s][i][0], G.v[s][i][1], G.v[s][i][2]);
            const int dx = nb.dx + (G.v[s][i][0] & 1 & bx), dy = nb.dy + (G.v[s][i][1] & 1 & by),
                      dz = nb.dz + (G.v[s][i][2] & 1 & bz), bt = nb.bt ^ b;
            const uint32_t* row = cur + dz * rowz + dy * rowy + bt * NP * wpp + (dx < 0 ? -1 : 0);
            uint32_t n[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q) n[q] = __builtin_amdgcn_alignbit(row[q * wpp + 1], row[q * wpp], (uint32_t)(dx & 31));
            P.add(o, n, valid, U[s]);
        }
    }
}

// Tiles t0, t0 + step, ... of configuration blockIdx.y: rows y .. y + ty - 1
// of planes z .. z + tz - 1 (all of x, or tw words of it) with two halo rows
// on either side in y and two halo planes above.  Staging reads every byte of
// the tile and its halo once, 16 bytes at a time, and writes a word of bits
// per 32; a thread then counts the sites of one word of a row at a time.
// Bound by VALU issue: 14 operations per direction and 32 bonds of 4 species
// (38 for 5), 25 directions per BCC site.  `bad` (may be NULL) is set
// when a byte is not a species below K.
template <int LAT, int KT>
__global__ __launch_bounds__(kBitBlock) void k_pair_bits(const uint8_t* occ, int64_t Nsites, BitTile T, int K, int S,
                                                         int64_t* counts, volatile uint32_t* bad)
{
    constexpr Geometry G = kGeom[LAT];
    constexpr int m = G.m, NP = planes_of(KT), NU = UnlikePairs<KT>::NU;
    extern __shared__ __align__(16) uint32_t bits[];
    const uint8_t* o = occ + (int64_t)blockIdx.y * Nsites;
    const int L0 = T.L[0], L1 = T.L[1], L2 = T.L[2];
    const int RY = T.ty + 4, wpp = T.tw + 2;  // rows per staged plane; words per basis site and species bit
    const int blk = blockDim.x;
    const bool split = T.nw > 1;
    const int wps = split ? wpp : T.tw;  // words staged per row
    const uint32_t addK = (uint32_t)(128 - K) * 0x01010101u;
    uint32_t U[kMaxShells][NU], N[KT];
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s)
#pragma unroll
        for (int u = 0; u < NU; ++u) U[s][u] = 0;
#pragma unroll
    for (int k = 0; k < KT; ++k) N[k] = 0;
    uint32_t over = 0;
    for (int t = blockIdx.x; t < T.tiles; t += gridDim.x) {
        const int tz = t / (T.nw * T.ny), tr = t - tz * (T.nw * T.ny), ty = tr / T.nw, tx = tr - ty * T.nw;
        const int z0 = tz * T.tz, y0 = ty * T.ty, w0 = tx * T.tw;
        const int nz = min(T.tz, L2 - z0), ny = min(T.ty, L1 - y0), nw = min(T.tw, T.W - w0);
        __syncthreads();  // the previous tile is counted
        const int nst = (nz + 2) * (ny + 4) * wps;
        for (int i = threadIdx.x; i < nst; i += blk) {
            const int w = i % wps, rr = i / wps, ry = rr % (ny + 4), rz = rr / (ny + 4);
            const int y = wrap(y0 + ry - 2, L1), z = wrap(z0 + rz, L2);
            const uint8_t* row = o + (int64_t)m * L0 * (y + (int64_t)L1 * z);
            uint32_t* dst = bits + (rz * RY + ry) * T.pitch;
            const int g = w0 + w - (split ? 1 : 0);  // word of the row; -1 and W: periodic images
            // bits x = 0, 1 and x = L0 - 2, L0 - 1 of every basis site and plane
            auto edge = [&](int x, int b, int q) {
                const uint8_t* c = row + (int64_t)m * x + b;
                return (((uint32_t)c[0] >> q) & 1u) | (((uint32_t)c[m] >> q) & 1u) << 1;
            };
            const int slot = split ? w : w + 1;
            if (g >= 0 && g < T.W) {
                const int n = min(32, L0 - 32 * g);
                uint32_t v[m][NP];
                pack_bits<m, NP>(row + (int64_t)m * 32 * g, n, addK, v, over);
                const bool last = g == T.W - 1, wrapl = !split && g == 0, wrapr = !split && last;
#pragma unroll
                for (int b = 0; b < m; ++b)
#pragma unroll
                    for (int q = 0; q < NP; ++q) {
                        uint32_t* d = dst + (b * NP + q) * wpp + slot;
                        uint64_t x = v[b][q];
                        if (last) x |= (uint64_t)edge(0, b, q) << n;  // the row goes on with its first cells
                        d[0] = (uint32_t)x;
                        if (wrapr) d[1] = (uint32_t)(x >> 32);
                        if (wrapl) d[-1] = edge(L0 - 2, b, q) << 30;
                    }
            } else if (g == -1 || g == T.W) {
                const int r = L0 - 32 * (T.W - 1);
#pragma unroll
                for (int b = 0; b < m; ++b)
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        dst[(b * NP + q) * wpp + slot] =
                            g < 0 ? edge(L0 - 2, b, q) << 30 : (uint32_t)(((uint64_t)edge(0, b, q) << r) >> 32);
            }
        }
        __syncthreads();
        const int items = nz * ny * nw;
        for (int i = threadIdx.x; i < items; i += blk) {
            const int w = i % nw, rr = i / nw, ry = rr % ny, rz = rr / ny;
            const int left = L0 - 32 * (w0 + w);
            const uint32_t valid = left >= 32 ? 0xFFFFFFFFu : (1u << left) - 1u;
            const uint32_t* cur = bits + (rz * RY + ry + 2) * T.pitch + w + 1;
            if constexpr (KT <= 4) {
#pragma unroll
                for (int b = 0; b < m; ++b) count_word<LAT, KT>(cur, b, T.pitch, RY * T.pitch, wpp, S, valid, U, N);
            } else {
#pragma unroll 1
                for (int b = 0; b < m; ++b) count_word<LAT, KT>(cur, b, T.pitch, RY * T.pitch, wpp, S, valid, U, N);
            }
        }
    }
    // wave sums into LDS, totals, one atomic per directed count
    __syncthreads();
    constexpr int NV = kMaxShells * NU + KT;
    const int NWV = blk / 64;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int s = 0; s < kMaxShells; ++s)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t v = wave_total(U[s][u]);
            if (lane == 63) bits[wave * NV + s * NU + u] = v;
        }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const uint32_t v = wave_total(N[k]);
        if (lane == 63) bits[wave * NV + kMaxShells * NU + k] = v;
    }
    if (bad && __ballot((over & 0x80808080u) != 0) && lane == 0) *bad = 1;
    __syncthreads();
    uint32_t* tot = bits + NWV * NV;
    for (int i = threadIdx.x; i < NV; i += blk) {
        uint32_t v = 0;
        for (int w = 0; w < NWV; ++w) v += bits[w * NV + i];
        tot[i] = v;
    }
    __syncthreads();
    // sites counted by this workgroup
    uint32_t sites = 0;
    for (int t = blockIdx.x; t < T.tiles; t += gridDim.x) {
        const int tz = t / (T.nw * T.ny), tr = t - tz * (T.nw * T.ny), ty = tr / T.nw, tx = tr - ty * T.nw;
        sites += (uint32_t)(m * min(32 * T.tw, L0 - 32 * tx * T.tw) * min(T.ty, L1 - ty * T.ty) * min(T.tz, L2 - tz * T.tz));
    }
    const uint32_t* n = tot + kMaxShells * NU;
    for (int i = threadIdx.x; i < S * K * K; i += blk) {
        const int s = i / (K * K), k = (i / K) % K, l = i % K;
        uint32_t c;
        auto pair = [&](int a, int b) { return UnlikePairs<KT>::finish(tot + s * NU, min(a, b), max(a, b)); };
        if (k != l) {
            c = pair(k, l);
        } else {
            uint32_t nk;
            if constexpr (KT <= 4) {
                // from the counts of the low bit, the high bit and both
                const uint32_t n1 = n[1], n2 = KT > 2 ? n[2] : 0u, n3 = KT > 2 ? n[0] : 0u;
                nk = k == 0 ? sites - n1 - n2 + n3 : (k == 1 ? n1 - n3 : (k == 2 ? n2 - n3 : n3));
            } else {
                nk = sites;
                for (int j = 1; j < KT; ++j) nk -= n[j];
                if (k > 0) nk = n[k];
            }
            c = (uint32_t)G.Z[s] * nk;
            for (int j = 0; j < K; ++j)
                if (j != k) c -= pair(k, j);
        }
        // like pairs of one workgroup's sites may come out negative (its bonds
        // reach into other workgroups' sites): only their sum is a count
        if (c) atomicAdd((unsigned long long*)&counts[(int64_t)blockIdx.y * S * K * K + i], (unsigned long long)(int64_t)(int32_t)c);
    }
}

}  // namespace

hipError_t launch_pair_counts(int lattice, int K, int S, const uint8_t* occ, int64_t N, const int32_t* L, int B,
                              int64_t* counts, volatile uint32_t* bad, hipStream_t st)
{
    if (B > 65535) return hipErrorInvalidValue;
    const int m = lattice == SMCX_BCC ? 2 : 4;
    const int KT = K <= 2 ? 2 : (K <= 4 ? 4 : (K <= 5 ? 5 : (K <= 6 ? 6 : 8)));
    const int NP = planes_of(KT);
    BitTile T{};
    for (int a = 0; a < 3; ++a) T.L[a] = L[a];
    T.W = (int)(((int64_t)L[0] + 31) / 32);
    // Rows whole, unless 5 x 3 of them pass the LDS budget (two or more
    // workgroups per CU), then in pieces of 64 words.
    const int budget = 20000;  // words
    auto pitch_of = [&](int64_t tw) { return (m * NP * (tw + 2)) | 1; };
    T.tw = pitch_of(T.W) * 15 <= budget ? T.W : std::min(T.W, 64);
    T.pitch = (int)pitch_of(T.tw);
    T.nw = (T.W + T.tw - 1) / T.tw;
    // Tile of rows x planes: the smallest cost of a pass over the lattice,
    // staging (about 60 operations per word and basis site) and counting
    // (about 400 per word and basis site, in rounds of the workgroup's
    // threads), where fewer than 768 tiles in the batch cost as much as 768.
    double best = 1e300;
    T.ty = T.tz = 1;
    auto parts = [](int64_t n, int64_t d) { return (n + d - 1) / d; };  // 64 bits: an axis may pass 2^30 cells
    for (int64_t ny = 1; ny <= L[1]; ny = ny < 8 ? ny + 1 : ny + (ny + 3) / 4) {
        const int64_t ty = parts(L[1], ny);
        for (int64_t nz = 1; nz <= L[2]; nz = nz < 8 ? nz + 1 : nz + (nz + 3) / 4) {
            const int64_t tz = parts(L[2], nz);
            if ((ty + 4) * (tz + 2) * T.pitch > budget) continue;
            const int64_t items = ty * tz * T.tw, staged = (ty + 4) * (tz + 2) * T.tw;
            const double rounds = (double)parts(items, 256) * 400.0 + (double)parts(staged, 256) * 60.0 + 150.0;
            const double tiles = (double)T.nw * parts(L[1], ty) * parts(L[2], tz) * B;
            const double cost = rounds * std::max(tiles, 768.0);
            if (cost < best) {
                best = cost;
                T.ty = (int)ty;
                T.tz = (int)tz;
            }
        }
    }
    T.ny = (int)parts(L[1], T.ty);
    T.nz = (int)parts(L[2], T.tz);
    const int64_t tiles = (int64_t)T.nw * T.ny * T.nz;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    T.tiles = (int)tiles;
    // up to about 1536 workgroups for the batch, each over several tiles; a
    // workgroup's signed 32-bit counts hold 2^31 / 24 sites
    int64_t gx = std::max<int64_t>(1, std::min<int64_t>(tiles, 1536 / B));
    gx = std::max(gx, std::min<int64_t>(tiles, N / (1 << 26) + 1));
    const int NU = KT * (KT - 1) / 2, NV = kMaxShells * NU + KT;
    // Large tiles leave two workgroups per CU: eight waves each where their
    // registers allow it (up to 4 species: BCC 800^3 1104 -> 845 us with the call,
    // FCC 400^3 319 -> 254; 5 species, BCC 500^3: 514 -> 574)
    const int threads = KT <= 4 && T.ty * T.tz * T.tw >= 1024 ? 512 : 256;
    const size_t lds = 4 * (size_t)std::max((T.ty + 4) * (T.tz + 2) * T.pitch, (threads / 64 + 1) * NV);
    const dim3 g((unsigned)gx, (unsigned)B), blk((unsigned)threads);
    auto go = [&](const void* kern) {
        (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        void* args[] = {(void*)&occ, (void*)&N, (void*)&T, (void*)&K, (void*)&S, (void*)&counts, (void*)&bad};
        return hipLaunchKernel(kern, g, blk, args, lds, st);
    };
    auto pick = [&](auto lat) -> const void* {
        constexpr int LAT = decltype(lat)::value;
        return KT == 2   ? (const void*)k_pair_bits<LAT, 2>
               : KT == 4 ? (const void*)k_pair_bits<LAT, 4>
               : KT == 5 ? (const void*)k_pair_bits<LAT, 5>
               : KT == 6 ? (const void*)k_pair_bits<LAT, 6>
                         : (const void*)k_pair_bits<LAT, 8>;
    };
    const hipError_t e = go(lattice == SMCX_BCC ? pick(std::integral_constant<int, SMCX_BCC>{})
                                                : pick(std::integral_constant<int, SMCX_FCC>{}));
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace smcx
