// Device code shared by the kernel files: random numbers, packed counters,
// table and window loads, the acceptance test, trial statistics and the row
// kernels' write-back.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smcx_internal.h"

namespace smcx {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  Ten rounds of the
// 4-word S-box: two 32x32->64 products of words 0 and 2 with the multipliers,
// high halves xored with words 1/3 and the round key, low halves kept; the
// key advances by the Weyl increments between rounds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t& o0,
                                              uint32_t& o1, uint32_t& o2, uint32_t& o3)
{
    // the key is wave-uniform: keep it in scalar registers and let the round
    // keys be formed here, not hoisted out of the trial loops as 20 live SGPRs
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        // round 0: words 1 and 3 are often wave-uniform, so their xor with
        // the key is left to scalar code; later rounds take one three-input
        // xor (truth table 0x96) instead of two xors
        const uint32_t n0 = r == 0 ? (uint32_t)(p1 >> 32) ^ (c1 ^ k0)
                                   : __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = r == 0 ? (uint32_t)(p0 >> 32) ^ (c3 ^ k1)
                                   : __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    o0 = c0; o1 = c1; o2 = c2; o3 = c3;
}

// Packed per-shell neighbour counters: F bits per species, one field per
// species, biased by `half` when two counters are subtracted so that every
// field of (n_a + bias - n_b) stays in [half - 24, half + 24] (a shell has at
// most 24 sites) and no borrow crosses fields.  Encoding 1: K <= 4, 8-bit
// fields in 32 bits; 3: K = 5, 6-bit fields in 32 bits; 4: K = 6, the same
// with two bits left for species 5, whose difference follows from the others
// (a shell's differences sum to zero); 2: K <= 8, 8-bit fields in 64 bits.
// The padded copy and the LDS window hold F * species.
// KP: species held, KT: those with a term of their own in the integer screen.
template <int E> struct Enc;
template <> struct Enc<1> {
    using T = uint32_t;
    static constexpr int F = 8, KP = 4, KT = 3, half = 128;
    static constexpr uint32_t bias = 0x80808080u, mask = 0xFF;
};
template <> struct Enc<3> {
    using T = uint32_t;
    static constexpr int F = 6, KP = 5, KT = 4, half = 32;
    static constexpr uint32_t bias = 32u | 32u << 6 | 32u << 12 | 32u << 18 | 32u << 24, mask = 0x3F;
};
template <> struct Enc<4> {
    using T = uint32_t;
    static constexpr int F = 6, KP = 6, KT = 5, half = 32;
    static constexpr uint32_t bias = Enc<3>::bias, mask = 0x3F;
};
template <> struct Enc<2> {
    using T = uint64_t;
    static constexpr int F = 8, KP = 8, KT = 7, half = 128;
    static constexpr uint64_t bias = 0x8080808080808080ull, mask = 0xFF;
};

// species from its stored form F * species (F = 8 or 6, species < 64)
__device__ __forceinline__ int species_of(int v, int F) { return F == 8 ? v >> 3 : (v * 43) >> 8; }

// acc + (1 << sh) in one instruction (v_lshl_add): the packed counter gains
// one in the 8-bit field of the neighbour's species (sh = 8 * species).
__device__ __forceinline__ uint32_t shl1_add(uint32_t sh, uint32_t acc)
{
    uint32_t r;
    asm("v_lshl_add_u32 %0, 1, %1, %2" : "=v"(r) : "v"(sh), "v"(acc));
    return r;
}

__device__ __forceinline__ uint64_t shl1_add(uint32_t sh, uint64_t acc) { return acc + ((uint64_t)1 << sh); }

// Four of them in one asm block: the compiler pads every inline asm that
// writes a VGPR with a wait state, so a block per neighbour cost one per add.
__device__ __forceinline__ uint32_t shl1_add4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t acc)
{
    uint32_t r;
    asm("v_lshl_add_u32 %0, 1, %1, %5\n\t"
        "v_lshl_add_u32 %0, 1, %2, %0\n\t"
        "v_lshl_add_u32 %0, 1, %3, %0\n\t"
        "v_lshl_add_u32 %0, 1, %4, %0"
        : "=&v"(r)
        : "v"(a), "v"(b), "v"(c), "v"(d), "v"(acc));
    return r;
}
__device__ __forceinline__ uint64_t shl1_add4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint64_t acc)
{
    return shl1_add(d, shl1_add(c, shl1_add(b, shl1_add(a, acc))));
}
__device__ __forceinline__ uint32_t shl1_add2(uint32_t a, uint32_t b, uint32_t acc)
{
    uint32_t r;
    asm("v_lshl_add_u32 %0, 1, %1, %3\n\t"
        "v_lshl_add_u32 %0, 1, %2, %0"
        : "=&v"(r)
        : "v"(a), "v"(b), "v"(acc));
    return r;
}
__device__ __forceinline__ uint64_t shl1_add2(uint32_t a, uint32_t b, uint64_t acc) { return shl1_add(b, shl1_add(a, acc)); }

struct Lds {
    const int32_t* Q;  // integer dE terms and their bias sum, a row per species pair
    float qscale;      // value of one integer unit (a power of two)
    float qeps;        // bound on |integer dE - binary64 dE| before the float conversion
    const int32_t* offB;
    const int8_t* pd;
};

__device__ __forceinline__ Lds lds_ptrs(const SweepArgs& A, uint8_t* smem)
{
    Lds l;
    l.Q = (const int32_t*)smem;
    // read at run time, like the tables, so that a captured graph follows smcx_set_epi
    using CI = const __attribute__((address_space(4))) int32_t;
    const int nq = qtab_entries(A.K, A.S);
    l.qscale = __int_as_float(((CI*)A.Qtab)[nq]);
    l.qeps = __int_as_float(((CI*)A.Qtab)[nq + 1]);
    l.offB = (const int32_t*)(smem + A.lds_offb);
    l.pd = (const int8_t*)(smem + A.lds_pd);
    return l;
}

// Copy the launch tables into LDS (a barrier follows before first use).
template <int LAT>
__device__ void load_tables(const SweepArgs& A, uint8_t* smem)
{
    constexpr int m = kGeom[LAT].m;
    int32_t* Q = (int32_t*)smem;
    const int nQ = qtab_entries(A.K, A.S);
    for (int i = threadIdx.x; i < nQ; i += blockDim.x) Q[i] = A.Qtab[i];
    int32_t* Bo = (int32_t*)(smem + A.lds_offb);
    int8_t* pd = (int8_t*)(smem + A.lds_pd);
    for (int i = threadIdx.x; i < m * A.Z1; i += blockDim.x) Bo[i] = A.offB[i];
    for (int i = threadIdx.x; i < 4 * m * A.Z1; i += blockDim.x) pd[i] = A.pdisp[i];
}

// ---------------------------------------------------------------------------
// Window geometry policies.  GeoRt reads tile shape and window pitches from
// the launch arguments (any partition); GeoFix<...> fixes them at compile
// time for uniform partitions, so that every LDS neighbour offset is an
// immediate and cell origins are c * ELL.
// ---------------------------------------------------------------------------
struct GeoRt {
    static constexpr bool fixed = false;
    static constexpr bool rows = false;
    static constexpr bool own_cp = false;
    static constexpr bool may_alias = true;  // a partner may have images in other shells (an edge of 2)
    static constexpr int ELL = 0;
    __device__ static int T(const SweepArgs& A, int a) { return A.T[a]; }
    __device__ static int LP(const SweepArgs& A) { return A.LP; }
    __device__ static int WY(const SweepArgs& A) { return A.WY; }
    __device__ static int WZ(const SweepArgs& A) { return A.WZ; }
    __device__ static int block(const SweepArgs&) { return blockDim.x; }
    __device__ static int K(const SweepArgs& A) { return A.K; }
    __device__ static int S(const SweepArgs& A) { return A.S; }
    __device__ static int CP(const RepDev& rep) { return rep.cp; }
};

// Row windows: the window holds whole padded x-rows (periodic images of the
// sites within two cells of the x faces included), so a written site must be
// copied to its image in the window too.  NS fixes the shell count at compile
// time (0: taken from the launch).
template <int NS>
struct GeoRow : GeoRt {
    static constexpr bool rows = true;
    static constexpr bool own_cp = true;  // replicas may differ in column pitch
    __device__ static int S(const SweepArgs& A) { return NS ? NS : A.S; }
};

struct TileGeom {
    int w0[3];   // window origin (replica conventional cells, >= -H)
    int n[3];    // window extent
    int gx0;     // first staged byte of each padded row
    int c0[3];   // first link cell of the tile
    int c1[3];   // one past the last link cell
};

template <class Geo>
__device__ __forceinline__ int cell_origin(const SweepArgs& A, const RepDev& rep, int a, int c)
{
    if constexpr (Geo::fixed) {
        return c * Geo::ELL;
    } else {
        const int32_t* org = A.origins + rep.cs_off;
        if (a > 0) org += rep.nc[0] + 1;
        if (a > 1) org += rep.nc[1] + 1;
        return org[c];
    }
}

// Issue the window loads of a tile straight into LDS (global_load_lds_dwordx4:
// lane i of a wave writes the 16 bytes at M0 + 16 i).  Window row R (plane
// R / WY, row R % WY) occupies LP bytes at buf + R LP.  Long rows go a wave
// per row (R = wave, wave + waves, ...): the row's source address is
// wave-uniform and a lane's part of it 16 bytes per chunk.  Short rows would
// leave most lanes of such a wave idle, so there window slot j (16 bytes at
// buf + 16 j: row j / (LP / 16), chunk j % (LP / 16)) goes to thread j, j +
// block, ..., each advancing its source address by fixed steps.  Blocks are
// whole waves.  The loads complete asynchronously; the caller waits on vmcnt
// and a barrier before reading the buffer.
template <int LAT, class Geo>
__device__ __forceinline__ void stage_async(const SweepArgs& A, const RepDev& rep, const TileGeom& tg,
                                            const uint8_t* pad, uint8_t* buf)
{
    constexpr int m = kGeom[LAT].m;
    const int LP = Geo::LP(A), LPc = LP >> 4;
    const int WY = Geo::WY(A);
    const int nrows = Geo::WZ(A) * WY;
    // row windows hold whole basis-planar rows; tile windows a byte range of
    // interleaved rows
    const int grow = Geo::rows ? rep.prowp : rep.prow;
    const int gx1 = Geo::rows ? rep.prowp : (m * (tg.w0[0] + tg.n[0] + kHalo) + 15) & ~15;
    const int n16 = min((gx1 - tg.gx0) >> 4, LPc);  // chunks of a row, never past the window's pitch
    // the window geometry is the same in every lane: scalar registers keep
    // the loops and the row addresses out of vector code
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int block = __builtin_amdgcn_readfirstlane(Geo::block(A));
    const int n1 = __builtin_amdgcn_readfirstlane(tg.n[1]), n2 = __builtin_amdgcn_readfirstlane(tg.n[2]);
    const uint64_t off = (uint64_t)(((int64_t)(tg.w0[2] + kHalo) * rep.prows + (tg.w0[1] + kHalo)) * grow + tg.gx0);
    // (the builtin returns a signed word: its sign must not reach the upper one)
    const uint8_t* base = pad + (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(off >> 32)) << 32 |
                                          (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)off));
    const int64_t plane = (int64_t)rep.prows * grow;
    if (n16 >= 40) {
        const int nwaves = block >> 6;
        int wz = wave / WY, wy = wave - wz * WY;
        for (int R = wave; R < nrows; R += nwaves) {
            if (wy < n1 && wz < n2) {
                const uint8_t* row = base + wz * plane + (int64_t)wy * grow;
                for (int cb = 0; cb < n16; cb += 64)
                    if (cb + lane < n16)
                        __builtin_amdgcn_global_load_lds(
                            (const __attribute__((address_space(1))) void*)(row + 16 * (cb + lane)),
                            (__attribute__((address_space(3))) void*)(buf + R * LP + 16 * cb), 16, 0, 0);
            }
            wy += nwaves;
            while (wy >= WY) {
                wy -= WY;
                ++wz;
            }
        }
        return;
    }
    const int nslots = nrows * LPc;
    int j = wave * 64 + lane;
    int R = j / LPc, col = j - R * LPc;
    int wz = R / WY, wy = R - wz * WY;
    const int dR = block / LPc, dcol = block - dR * LPc;
    const uint8_t* src = base + wz * plane + (int64_t)wy * grow + 16 * col;
    const int64_t step = (int64_t)dR * grow + 16 * dcol, wrap_col = grow - 16 * LPc, wrap_row = plane - (int64_t)WY * grow;
    for (int jb = wave * 64; jb < nslots; jb += block) {
        if (jb + lane < nslots && col < n16 && wy < n1 && wz < n2)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(buf + 16 * jb), 16, 0, 0);
        col += dcol;
        wy += dR;
        src += step;
        if (col >= LPc) {
            col -= LPc;
            ++wy;
            src += wrap_col;
        }
        while (wy >= WY) {
            wy -= WY;
            ++wz;
            src += wrap_row;
        }
    }
}

// The decision of a trial the integer screen leaves open (a few in 1e5 at
// the benchmark's temperature): dE summed in binary64, s and t ascending, from
// D[s][t][p][q] (pq: the lane's (p, q) entry), then the float screen
// and, where that cannot decide either, exp in binary64, the test u < P and
// the near-tie check.  The sum starts from the first product rather than from
// +0.0 + it: the two differ only in the sign of a zero sum, and dE <= 0
// accepts either.  Out of line: inlined, its registers would weigh on every
// trial's code.  Returns bit 0: accepted, bit 1: near-tie.
template <int E>
__device__ __noinline__ int decide_binary64(const double* Dtab, int pq, typename Enc<E>::T d0, typename Enc<E>::T d1,
                                            typename Enc<E>::T d2, typename Enc<E>::T d3, int K, int S, double beta,
                                            uint32_t w1, uint32_t w2)
{
    using EN = Enc<E>;
    using CT = typename EN::T;
    // Three or four terms are read together (one by one, each waited for: up to 10 % more
    // for a whole sweep of a tensor with many a dE of zero; more at a time would
    // take registers that every caller has to keep free).  One table for all
    // lanes: a scalar base and 32-bit offsets.
    using CD = const __attribute__((address_space(1))) double;
    using CB = const __attribute__((address_space(1))) uint8_t;
    const uint64_t base = (uint64_t)Dtab;
    CB* D = (CB*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32 |
                  (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base));
    constexpr int U = EN::KP == 5 || EN::KP == 6 ? 3 : 4;
    const uint32_t step = 8u * (uint32_t)(K * K);
    uint32_t at = 8u * (uint32_t)pq;
    double dE = 0.0;
    for (int s = 0, s_end = __builtin_amdgcn_readfirstlane(S); s < s_end; ++s) {
        CT f = d0;
        d0 = d1;
        d1 = d2;
        d2 = d3;
        int rest = 0;
#pragma unroll 1
        for (int t0 = 0; t0 < EN::KP; t0 += U) {
            double v[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                v[j] = *(CD*)(D + at);
                at += t0 + j < K - 1 ? step : 0u;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int tt = t0 + j;
                // a species whose field has no room for it is what the others leave
                const bool whole = EN::F * EN::KP <= 8 * (int)sizeof(CT) || tt < EN::KP - 1;
                const int c = whole ? (int)(f & EN::mask) - EN::half : -rest;
                rest += c;
                f >>= EN::F;
                if (tt < K) {
                    const double term = (double)c * v[j];
                    dE = s == 0 && tt == 0 ? term : dE + term;
                }
            }
        }
        at += step;
    }
    if (dE <= 0.0) return 1;
    const double x = beta * dE;
    // A float estimate settles u < exp(-x) whenever u lies farther from it
    // than the estimate's error: the binary64 test then gives the same answer
    // and the trial is no near-tie.  For x <= 30, rounding x and x log2(e) to
    // float moves the exponent by < 8e-6, so exp2 is off by < 6e-6 relative
    // (plus an ulp or two of v_exp_f32); the margin is 1e-4 relative plus
    // 1e-9 for u's truncation and rounding.
    if (x > 30.0) {
        if (w1 != 0) return 0;
    } else {
        const float uf = (float)w1 * 0x1p-32f;
        const float Pf = __builtin_amdgcn_exp2f((float)x * -1.44269504f);
        if (fabsf(uf - Pf) > 1e-4f * Pf + 1e-9f) return uf < Pf ? 1 : 0;
    }
    const double P = exp(-x);
    const double u = (double)(((uint64_t)w1 << 21) | (uint64_t)(w2 >> 11)) * 0x1p-53;
    return (u < P ? 1 : 0) | (fabs(u - P) < 1e-12 ? 2 : 0);
}

// The decision of a trial from the integer screen's sum qacc (exact sum of
// c_t Q in units of qscale, see trial_finish), where the screen's uncertainty
// qeps cannot change it (`settled`; such a trial is no near-tie).  Straight
// line: one divergent branch less per outcome.
//  e <= -eps: dE <= e + eps <= 0, accepted.
//  e > eps: dE > 0 and beta dE lies in [bf (e - eps), bf (e + eps)] up to float
// rounding.  u = (w1 2^21 + (w2 >> 11)) 2^-53 lies in [w1 2^-32, (w1 + 1)
// 2^-32).  With y = bf eps <= 1/4, exp(-beta dE) is within a factor exp(+-y)
// (<= 1.14 y relative) of exp(-bf e), and the float estimate of that is within
// 2e-5 relative for beta dE <= 31, so a margin of 1e-4 + 1.2 y relative plus
// 1e-9 for u's truncation settles u < exp(-beta dE) exactly.  Beyond
// beta dE = 30, exp(-beta dE) < 1e-13 while u >= 2^-32 unless w1 == 0.
__device__ __forceinline__ int screen(uint32_t qacc, float qscale, float qeps, double beta, uint32_t w1, bool& settled)
{
    const float e = (float)(int32_t)qacc * qscale;
    const float eps = qeps + fabsf(e) * 0x1p-22f;
    const float bf = (float)beta;
    const bool down = e <= -eps;
    const bool up = (e > eps) & (bf >= 0.0f) & (bf * eps < 0.25f);
    const bool far = bf * (e - eps) * (1.0f - 0x1p-20f) > 30.0f;
    const float uf = (float)w1 * 0x1p-32f;
    const float Pf = __builtin_amdgcn_exp2f(bf * e * -1.44269504f);
    const bool apart = fabsf(uf - Pf) > (1e-4f + 1.2f * bf * eps) * Pf + 1e-9f;
    settled = down | (up & (far ? w1 != 0 : apart));
    return (down | (up & !far & (uf < Pf))) ? 1 : 0;
}

// The same for the trials the float screen leaves open (about 1 in 2e4 at the
// benchmark's temperature, more for few shells, where two sites often have the
// same neighbours), before the sum in binary64 with its table reads is called
// for.  No neighbour count differs (`same`): dE is a zero, accepted.  Else
// x = beta e log2(e) in binary64, exp2 of its fraction in float: relative
// error below 3e-7 (the fraction's rounding, v_exp_f32's ulp, u's rounding),
// so a margin of 1e-6 + 1.2 beta eps relative plus 1e-9 for u's truncation
// settles u < exp(-beta dE) as above.
__device__ __forceinline__ int screen_fine(uint32_t qacc, float qscale, float qeps, double beta, uint32_t w1, bool same,
                                           bool& settled)
{
    const double e = (double)(int32_t)qacc * (double)qscale;  // exact: a 32-bit integer times a power of two
    const double eps = (double)qeps, y = beta * eps;
    settled = same | (e <= -eps);
    if (settled) return 1;
    const double x = beta * e * 1.4426950408889634, n = rint(x);
    if (!(e > eps && y >= 0.0 && y < 0.25 && x < 100.0)) return 0;
    const float P = ldexpf(__builtin_amdgcn_exp2f((float)(n - x)), -(int)n);
    const float uf = (float)w1 * 0x1p-32f;
    settled = fabsf(uf - P) > (1e-6f + 1.2f * (float)y) * P + 1e-9f;
    return uf < P ? 1 : 0;
}

// The species pair (p, q) of a trial from their stored forms: F (p K + q).
// Species were checked < K at init; the clamp keeps table reads in bounds
// regardless.
template <int E>
__device__ __forceinline__ int species_pair(int p8, int q8, int K)
{
    return min(__mul24(p8, K) + q8, __mul24(Enc<E>::F, K * K - 1));
}

// Its row of the integer dE table.
template <int E>
__device__ __forceinline__ const int32_t* qtab_row(const int32_t* Q, int pair, int S)
{
    using EN = Enc<E>;
    static_assert(EN::F == field_bits_of(EN::KP), "field width");
    return (const int32_t*)((const uint8_t*)Q + __mul24(pair, 4 * qtab_pitch(EN::KP, S) / EN::F));
}

// The decision of a trial of species pair `pair`: the screens, or
// decide_binary64 from the biased count differences d0 .. d3.  Returns bit 0: accepted, bit 1: near-tie.
template <int E>
__device__ __forceinline__ int metropolis(uint32_t qacc, float qscale, float qeps, const double* D, int pair,
                                          typename Enc<E>::T d0, typename Enc<E>::T d1, typename Enc<E>::T d2,
                                          typename Enc<E>::T d3, int K, int S, double beta, uint32_t w1, uint32_t w2)
{
    bool settled;
    int f = screen(qacc, qscale, qeps, beta, w1, settled);
    if (!settled) {
        constexpr typename Enc<E>::T z = Enc<E>::bias;
        // (a sum that is not zero all the same marks a tensor that the screen must
        // not judge: it may hold infinities, and 0 times one is no zero)
        const bool same = ((d0 ^ z) | (S > 1 ? d1 ^ z : 0) | (S > 2 ? d2 ^ z : 0) | (S > 3 ? d3 ^ z : 0) | qacc) == 0;
        f = screen_fine(qacc, qscale, qeps, beta, w1, same, settled);
        if (!settled) f = decide_binary64<E>(D, species_of(pair, Enc<E>::F), d0, d1, d2, d3, K, S, beta, w1, w2);
    }
    return f;
}

// Append a near-tie to the log (counted past its capacity, stored up to it).
__device__ __forceinline__ void log_tie(const SweepArgs& A, int r, uint32_t t, int64_t site, bool acc)
{
    const int slot = atomicAdd(A.tie_count, 1);
    if (slot < A.tie_cap) {
        smcx_tie e;
        e.replica = r;
        e.sweep = t;
        e.site = site;
        e.decision = acc ? 1 : 0;
        e.pad = 0;
        A.ties[slot] = e;
    }
}

// acc + p[0] + p[STRIDE] + ... + p[STRIDE (n - 1)] in that order; the next
// reads are on their way during the adds.
template <int STRIDE>
__device__ __forceinline__ double sum_in_order(double acc, const double* p, int n)
{
    constexpr int U = 16;
    const int full = n / U;
    double v[2][U];
    auto read = [&](int c, double(&x)[U]) {
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = p[STRIDE * (U * c + k)];
    };
    auto add = [&](const double(&x)[U]) {
#pragma unroll
        for (int k = 0; k < U; ++k) acc = acc + x[k];
    };
    if (full > 0) read(0, v[0]);
    int c = 0;
    for (; c + 1 < full; c += 2) {
        read(c + 1, v[1]);
        __builtin_amdgcn_sched_barrier(0);
        add(v[0]);
        read(min(c + 2, full - 1), v[0]);
        __builtin_amdgcn_sched_barrier(0);
        add(v[1]);
    }
    if (c < full) add(v[0]);
    for (int i = full * U; i < n; ++i) acc = acc + p[STRIDE * i];
    return acc;
}

// Per-thread trial statistics, flushed with one wave reduction and three
// atomics per wave.
struct Stats {
    int att = 0, acc = 0, tie = 0;
};

// This workgroup's counters of replica r.
__device__ __forceinline__ unsigned long long* stat_slot(const SweepArgs& A, int r)
{
    return (unsigned long long*)(A.stats + ((int64_t)r * A.stat_parts + blockIdx.x % A.stat_parts) * A.stat_stride);
}

__device__ __forceinline__ int wave_sum_i(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ void flush_stats(const SweepArgs& A, int r, Stats& st)
{
    const int a = wave_sum_i(st.att), c = wave_sum_i(st.acc), t = wave_sum_i(st.tie);
    if ((threadIdx.x & 63) == 0 && r >= 0) {
        unsigned long long* p = stat_slot(A, r);
        if (a) atomicAdd(p + 0, (unsigned long long)a);
        if (c) atomicAdd(p + 1, (unsigned long long)c);
        if (t) atomicAdd(p + 2, (unsigned long long)t);
    }
    st = Stats();
}

// The same for a whole workgroup at a point every thread reaches: the waves'
// sums meet in LDS and one thread adds them to the replica's counters (one
// global atomic per counter and workgroup instead of per wave).
__device__ __forceinline__ void flush_stats_block(const SweepArgs& A, int r, Stats& st)
{
    __shared__ int red[3];
    if (threadIdx.x == 0) red[0] = red[1] = red[2] = 0;
    __syncthreads();
    const int a = wave_sum_i(st.att), c = wave_sum_i(st.acc), t = wave_sum_i(st.tie);
    if ((threadIdx.x & 63) == 0) {
        if (a) atomicAdd(&red[0], a);
        if (c) atomicAdd(&red[1], c);
        if (t) atomicAdd(&red[2], t);
    }
    __syncthreads();
    if (threadIdx.x == 0 && r >= 0) {
        unsigned long long* p = stat_slot(A, r);
        if (red[0]) atomicAdd(p + 0, (unsigned long long)red[0]);
        if (red[1]) atomicAdd(p + 1, (unsigned long long)red[1]);
        if (red[2]) atomicAdd(p + 2, (unsigned long long)red[2]);
    }
    st = Stats();
}

// Block barrier that orders LDS accesses only: global loads issued before it
// stay in flight (a full __syncthreads also drains them).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The replica table is read-only during a launch: reading it through the
// constant address space (with a wave-uniform index) lets the compiler use
// scalar loads instead of per-lane ones.
__device__ __forceinline__ const RepDev& rep_at(const RepDev* reps, int r)
{
    using CRep = const __attribute__((address_space(4))) RepDev;
    return *(const RepDev*)((CRep*)reps + r);
}
__device__ __forceinline__ const RepDev& rep_of(const SweepArgs& A, int r) { return rep_at(A.reps, r); }

// Same for other tables a launch only reads (tile prefix sums, betas).
template <typename T>
__device__ __forceinline__ T ld_const(const T* p, int64_t i)
{
    using CT = const __attribute__((address_space(4))) T;
    return ((CT*)p)[i];
}

// The replica and tile of a loop step are the same in every lane; saying so
// lets the compiler read the replica's table through scalar loads.
__device__ __forceinline__ void uniform(int& r, int64_t& tile)
{
    r = __builtin_amdgcn_readfirstlane(r);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)tile);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)tile >> 32));
    tile = (int64_t)(((uint64_t)hi << 32) | lo);
}

// Basis-planar row segments a row group's trials can write: for a cell row
// whose active sites lie in row (ya, za), the active sites' own columns (every
// basis site) in that row, and for every partner direction the partner's
// column in the row it falls in.  Any other column of the rows around stays
// as it was staged.  Worked out at compile time from the shell-1 vectors.
struct WbSeg {
    int dy, dz, col;
};
struct WbPlan {
    int n;
    WbSeg seg[4 * 2 * kMaxZ1];
};

constexpr WbPlan make_wb_plan(const Geometry& G)
{
    WbPlan P{};
    P.n = 0;
    auto add = [&P](int dy, int dz, int col) {
        for (int i = 0; i < P.n; ++i)
            if (P.seg[i].dy == dy && P.seg[i].dz == dz && P.seg[i].col == col) return;
        P.seg[P.n].dy = dy;
        P.seg[P.n].dz = dz;
        P.seg[P.n].col = col;
        ++P.n;
    };
    for (int b = 0; b < G.m; ++b) {
        add(0, 0, b);
        for (int k = 0; k < G.Z[0]; ++k) {
            const Nb nb = nb_of(G, b, G.v[0][k][0], G.v[0][k][1], G.v[0][k][2]);
            add(nb.dy, nb.dz, nb.bt);
        }
    }
    return P;
}

// Copy the window row segments a row group's trials can have changed back to
// the padded copy: each segment (a basis column of a row within a partner's
// reach of the active row) to its own row and to its halo images when the row
// lies within H of a y or z face.  A whole column goes out, x-images included
// (the trials keep those current in the window).  No other workgroup of the
// launch changes these rows (their cells' active rows lie at least a cell edge
// away), so writing back bytes that did not change is harmless.  The T0 lanes
// of the cell row share its segments, 16 bytes per lane and item.
template <int LAT, class Geo>
__device__ __forceinline__ void rows_writeback(const SweepArgs& A, const RepDev& rep, const TileGeom& tg, int lx,
                                               int T0, int ya, int za, uint8_t* pad, const uint8_t* win)
{
    constexpr WbPlan W = make_wb_plan(kGeom[LAT]);
    constexpr int NS = W.n;
    const int LP = Geo::LP(A), WY = Geo::WY(A);
    const int cp = Geo::CP(rep), nc16 = cp >> 4;  // chunks of one basis column
    const int Ly = rep.L[1], Lz = rep.L[2];
    const int64_t prowp = rep.prowp, plane = (int64_t)rep.prows * prowp;
    // g lanes per segment, consecutive lanes on consecutive 16-byte chunks,
    // so a segment's addresses are worked out once per lane; with fewer lanes
    // than segments a lane takes segments lx, lx + T0, ...
    const int g = T0 / NS;
    int d = lx, dstep = T0, c0 = 0, cstep = 1;
    if (g > 0) {
        if (lx >= g * NS) return;
        d = lx / g;
        dstep = NS;
        c0 = lx - d * g;
        cstep = g;
    }
    for (; d < NS; d += dstep) {
        int dy = 0, dz = 0, col = 0;
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i == d) {
                dy = W.seg[i].dy;
                dz = W.seg[i].dz;
                col = W.seg[i].col;
            }
        const int y = ya + dy, z = za + dz;  // in [-1, L]
        const int yr = y < 0 ? y + Ly : (y >= Ly ? y - Ly : y);
        const int zr = z < 0 ? z + Lz : (z >= Lz ? z - Lz : z);
        const int yi = yr < kHalo ? yr + Ly : (yr >= Ly - kHalo ? yr - Ly : yr);  // image, or yr itself
        const int zi = zr < kHalo ? zr + Lz : (zr >= Lz - kHalo ? zr - Lz : zr);
        const uint8_t* src = win + ((z - tg.w0[2]) * WY + (y - tg.w0[1])) * LP + col * cp + 16 * c0;
        uint8_t* dst = pad + (zr + kHalo) * plane + (yr + kHalo) * prowp + col * cp + 16 * c0;
        const int64_t ddy = (int64_t)(yi - yr) * prowp, ddz = (int64_t)(zi - zr) * plane;  // images (0: none)
        for (int c = c0; c < nc16; c += cstep) {
            const uint4 v = *(const uint4*)src;
            *(uint4*)dst = v;
            if (ddy) *(uint4*)(dst + ddy) = v;
            if (ddz) *(uint4*)(dst + ddz) = v;
            if (ddy && ddz) *(uint4*)(dst + ddy + ddz) = v;
            src += 16 * cstep;
            dst += 16 * cstep;
        }
    }
}

}  // namespace smcx
