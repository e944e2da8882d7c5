// sweep_rq.hip -- Metropolis sweeps with real couplings (paper Sec. II.A and
// Sec. III.A) for gfx950: replicas as bits of a word, decisions from tables
// per site.
//
// As in sweep_rb.hip, up to 32 replicas share an LDS word per site and a lane
// takes a Philox block (four sites of a colour) of a set of m replicas, so
// that word j of dE's six (square lattice: four) bonds, x_d = own ^ neighbour,
// serves all of them.  What a site does with the NB bits of one replica
// depends on the site alone, so each workgroup builds tables of it in LDS and
// its sets share them:
//   kThr   the threshold itself, one entry for each of the 2^NB patterns
//          (the recipe of step_common.h, evaluated once per site and pattern):
//          an attempt is its draw, one LDS read and a compare.  256 bytes a
//          site on the cubic lattice (L <= 8), 64 on the square one (L <= 45);
//   kField the bond sums of two halves of the bonds, 64 bytes a site
//          (L <= 12), 32 on the square lattice (all L).  The decision compares
//          log2 of the draw with the move's exponent and takes the exact
//          recipe where the two are closer than the error of either;
//   kBonds (cubic, L >= 13) the three couplings that start at the site, 12
//          bytes; a lane keeps its block's in registers through a colour step
//          and sums them for each replica.  The decision as in kField.
// Entry e of all sites is one array, so that a lane's bank follows from its
// site alone (site planes are multiples of 64 words): no entry chosen by any
// lane conflicts with another's.
//
// What bounds it: instruction issue, 16 instructions an attempt (kThr), 28
// (kField) or 32 (kBonds) with two to four waves a SIMD; the tables fill the
// LDS.  Attempts per ns at 10 sweeps a step, beta = 1.5, against a form that
// swept replica quads with neighbours and couplings in registers (53
// instructions an attempt, two waves a SIMD and spills beyond L = 17): cubic
// L = 8, R = 10^5: 542 -> 1448; L = 10, R = 5 10^4: 527 -> 1098; L = 12,
// R = 3 10^4: 459 -> 978; L = 13, R = 2 10^4: 308 -> 783; L = 16, R = 2 10^4:
// 584 -> 1010; L = 20, R = 10^4: 263 -> 926; square L = 32, R = 5 10^4: 595 ->
// 1740; L = 64, R = 2 10^4: 648 -> 1003.
#include <algorithm>

#include "launch.h"
#include "pamc_dev.h"
#include "rb_common.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

namespace {

// acc = 2 acc + [u <= Q], acc = 2 acc + [v > 0]
__device__ __forceinline__ void push_le(uint32_t &acc, uint32_t u, uint32_t Q)
{
    asm("v_cmp_le_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(acc) : "v"(u), "v"(Q) : "vcc");
}
__device__ __forceinline__ void push_positive(uint32_t &acc, float v)
{
    asm("v_cmp_lt_f32 vcc, 0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(acc) : "v"(v) : "vcc");
}

// Coupling of bond d of site i of block g of colour c.
typedef __attribute__((address_space(1))) const int32_t *GlobalInt;
struct RQInst {
    GlobalInt J;  // [ncol][gmax][24], [direction][site]
    float bq;     // beta 2^-20
    float scale;  // -2 log2(e) bq, finite (see kNear)
};
__device__ __forceinline__ int32_t coupling(const RBInst &X, const RQInst &Q, int c, int g, int d, int i)
{
    return Q.J[(size_t)(uint32_t)(c * X.gmax + g) * 24 + 4 * d + i];
}

// Entry e of site i of the row's block b is word e 4 plane + i plane + b.
// Bond sum sum_d J_d (1 - 2 x_d) of pattern bits [lo, hi) (dE is twice that
// over all bonds).
template <int NB>
__device__ __forceinline__ int32_t bond_sum(const int32_t (&J)[NB], int lo, int hi, uint32_t bits)
{
    int32_t h = 0;
#pragma unroll
    for (int d = 0; d < NB; ++d)
        if (d >= lo && d < hi) h += (bits >> (d - lo)) & 1u ? -J[d] : J[d];
    return h;
}

// Threshold of dE > 0 as the largest accepted draw Q: u <= Q accepts.  A move
// that no draw accepts has Q = 0 as well: draws of 0 are told
// apart by the exact rule.
__device__ __forceinline__ uint32_t threshold(float bq, int32_t dE)
{
    const float x = -(bq * (float)dE);
    const float e = exp_recipe(__builtin_fmaxf(x, -24.0f));
    if (!(x >= -23.0f)) return 0u;
    if (e >= 1.0f) return 0xFFFFFFFFu;
    const uint32_t T = (uint32_t)(e * 4294967296.0f);
    return T > 0u ? T - 1u : 0u;
}

// The workgroup's table.  fields: the half sums even where KIND has
// thresholds (for the energies).
template <int NB, int KIND>
__device__ __forceinline__ void build_table(const RBInst &X, const RQInst &Q, uint32_t *table, bool fields, int tid)
{
    constexpr int H = NB / 2, P = 1 << H;
    const int entry = 4 * X.plane, sites = 4 * X.gmax * X.ncol;
    // kThr: pattern and complement have opposite dE, 2^(NB-1) pairs a site in
    // rows of eight; several threads a site where there are more threads
    constexpr int kRows = NB == 6 ? 4 : 1;
    const int parts = KIND == kRQThr && !fields ? max(1, min(kRows, (int)blockDim.x / sites)) : 1;
    for (int it = tid; it < sites * parts; it += blockDim.x) {
        const int part = it / sites, site = it - part * sites;
        const int ci = site / X.gmax, g = site - ci * X.gmax, c = ci >> 2, i = ci & 3;
        if (g >= pick3(X.gcs, c)) continue;
        int32_t J[NB], lo[8];
#pragma unroll
        for (int d = 0; d < NB; ++d) J[d] = coupling(X, Q, c, g, d, i);
        uint32_t *t = table + i * X.plane + pick3(X.base, c) + g;
        if (KIND == kRQBonds) {
#pragma unroll
            for (int d = 0; d < NB; d += 2) t[(d >> 1) * entry] = (uint32_t)J[d];
        } else if (KIND == kRQThr && !fields) {
            // (the first three bonds' sums of every pattern)
#pragma unroll
            for (int p = 0; p < 8; ++p) lo[p] = bond_sum<NB>(J, 0, 3, (uint32_t)p);
#pragma unroll 1
            for (int row = part; row < kRows; row += parts) {
                const int32_t hi = bond_sum<NB>(J, 3, NB, (uint32_t)row);
                uint32_t *tp = t + 8 * row * entry, *tc = t + ((1 << NB) - 1 - 8 * row) * entry;
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const int32_t dE = 2 * (lo[p] + hi);
                    const uint32_t T = threshold(Q.bq, abs(dE));
                    tp[p * entry] = dE > 0 ? T : 0xFFFFFFFFu;
                    tc[-p * entry] = dE < 0 ? T : 0xFFFFFFFFu;
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                t[p * entry] = (uint32_t)bond_sum<NB>(J, 0, H, (uint32_t)p);
                t[(P + p) * entry] = (uint32_t)bond_sum<NB>(J, H, NB, (uint32_t)p);
            }
        }
    }
}

// x[i][d]: own ^ neighbour of the four sites of a block, all replicas.
template <int NB>
struct Bonds {
    uint32_t own[4], x[4][NB];
};
template <int NB>
__device__ __forceinline__ void block_bonds(const uint32_t *lds, const Record &rec, int own, int plane, Bonds<NB> &f)
{
    const u32x4 q0 = rec.q[0], q1 = rec.q[1], q2 = rec.q[2];
    const uint32_t e[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
#pragma unroll
    for (int d = 0; d < NB; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = e[2 * d + (i >> 1)];
            f.x[i][d] = lds[(i & 1) ? w >> 16 : w & 0xFFFFu];
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f.own[i] = lds[own + i * plane];
#pragma unroll
        for (int d = 0; d < NB; ++d) f.x[i][d] ^= f.own[i];
    }
}

// Couplings of a block's bonds (kRQBonds): the one to s + e_d is entry d of
// the site, the one to s - e_d entry d of that neighbour.
template <int NB>
__device__ __forceinline__ void block_couplings(const uint32_t *table, const Record &rec, int own, int plane, int32_t (&J)[4][NB],
                                                int32_t (&sum)[4])
{
    const u32x4 q0 = rec.q[0], q1 = rec.q[1], q2 = rec.q[2];
    const uint32_t e[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sum[i] = 0;
#pragma unroll
        for (int d = 0; d < NB; ++d) {
            const uint32_t w = e[2 * d + (i >> 1)];
            const uint32_t at = d & 1 ? ((i & 1) ? w >> 16 : w & 0xFFFFu) : (uint32_t)(own + i * plane);
            J[i][d] = (int32_t)table[(d >> 1) * 4 * plane + at];
            sum[i] += J[i][d];
        }
    }
}
// acc += a b, factors of 24 bits
__device__ __forceinline__ void mad24(int32_t &acc, int32_t a, int32_t b)
{
    asm("v_mad_i32_i24 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// Bond sum of a site in replica r: sum J_d (1 - 2 x_d), |J_d| < 2^23.
template <int NB>
__device__ __forceinline__ int32_t field_from_bonds(const uint32_t (&x)[NB], const int32_t (&J)[NB], int32_t sum, int r)
{
    int32_t a = 0;
#pragma unroll
    for (int d = 0; d < NB; ++d) mad24(a, __builtin_amdgcn_sbfe((int)x[d], (uint32_t)r, 1u), J[d]);
    return sum + 2 * a;
}

// Within each byte, bit j of a[i] <-> bit i of a[j]: afterwards byte b of a[k]
// holds, in bit i, bit 8 b + k of the i-th word.
__device__ __forceinline__ void transpose8(uint32_t (&a)[8])
{
    constexpr uint32_t mask[3] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu};
#pragma unroll
    for (int t = 2; t >= 0; --t) {
        const int s = 1 << t;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (k & s) continue;
            const uint32_t lo = a[k], hi = a[k + s];
            a[k] = (lo & mask[t]) | ((hi << s) & ~mask[t]);
            a[k + s] = ((lo >> s) & mask[t]) | (hi & ~mask[t]);
        }
    }
}

// Exact decision of site i in replica r of the set.
template <int NB>
__device__ __forceinline__ bool exact_accept(const RBInst &X, const RQInst &Q, const Bonds<NB> &f, int c, int g, int i,
                                             int r, uint32_t u)
{
    int32_t h = 0;
#pragma unroll
    for (int d = 0; d < NB; ++d) {
        const int32_t j = coupling(X, Q, c, g, d, i);
        h += (f.x[i][d] >> r) & 1u ? -j : j;
    }
    const int32_t dE = 2 * h;
    return dE <= 0 || real_accept(Q.bq, dE, u);
}

// Patterns of a block: byte b of w[i][kk] holds, in bit d, bond d of site i in
// replica 8 b + kk.
template <int NB>
__device__ __forceinline__ void patterns(const Bonds<NB> &f, uint32_t (&w)[4][8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int d = 0; d < 8; ++d) w[i][d] = d < NB ? f.x[i][d < NB ? d : 0] : 0u;
        transpose8(w[i]);
    }
}
// The entry of n pattern bits of w from bit `at` on; t: entry 0 of the site,
// `stride` bytes an entry.
template <int N>
__device__ __forceinline__ uint32_t entry_of(const uint32_t *t, uint32_t stride, uint32_t w, int at)
{
    const uint32_t p = (w >> at) & ((1u << N) - 1u);
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(t) + __umul24(p, stride));
}
// Sum of the bonds of a site, from the two half tables.
template <int NB>
__device__ __forceinline__ int32_t field_of(const uint32_t *t, const uint32_t *t2, uint32_t stride, uint32_t w, int at)
{
    constexpr int H = NB / 2;
    return (int32_t)(entry_of<H>(t, stride, w, at) + entry_of<H>(t2, stride, w, at + H));
}

// kField: log2 of the draw against the exponent.  A move with bond sum h is
// accepted when u < floor(e 2^32), e = exp(-bq 2 h) by the recipe, that is
// when log2(u + 1) <= 32 + log2 e; y = 32 - 2 bq log2(e) h and
// l = log2(u + 1) in binary32.  For moves that any draw can accept (y >= -1)
// the errors in units of log2 are: y, three roundings of a product of at most
// 33 and one of a sum of at most 32, below 8e-6; l, the rounding of u + 1 (two
// of 2^-24 relative: 2e-7) and one ulp of the logarithm (below 32: 4e-6); the
// recipe's argument, two roundings of at most 23 / ln 2 = 33 (4e-6), its
// result, four ulps (7e-7), and the floor, which moves the boundary by less
// than one draw, exact in u + 1.  Together below 2e-5; closer pairs than
// kNear are decided by the recipe.  The factor of h is held finite: from
// beta = 1.2e44 on it would be infinite, and its product with h = 0 (dE = 0,
// always accepted) not a number; any other h puts y beyond every draw either
// way.
constexpr float kNear = 4.0e-5f;

// One colour step of block g for the m replicas from row rb on (see rb_block).
template <int NB, int KIND, bool UNI, bool ALL>
__device__ __forceinline__ void rq_block(const RBInst &X, const RQInst &Q, uint32_t *lds, const uint32_t *table, int c, int g,
                                         bool has, uint32_t rb, int m, int k, int t, Record &rec, int next_c, int next_g)
{
    const int plane = X.plane, own = pick3(X.base, c) + g;
    const uint32_t k0 = X.k0, k1 = X.k1, ctr = ((uint32_t)c << 24) | (uint32_t)g;
    const uint32_t valid = rec.q[3].y;
    uint32_t flip[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    // (opaque: each replica's part of the draws and comparison with m would be
    // hoisted out of the sweeps, some hundred registers)
    if constexpr (UNI)
        asm volatile("" : "+s"(rb), "+s"(m));
    else
        asm volatile("" : "+v"(rb), "+s"(m));
    Bonds<NB> f;
    if constexpr (ALL) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f.own[i] = lds[own + i * plane];
        rec = load_record(X, next_c, next_g);
    } else {
        block_bonds<NB>(lds, rec, own, plane, f);
        [[maybe_unused]] int32_t J[4][NB], Jsum[4];
        if constexpr (KIND == kRQBonds) block_couplings<NB>(table, rec, own, plane, J, Jsum);
        // the next block's record is on its way while this one draws
        rec = load_record(X, next_c, next_g);
        const LaneDraw d = lane_draw(ctr, k, t, k0, k1);
        const uint32_t *tab[4], *tab2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tab[i] = table + own + i * plane;
            tab2[i] = tab[i] + (4 * plane << (NB / 2));
        }
        const uint32_t stride = 16u * (uint32_t)plane;
        uint32_t acc[4][4] = {};  // [byte][site]: replicas 8 b ... 8 b + 7
        uint32_t again = 0u;  // kThr: any, kField: the r & 7 of draws to decide exactly
        uint32_t mn = 0xFFFFFFFFu;
        float near = 1.0f;
        // replica r: its pattern in w[i] from bit `at` on, its decisions to a
        auto attempt = [&](int r, const uint32_t (&w)[4], int at, uint32_t (&a)[4]) {
            uint32_t e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                e[i] = KIND == kRQThr     ? entry_of<NB>(tab[i], stride, w[i], at)
                       : KIND == kRQField ? (uint32_t)field_of<NB>(tab[i], tab2[i], stride, w[i], at)
                                          : (uint32_t)field_from_bonds<NB>(f.x[i], J[i], Jsum[i], r);
            const uint4 u = replica_draw<UNI>(d, rb + (uint32_t)r, k, k0, k1);
            if constexpr (KIND == kRQThr) {
#pragma unroll
                for (int i = 0; i < 4; ++i) push_le(a[i], word_of(u, i), e[i]);
                mn = min(min(min(min(mn, u.x), u.y), u.z), u.w);
            } else {
                float diff[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float y = __builtin_fmaf((float)(int32_t)e[i], Q.scale, 32.0f);
                    diff[i] = y - __builtin_amdgcn_logf((float)word_of(u, i) + 1.0f);
                    push_positive(a[i], diff[i]);
                }
                near = __builtin_fminf(__builtin_fminf(near, __builtin_fabsf(diff[0])), __builtin_fabsf(diff[1]));
                near = __builtin_fminf(__builtin_fminf(near, __builtin_fabsf(diff[2])), __builtin_fabsf(diff[3]));
            }
        };
        if (m <= 4) {
            // (the transposes of `patterns` cost more than picking the bits)
#pragma unroll 1
            for (int r = m - 1; r >= 0; --r) {
                uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int i = 0; i < (KIND == kRQBonds ? 0 : 4); ++i)
#pragma unroll
                    for (int dd = 0; dd < NB; ++dd) w[i] |= __builtin_amdgcn_ubfe(f.x[i][dd], (uint32_t)r, 1u) << dd;
                attempt(r, w, 0, acc[0]);
            }
            if constexpr (KIND != kRQThr) again = __builtin_amdgcn_ballot_w64(near < kNear) != 0ull ? 0xFFu : 0u;
        } else {
            uint32_t w[4][8];
            if constexpr (KIND != kRQBonds) patterns<NB>(f, w);
#pragma unroll
            for (int kk = 7; kk >= 0; --kk) {
                near = 1.0f;
                uint32_t wk[4];
                if constexpr (KIND != kRQBonds)
                    for (int i = 0; i < 4; ++i) wk[i] = w[i][kk];
#pragma unroll
                for (int b = 3; b >= 0; --b)
                    if (8 * b + kk < m) attempt(8 * b + kk, wk, 8 * b, acc[b]);
                if constexpr (KIND != kRQThr)
                    again |= __builtin_amdgcn_ballot_w64(near < kNear) != 0ull ? 1u << kk : 0u;
            }
        }
        if constexpr (KIND == kRQThr) again = __builtin_amdgcn_ballot_w64(mn == 0u) != 0ull ? 0xFFu : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) flip[i] = acc[0][i] | (acc[1][i] << 8) | (acc[2][i] << 16) | (acc[3][i] << 24);
        if (__builtin_expect(again != 0u, 0)) {
            // (the neighbours have not changed since)
            Bonds<NB> f2;
            block_bonds<NB>(lds, load_record(X, c, g), own, plane, f2);
#pragma unroll 1
            for (int r = 0; r < m; ++r) {
                if (!((again >> (r & 7)) & 1u)) continue;
                const uint4 u = replica_draw<UNI>(d, rb + (uint32_t)r, k, k0, k1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (KIND == kRQThr && word_of(u, i) != 0u) continue;
                    const bool ok = exact_accept<NB>(X, Q, f2, c, g, i, r, word_of(u, i));
                    flip[i] = (flip[i] & ~(1u << r)) | ((ok ? 1u : 0u) << r);
                }
            }
        }
    }
    const bool whole = __builtin_amdgcn_ballot_w64(has && valid != 15u) == 0ull;
    if (!has) return;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (whole || ((valid >> i) & 1u)) lds[own + i * plane] = f.own[i] ^ flip[i];
}

// UNI: wps waves per set, so the replica index is uniform; else the blocks of
// all sets side by side.
struct Place {
    int set, g0, step;
    bool act;
};
template <bool UNI>
__device__ __forceinline__ Place place(const RBInst &X, int sets, int tid)
{
    Place p;
    if constexpr (UNI) {
        const int wps = ((int)blockDim.x >> 6) / sets, wave = scalar(tid >> 6);
        p.set = wave / wps;
        p.g0 = (wave - p.set * wps) * 64 + (tid & 63);
        p.step = 64 * wps;
    } else {
        p.set = tid / X.gmax;
        p.g0 = tid - p.set * X.gmax;
        p.step = X.gmax;
    }
    p.act = p.set < sets;
    if (!p.act) p.set = 0;
    return p;
}

template <int NB, int KIND, bool UNI, bool ALL>
__device__ __forceinline__ void rq_sweeps(const RBInst &X, const RQInst &Q, int k, uint32_t *lds, const uint32_t *table,
                                          int r0, int m, int sets, int t0, int t1, int tid)
{
    const bool local = UNI && (int)blockDim.x == 64 * sets;
    const Place p = place<UNI>(X, sets, tid);
    uint32_t *sp = lds + p.set * 4 * X.plane;
    uint32_t rb = (uint32_t)(r0 + p.set * m);
    if constexpr (UNI) rb = scalar(rb);
    const int last = X.gmax - 1;  // (records past a colour's blocks are zeros)
    Record rec = load_record(X, 0, min(p.g0, last));
    for (int t = t0; t < t1; ++t) {
        // (waves of their own sets: the workgroup is done when the last is;
        // L = 8, R = 10^5: 395 -> 375 us)
        if (local) even_progress(t, t0, t1);
        for (int c = 0; c < X.ncol; ++c) {
            const int nc = c + 1 < X.ncol ? c + 1 : 0;
            for (int first = 0; first <= last; first += p.step) {
                const int g = p.g0 + first;
                const bool more = first + p.step <= last;
                rq_block<NB, KIND, UNI, ALL>(X, Q, sp, table, c, min(g, last), p.act && g < pick3(X.gcs, c), rb, m, k, t, rec,
                                             more ? c : nc, min(more ? g + p.step : p.g0, last));
            }
            set_barrier(local);
        }
    }
    if (local) __builtin_amdgcn_s_setprio(3);
}

// Energies E = -sum_b J S S from the sites' bond sums h = sum_d J_d (1 - 2 x_d):
// with two colours the sites of colour 0 see each bond once (E = -sum h), with
// three all sites see it twice (E = -1/2 sum h).  eacc (zeroed) collects the
// sums of h.
template <int NB, int KIND, bool UNI>
__device__ __forceinline__ void rq_energy(const RBInst &X, const RQInst &Q, const uint32_t *lds, const uint32_t *table,
                                          unsigned long long *eacc, int m, int sets, int tid)
{
    const Place p = place<UNI>(X, sets, tid);
    const uint32_t *sp = lds + p.set * 4 * X.plane;
    const int nc = X.ncol == 2 ? 1 : X.ncol, last = X.gmax - 1;
    // (opaque: atomics on an address known to be uniform are serialised lane
    // by lane)
    int zero = 0;
    asm volatile("" : "+v"(zero));
    unsigned long long *es = eacc + p.set * m + zero;
    for (int c = 0; c < nc; ++c)
        for (int first = 0; first <= last; first += p.step) {
            const int g = min(p.g0 + first, last);
            const bool has = p.act && p.g0 + first < pick3(X.gcs, c);
            const Record rec = load_record(X, c, g);
            const uint32_t valid = has ? rec.q[3].y : 0u;
            const int own = pick3(X.base, c) + g;
            Bonds<NB> f;
            block_bonds<NB>(sp, rec, own, X.plane, f);
            [[maybe_unused]] int32_t J[4][NB], Jsum[4];
            uint32_t w[4][8];
            if constexpr (KIND == kRQBonds)
                block_couplings<NB>(table, rec, own, X.plane, J, Jsum);
            else
                patterns<NB>(f, w);
            int n = m;  // (opaque, as in rq_block)
            asm volatile("" : "+s"(n));
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int r = 8 * b + kk;
                    if (r >= n) continue;
                    int32_t h = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t *t = table + own + i * X.plane;
                        int32_t s;
                        if constexpr (KIND == kRQBonds)
                            s = field_from_bonds<NB>(f.x[i], J[i], Jsum[i], r);
                        else
                            s = field_of<NB>(t, t + (4 * X.plane << (NB / 2)), 16u * (uint32_t)X.plane, w[i][kk], 8 * b);
                        h += (valid >> i) & 1u ? s : 0;
                    }
                    if constexpr (UNI) {
                        h += __builtin_amdgcn_mov_dpp(h, 0xB1, 0xF, 0xF, true);   // quad_perm 1 0 3 2
                        h += __builtin_amdgcn_mov_dpp(h, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
                        h += __builtin_amdgcn_mov_dpp(h, 0x141, 0xF, 0xF, true);  // row_half_mirror
                        if ((tid & 7) == 0) atomicAdd(&es[r], (unsigned long long)(long long)h);
                    } else if (has) {
                        atomicAdd(&es[r], (unsigned long long)(long long)h);
                    }
                }
        }
}

// The workgroup's LDS: the table, the sets' words, then per set 32 energies
// (64 bits), 32 source rows and 32 family ids.
template <int NB, int KIND, bool UNI>
__device__ __forceinline__ void rq_tile(const Inst &I, int k, uint32_t *table, int r0, int nrows, int m, int sets,
                                        int phase)
{
    constexpr int words = KIND == kRQThr ? 1 << NB : KIND == kRQField ? 2 << (NB / 2) : NB / 2;
    const int pass = m * sets;
    const TileIO io = tile_io(I);
    const RBInst X = rb_inst(I, io);
    RQInst Q;
    Q.J = (GlobalInt)scalar_ptr(I.cmj);
    Q.bq = __uint_as_float(scalar(__float_as_uint(I.bq[k])));
    Q.scale = __uint_as_float(scalar(__float_as_uint(__builtin_fmaxf(-2.0f * 1.44269504f * Q.bq, -3.0e38f))));
    const bool all = scalar(I.thr[k].w) != 0u;
    const int ns = scalar(I.NS), t0 = phase == 2 ? ns / 2 : 0, t1 = phase == 1 ? ns / 2 : ns;
    uint32_t *lds = table + 4 * X.plane * words;
    unsigned long long *eacc = reinterpret_cast<unsigned long long *>(lds + 4 * X.plane * sets);
    uint32_t *src = reinterpret_cast<uint32_t *>(eacc + 32 * sets), *fam = src + 32 * sets;
    for (int q0 = 0; q0 < nrows; q0 += pass) {
        const int row0 = r0 + q0, nr = min(pass, nrows - q0);
        // (opaque: what follows from it would be hoisted out of this loop and
        // its registers held through the sweeps)
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));
        // rows past the end are swept as copies of the pass's first row and
        // never stored
        for (int q = tid; q < pass; q += blockDim.x) {
            uint32_t r = (uint32_t)(row0 + (q < nr ? q : 0));
            if (io.map) r = io.map[r];
            src[q] = r;
            eacc[q] = 0ull;
        }
        if (KIND != kRQThr ? q0 == 0 : !all) build_table<NB, KIND>(X, Q, table, false, tid);
        __syncthreads();
        rb_load<false>(X, lds, src, m, sets, tid);
        for (int q = tid; q < nr; q += blockDim.x) fam[q] = io.fsrc[src[q]];
        __syncthreads();
        if (all)
            rq_sweeps<NB, KIND, UNI, true>(X, Q, k, lds, table, row0, m, sets, t0, t1, tid);
        else
            rq_sweeps<NB, KIND, UNI, false>(X, Q, k, lds, table, row0, m, sets, t0, t1, tid);
        __syncthreads();
        if (phase != 1) {
            if (KIND == kRQThr) {
                build_table<NB, KIND>(X, Q, table, true, tid);
                __syncthreads();
            }
            rq_energy<NB, KIND, UNI>(X, Q, lds, table, eacc, m, sets, tid);
        }
        rb_store<false>(X, lds, row0, nr, m, sets, tid);
        if (io.map)
            for (int q = tid; q < nr; q += blockDim.x) io.fdst[row0 + q] = fam[q];
        __syncthreads();
        if (phase != 1) {
            for (int q = tid; q < nr; q += blockDim.x) {
                const long long h = (long long)eacc[q];
                eacc[q] = (unsigned long long)(X.ncol == 2 ? -h : -(h / 2));
            }
            __syncthreads();
            tile_energies_real(I, io, eacc, row0, nr);
            tile_family_count(I, fam, nr);
            __syncthreads();
        }
    }
}

}  // namespace

template <int NB, int KIND, bool UNI>
__global__ __launch_bounds__(1024) void k_sweep_rq(const Inst *insts, const Work *work, int tile_rows, int m, int sets,
                                                    int phase)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = scalar(*I.k);
    if (k >= I.nT || I.status[0]) return;
    const int Rk = (int)I.Rk[k];
    const int r0 = scalar((int)w.row0);
    const int nrows = scalar(min(tile_rows, Rk - r0));
    if (nrows > 0) rq_tile<NB, KIND, UNI>(I, k, reinterpret_cast<uint32_t *>(lds), r0, nrows, m, sets, phase);
    if (phase == 1) phase1_done(I, w.n);
}

// Thresholds cost their making once a workgroup (32 evaluations of the recipe
// a site on the cubic lattice, 8 on the square one, some 40 instructions
// each) and save 12 instructions an attempt: from 16 and 4 rows on at 10
// sweeps a step.
int rq_kind(int variant, int rows)
{
    if (variant == kSweepRQ3Bonds) return kRQBonds;
    return (variant == kSweepRQ3Thr && rows >= 16) || (variant == kSweepRQ2Thr && rows >= 4) ? kRQThr : kRQField;
}
int64_t rq_lds(int variant, int plane, int m, int sets)
{
    const bool cubic = variant == kSweepRQ3Thr || variant == kSweepRQ3Field;
    const int words = variant == kSweepRQ3Bonds                  ? 3
                      : rq_kind(variant, m * sets) == kRQThr ? (cubic ? 64 : 16)
                                                             : (cubic ? 16 : 8);
    return (int64_t)16 * plane * words + (int64_t)(16 * plane + 512) * sets;
}

// Waves of one set each where they waste few lanes, else the blocks of all
// sets side by side.
bool rq_uniform(int G) { return G >= 48 && 100 * G >= 84 * 64 * ((G + 63) / 64); }
int rq_threads(int G, int sets)
{
    return rq_uniform(G) ? (G + 63) / 64 * 64 * sets : (G * sets + 63) / 64 * 64;
}

hipError_t sweep_rq_init()
{
    const void *fns[] = {
        (const void *)&k_sweep_rq<6, kRQThr, true>,   (const void *)&k_sweep_rq<6, kRQThr, false>,
        (const void *)&k_sweep_rq<6, kRQField, true>, (const void *)&k_sweep_rq<6, kRQField, false>,
        (const void *)&k_sweep_rq<6, kRQBonds, true>, (const void *)&k_sweep_rq<6, kRQBonds, false>,
        (const void *)&k_sweep_rq<4, kRQThr, true>,   (const void *)&k_sweep_rq<4, kRQThr, false>,
        (const void *)&k_sweep_rq<4, kRQField, true>, (const void *)&k_sweep_rq<4, kRQField, false>,
    };
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxWordLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void launch_sweep_rq(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    const bool uni = rq_uniform(sh.G);
    const int nt = rq_threads(sh.G, sh.sets);
    const int nb = sh.variant == kSweepRQ2Thr || sh.variant == kSweepRQ2Field ? 4 : 6;
    const int kind = rq_kind(sh.variant, sh.M * sh.sets);
    const size_t lds = (size_t)rq_lds(sh.variant, sh.plane, sh.M, sh.sets);
#define PAMC_RQ(NB, KIND)                                                                                             \
    if (nb == NB && kind == KIND) {                                                                                   \
        if (uni)                                                                                                      \
            k_sweep_rq<NB, KIND, true><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.M, sh.sets, phase);      \
        else                                                                                                          \
            k_sweep_rq<NB, KIND, false><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.M, sh.sets, phase);     \
    }
    PAMC_RQ(6, kRQThr)
    PAMC_RQ(6, kRQField)
    PAMC_RQ(6, kRQBonds)
    PAMC_RQ(4, kRQThr)
    PAMC_RQ(4, kRQField)
#undef PAMC_RQ
}

}  // namespace pamc
