// resample.hip -- resampling and the per-step statistics (paper Sec. II.B,
// Eq. (2), Sec. V.A) for gfx950.
//
// After the sweeps, one post launch runs four kinds of workgroups per
// instance:
//   copies    the step's normaliser, and n_r = floor(tau) + [u_r < frac(tau)
//             2^32] for 1024 rows with their exclusive scan inside the
//             workgroup;
//   measure   the step's energy record;
//   families  n ln n of 2048 family ids, summed by the pairwise tree;
//   overlap   spin overlaps of 2048 replica pairs (at overlap steps).
// The last workgroup of an instance to finish scans the per-workgroup
// totals into offsets, sets R_{k+1} and the capacity / extinction status,
// folds the family partial sums, and advances the step.  Small populations
// get their copy map (destination row -> source row, stable order) from it as
// well, the others from an expand launch, which also clears the step's energy
// histogram; the next sweep reads its tile through the map.
//
// What bounds it: a chain of dependent steps, not bytes: reads of the
// descriptor, the step's state and the energies in turn, and instructions that
// each launch fetches anew (the same routine took twice as long on its first
// call in a launch as on its second).  With trees and scans in registers
// instead of through LDS (two barriers a level), the energy sums in a
// workgroup of their own, the histogram's parts read once, uniform values in
// scalar registers, families of small populations counted here instead of by
// atomics of the sweep's workgroups, and no launch for a small map, the
// launches after a sweep take 12.5 us at L = 4, R = 1000 (21 before), 25 at
// L = 10, R = 20000 (34) and 24 at L = 8, R = 10^5 (35).
#include "launch.h"
#include "pamc_dev.h"
#include "step_common.h"

namespace pamc {

// Lowest energy of the step, from its parts (every lane returns it).
__device__ __forceinline__ long long lowest_energy(const Inst &I)
{
    static_assert(kMinParts == 64, "one part per lane");
    long long e = I.emin[threadIdx.x & 63];
    for (int off = 32; off > 0; off >>= 1) {
        const long long o = __shfl_xor(e, off);
        e = o < e ? o : e;
    }
    return e;
}

struct MomentSum {
    long long emax;
    unsigned long long sum, lo, hi;
    __device__ __forceinline__ void add(const MomentSum &o)
    {
        emax = o.emax > emax ? o.emax : emax;
        sum += o.sum;
        const unsigned long long l = lo + o.lo;
        hi += o.hi + (l < lo ? 1ull : 0ull);
        lo = l;
    }
    // over the workgroup, into thread 0 (one barrier)
    __device__ __forceinline__ void reduce(MomentSum *sh)
    {
        for (int off = 32; off > 0; off >>= 1) {
            MomentSum o{__shfl_xor(emax, off), __shfl_xor(sum, off), __shfl_xor(lo, off), __shfl_xor(hi, off)};
            add(o);
        }
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = *this;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w) add(sh[w]);
    }
};

// Where the blocks' moments wait between the weights launch and the next one:
// the copy map, which the sweeps have consumed and the next expand writes.
__device__ __forceinline__ BlockMoments *block_moments(const Inst &I) { return reinterpret_cast<BlockMoments *>(I.map); }

// Resampling weights with real couplings (Sec. II.B), for rows
// [row0, row0 + 1024) of one instance after the sweeps of step k:
// w_r = exp(-dbeta (E_r - E_min)) as the product over the set bits b of
// E_r - E_min (units of 2^-20) of exp(-dbeta 2^(b-20)), in ascending b.  The
// block's 1024 leaves (zero beyond R_k) form an aligned subtree of the
// pairwise tree over rows 0 .. P-1 (P the smallest power of two >= R_k); the
// copies workgroups fold the block roots (real_normaliser).  For P < 1024 the
// block tree adds only zeros above the P-leaf subtree, which leaves its sum
// unchanged.  The block's moments go to measure_role.
__global__ __launch_bounds__(512) void k_weights(const Inst *insts, const Work *work)
{
    __shared__ double pw[40];
    __shared__ double a[512];
    __shared__ MomentSum sh[8];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int4 ctl = *reinterpret_cast<const int4 *>(I.k);
    const int k = scalar(ctl.x), row0 = scalar((int)w.row0);
    if (!inst_live(I, k)) return;
    const bool resample = k < scalar(I.nT) - 1;
    const int Rk = (int)scalar(I.Rk[k]);
    if (row0 >= Rk && !resample) return;
    const int t = threadIdx.x;
    if (resample && t < 40) pw[t] = I.gpw[(size_t)k * 40 + t];
    const long long emin = lowest_energy(I);
    const int64_t *E = I.Eq[scalar(ctl.y ^ ctl.z)];
    int64_t e[2] = {0, 0};
    MomentSum m{-kNoEnergy - 1, 0ull, 0ull, 0ull};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = row0 + 2 * t + j;
        if (r < Rk) e[j] = E[r];
    }
    if (resample) {
        __syncthreads();
        double l[2] = {0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = row0 + 2 * t + j;
            if (r < Rk) {
                const double x = weight64(pw, (uint64_t)(e[j] - emin));
                I.wrep[r] = x;
                l[j] = x;
            }
        }
        const double root = wg_tree(l[0] + l[1], 512, a);
        if (t == 0) I.wpart[row0 / kRowsPerBlock] = root;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (row0 + 2 * t + j < Rk) {
            const unsigned __int128 e2 = (unsigned __int128)((__int128)e[j] * (__int128)e[j]);
            m.add(MomentSum{e[j], (unsigned long long)e[j], (unsigned long long)e2, (unsigned long long)(e2 >> 64)});
        }
    m.reduce(sh);
    if (t == 0) block_moments(I)[row0 / kRowsPerBlock] = BlockMoments{m.emax, m.sum, m.lo, m.hi};
}

// The normaliser of a step with real couplings: the pairwise tree over the
// block roots (zero for blocks beyond R_k).
__device__ __forceinline__ double real_normaliser(const Inst &I, int Rk, double *a)
{
    int P = 1;
    while (P < Rk) P <<= 1;
    const int nroot = P > kRowsPerBlock ? P / kRowsPerBlock : 1;
    return tree_sum<1024>(
        nroot, [&](int b) { return b * kRowsPerBlock < Rk ? I.wpart[b] : 0.0; }, a, a + 1024);
}

// Inclusive scan over a wave (DPP row shifts, then the rows' totals).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr 1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast 15, rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast 31, rows 2 and 3
    return v;
}

// Exclusive scan over the workgroup (at most 1024 threads).
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t *sh, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t x = wave_scan(v);
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    const uint32_t sums = wave_scan(lane < (int)(blockDim.x >> 6) ? sh[lane] : 0u);
    *total = (uint32_t)__builtin_amdgcn_readlane((int)sums, 63);
    const uint32_t before = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)sums, wave - 1) : 0u;
    __syncthreads();
    return before + x - v;
}

// Energies of a step with +-1 couplings, by a workgroup of 1024 threads: the
// lowest and highest occupied level (level m: E = 2 m - 3 N), and for
// k < nT-1 the level weights w[m] = exp(-2 dbeta m) as a fixed product of
// rho^(2^b) and their normaliser S by the pairwise tree over
// 2^ceil(log2(M+1)) levels.  Every copies workgroup takes them for itself: its
// pass over the energies or the histogram comes out of the L2 (12 loads a
// thread at L = 8), where one workgroup at the end of the sweep launch kept
// the whole chip waiting (64 threads at L = 8: about 25 us a step) and every
// other one had to count itself in.
//   Up to kDirectRows rows: the energies themselves, 32 a thread, with the
// histogram built in LDS (a sweep launch then counts nothing: its atomics on
// the few energies of a cold population follow each other about 0.1 us apart
// on each address, 15-50 us a launch at 10^4 rows).
//   Beyond: the histogram that the sweep's workgroups have counted.
// The energy sums are taken by one more workgroup (measure_role) beside them:
// 64-bit arithmetic per row that no copy count waits for.
// pw: kLevelBits doubles, a: 4096 doubles, of LDS.
// The parts of the energy histogram (global memory, the addresses read once).
typedef __attribute__((address_space(1))) const uint32_t *GlobalCounts;
struct HistParts {
    GlobalCounts first, others;
    int nlev;
    __device__ __forceinline__ HistParts(const Inst &I, int n)
        : first((GlobalCounts)scalar_ptr(I.hist)), others((GlobalCounts)scalar_ptr(I.loff)), nlev(n)
    {
    }
    __device__ __forceinline__ uint32_t count(int m, int copies) const
    {
        uint32_t c = first[m];
        const GlobalCounts p = others + m;
#pragma unroll 8
        for (int i = 0; i < copies - 1; ++i) c += p[(size_t)((uint32_t)i * (uint32_t)nlev)];
        return c;
    }
};
constexpr int kLevelRing = 4096;

struct Levels {
    int lmin;
    double S;
};

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// Lowest and highest level over the workgroup.
__device__ __forceinline__ void level_range(int &lmin, int &lmax)
{
    __shared__ int32_t sh[2][16];
    lmin = wave_fold(lmin, imin);
    lmax = wave_fold(lmax, imax);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = ((int)blockDim.x + 63) >> 6;
    if (lane == 0) {
        sh[0][wave] = lmin;
        sh[1][wave] = lmax;
    }
    __syncthreads();
    lmin = scalar(wave_fold(sh[0][imin(lane, nw - 1)], imin));
    lmax = scalar(wave_fold(sh[1][imin(lane, nw - 1)], imax));
    __syncthreads();
}

// S from the levels of up to 32 rows a thread (lev[i] of row 1024 i + t, -1:
// none), 2048 levels at a time (an aligned subtree of the tree).
__device__ double normaliser_direct(const int (&lev)[32], int groups, int lmin, int nl, const double *pw, double *a)
{
    uint32_t *h = reinterpret_cast<uint32_t *>(a + 3072);
    double *roots = a + 2048;
    int P = 1;
    while (P < nl) P <<= 1;
    const int nchunks = P > 2048 ? P / 2048 : 1;
    const int lane = threadIdx.x & 63;
    double S = 0.0;
    for (int c = 0; c < nchunks; ++c) {
        for (int i = threadIdx.x; i < 2048; i += 1024) h[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (g >= groups) break;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t i = (uint32_t)(lev[8 * g + u] - lmin - 2048 * c);
                bool on = lev[8 * g + u] >= 0 && i < 2048u;
                // the first lane's level in one count: a cold population has
                // hardly another
                const uint64_t m = __ballot(on);
                if (m == 0ull) continue;
                const int lead = __builtin_ctzll(m);
                const uint32_t li = (uint32_t)__builtin_amdgcn_readlane((int)i, lead);
                const uint64_t same = __ballot(on && i == li);
                if (lane == lead)
                    atomicAdd(&h[li], (uint32_t)__builtin_popcountll(same));
                else if (on && i != li)
                    atomicAdd(&h[i], 1u);
            }
        }
        __syncthreads();
        S = tree_sum<1024>(
            nchunks > 1 ? 2048 : P,
            [&](int m) {
                const int l = 2048 * c + m;
                return l < nl ? (double)h[m] * level_weight(pw, (uint32_t)l) : 0.0;
            },
            a, a + 1024);
        if (nchunks > 1) {
            if (threadIdx.x == 0) roots[c] = S;
            __syncthreads();
        }
    }
    return nchunks > 1 ? lds_pairwise(roots, nchunks) : S;
}

__device__ Levels measure_levels(const Inst &I, int k, int buf, int Rk, double *pw, double *a)
{
    // loaded before the pass over the energies so that its latency overlaps it
    const double rho_k = I.rho[k];
    const int N3 = 3 * scalar(I.N), nlev = scalar(I.nlev), copies = scalar(I.hist_copies);
    const bool direct = copies == 0;
    uint32_t *ring = reinterpret_cast<uint32_t *>(a + 2048);
    int lmin = 0x7FFFFFFF, lmax = -1;
    int lev[32];
    const int groups = (Rk + 8191) / 8192;
    // loads eight at a time before any is used: the pass waits for about one
    // memory latency per eight of a thread
    if (direct) {
        const auto E = (__attribute__((address_space(1))) const int32_t *)scalar_ptr(I.E[buf]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (g < groups) {
                int e[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = (8 * g + u) * 1024 + (int)threadIdx.x;
                    e[u] = r < Rk ? E[r] : 0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = (8 * g + u) * 1024 + (int)threadIdx.x;
                    const int l = (e[u] + N3) >> 1;
                    lev[8 * g + u] = r < Rk ? l : -1;
                    lmin = imin(lmin, r < Rk ? l : 0x7FFFFFFF);
                    lmax = imax(lmax, lev[8 * g + u]);
                }
            }
        }
    } else {
        // (the levels' counts stay in LDS, modulo kLevelRing, for the
        // normaliser: a population spreads over far fewer)
        const HistParts parts(I, nlev);
        for (int i = threadIdx.x; i < kLevelRing; i += 1024) ring[i] = 0u;
        __syncthreads();
        for (int m = threadIdx.x; m < nlev; m += 1024) {
            const uint32_t c = parts.count(m, copies);
            if (c) {
                lmin = imin(lmin, m);
                lmax = imax(lmax, m);
                ring[m % kLevelRing] = c;
            }
        }
    }
    if (threadIdx.x == 0) {
        double p = rho_k;
        for (int b = 0; b < kLevelBits; ++b, p = p * p) pw[b] = p;
    }
    level_range(lmin, lmax);
    const int nl = lmax - lmin + 1;
    double S;
    if (direct) {
        S = normaliser_direct(lev, groups, lmin, nl, pw, a);
    } else {
        int P = 1;
        while (P < nl) P <<= 1;
        S = tree_sum<1024>(
            P,
            [&](int m) {
                if (m >= nl) return 0.0;
                const uint32_t h = nl <= kLevelRing ? ring[(lmin + m) % kLevelRing] : HistParts(I, nlev).count(lmin + m, copies);
                return (double)h * level_weight(pw, (uint32_t)m);
            },
            a, a + 1024);
    }
    return Levels{lmin, S};
}

// The energy record of step k: E_min, E_max, sum E and sum E^2 (exact
// integers; with real couplings sum E^2 in 128 bits).
__device__ void measure_real(const Inst &I, int k, int Rk)
{
    __shared__ MomentSum sh[16];
    MomentSum m{-kNoEnergy - 1, 0ull, 0ull, 0ull};
    const BlockMoments *b = block_moments(I);
    for (int i = threadIdx.x; i < (Rk + kRowsPerBlock - 1) / kRowsPerBlock; i += blockDim.x)
        m.add(MomentSum{b[i].emax, b[i].sum, b[i].sq_lo, b[i].sq_hi});
    const long long emin = lowest_energy(I);
    m.reduce(sh);
    if (threadIdx.x == 0) {
        StepRec *rec = I.rec + k;
        rec->R = Rk;
        rec->sumE = (int64_t)m.sum;
        rec->sumE2 = m.lo;
        rec->sumE2_hi = (int64_t)m.hi;
        rec->Emin = emin;
        rec->Emax = m.emax;
        if (k == I.nT - 1) rec->S = __builtin_nan("");
    }
}
__device__ void measure_role(const Inst &I, int k, int buf, int Rk)
{
    __shared__ int64_t sh[2][16];
    if (scalar(I.real)) {
        measure_real(I, k, Rk);
        return;
    }
    const int N3 = 3 * scalar(I.N), nlev = scalar(I.nlev), copies = scalar(I.hist_copies);
    int64_t s1 = 0, s2 = 0;
    int lmin = 0x7FFFFFFF, lmax = -1;
    auto add = [&](int m, int64_t c) {
        const int64_t e = 2 * m - N3;
        s1 += c * e;
        s2 += c * e * e;
        lmin = imin(lmin, m);
        lmax = imax(lmax, m);
    };
    if (copies == 0) {
        const auto E = (__attribute__((address_space(1))) const int32_t *)scalar_ptr(I.E[buf]);
#pragma unroll 8
        for (int r = threadIdx.x; r < Rk; r += 1024) add((E[r] + N3) >> 1, 1);
    } else {
        const HistParts parts(I, nlev);
        for (int m = threadIdx.x; m < nlev; m += 1024) {
            const uint32_t c = parts.count(m, copies);
            if (c) add(m, (int64_t)c);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_xor(s1, off);
        s2 += __shfl_xor(s2, off);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = s1;
        sh[1][threadIdx.x >> 6] = s2;
    }
    level_range(lmin, lmax);
    if (threadIdx.x == 0) {
        for (int i = 1; i < 16; ++i) {
            s1 += sh[0][i];
            s2 += sh[1][i];
        }
        StepRec *rec = I.rec + k;
        rec->R = Rk;
        rec->sumE = s1;
        rec->sumE2 = (uint64_t)s2;
        rec->sumE2_hi = 0;
        rec->Emin = 2 * lmin - N3;
        rec->Emax = 2 * lmax - N3;
        if (k == I.nT - 1) rec->S = __builtin_nan("");
    }
}

// Where the offsets of the resampled rows go: the energy buffer that the next
// sweep will fill (real couplings: memory of their own).
__device__ __forceinline__ uint32_t *row_offsets(const Inst &I, int idle)
{
    return I.real ? I.loff : reinterpret_cast<uint32_t *>(I.E[idle]);
}

// Copy counts of rows [row0, row0 + 1024) and their offsets in the block:
// tau = R' w / S, floor(tau) copies and one more when the row's draw is below
// floor(frac(tau) 2^32).
__device__ void copies_role(const Inst &I, int k, int buf, int Rk, uint32_t row0, uint32_t *sh, double *pw, double *a)
{
    const int r = (int)row0 + (int)threadIdx.x;
    if (k == I.nT - 1) return;
    // (issued before the measurement, whose latency covers it)
    const int E = !I.real && r < Rk ? I.E[buf][r] : 0;
    const uint32_t u = philox10(make_uint4(0u, (uint32_t)r, (uint32_t)k, kTagResample), I.key0, I.key1).x;
    Levels lv{0, 0.0};
    if (I.real)
        lv.S = real_normaliser(I, Rk, a);
    else
        lv = measure_levels(I, k, buf, Rk, pw, a);
    if (row0 == 0 && threadIdx.x == 0) I.rec[k].S = lv.S;
    uint32_t n = 0;
    if (r < Rk) {
        // (real couplings: the row's weight from the weights launch)
        const double w = I.real ? I.wrep[r] : level_weight(pw, (uint32_t)(((E + 3 * I.N) >> 1) - lv.lmin));
        const double tau = (I.Rt[k + 1] * w) / lv.S;
        const double fl = __builtin_floor(tau);
        n = (uint32_t)fl + (u < (uint32_t)__builtin_floor((tau - fl) * 4294967296.0) ? 1u : 0u);
    }
    uint32_t total;
    const uint32_t off = block_exscan(n, sh, &total);
    if (r < I.Rcap) row_offsets(I, buf ^ 1)[r] = off;
    if (threadIdx.x == 0) I.bsum[row0 / kRowsPerBlock] = total;
}

// Pairwise tree of n ln n over family ids [base, base + 2048) (zero for ids
// without descendants and beyond R).  Up to kDirectRows rows (capacity) the
// descendants are counted here from the rows' families, in LDS; beyond, the
// sweep's workgroups have counted them, and the counts are cleared for the
// next step.
__device__ void families_role(const Inst &I, int k, int buf, int Rk, uint32_t base, double *a)
{
    const int n = min(2048, scalar(I.fam_pow2));
    const int t = threadIdx.x;
    uint32_t c[2] = {0u, 0u};
    if (scalar(I.Rcap) <= kDirectRows) {
        uint32_t *cnt = reinterpret_cast<uint32_t *>(a);
        cnt[2 * t] = cnt[2 * t + 1] = 0u;
        const auto fam = (GlobalCounts)scalar_ptr(I.fam[buf]);
        __syncthreads();
        for (int r0 = 0; r0 < Rk; r0 += 8192) {
            uint32_t f[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = r0 + 1024 * u + t;
                f[u] = r < Rk ? fam[r] - base : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (__ballot(f[u] < 2048u)) count_runs(cnt, f[u], f[u] < 2048u);
        }
        __syncthreads();
        c[0] = cnt[2 * t];
        c[1] = cnt[2 * t + 1];
        __syncthreads();
    } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int f = (int)base + 2 * t + j;
            if (2 * t + j < n && f < I.R) {
                c[j] = I.cnt[f];
                I.cnt[f] = 0u;
            }
        }
    }
    double l[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (2 * t + j < n && (int)base + 2 * t + j < I.R) l[j] = I.nlnn[c[j]];
    const double s = wg_tree(n >= 2 ? l[0] + l[1] : l[0], n >= 2 ? n / 2 : 1, a);
    if (threadIdx.x == 0) {
        if (I.fam_pow2 <= 2048)
            I.rec[k].T = s;
        else
            I.fpart[base / 2048] = s;
    }
}

// Overlap histogram: row r pairs with r + floor(R_k / 2); this workgroup
// takes the kOvlPairs pairs from row p0.  Spins are 0/1 bytes, so the number
// of differing sites is the popcount of the XOR.  A pair is read by a group
// of lanes sized to its row (16-byte loads), several pairs per wave for
// short rows.  Low temperatures put most pairs into a few bins, so the
// counts go to an LDS histogram first and only its non-empty bins reach
// global memory.
__device__ void overlap_role(const Inst &I, int k, int buf, int Rk, uint32_t p0, uint32_t *qh)
{
    const int slot = I.ovl_slot[k];
    if (slot < 0) return;
    const int h = Rk / 2;
    if ((int)p0 >= h) return;
    const int npairs = min(kOvlPairs, h - (int)p0);
    const int nb = 2 * I.N + 1;
    uint32_t *gh = I.qhist + (size_t)slot * nb;
    const bool local = nb <= kOvlLdsBins;
    if (local) {
        for (int i = threadIdx.x; i < nb; i += blockDim.x) qh[i] = 0u;
        __syncthreads();
    }
    const uint8_t *sp = I.spins[buf];
    // 16-byte words of a stored row: bytes 0/1, or bits (both count the
    // differing sites as the popcount of the XOR)
    const int words = I.srow_bytes >> 4;
    int lpp = 1;  // lanes per pair, a power of two <= 64
    while (lpp < words && lpp < 64) lpp <<= 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int sub = lane / lpp, j = lane & (lpp - 1), ppw = 64 / lpp;
    for (int q0 = wave * ppw; q0 < npairs; q0 += nw * ppw) {
        const int q = q0 + sub;
        int diff = 0;
        if (q < npairs) {
            const int r = (int)p0 + q;
            const uint4 *a = reinterpret_cast<const uint4 *>(sp + (size_t)r * I.srow_bytes);
            const uint4 *b = reinterpret_cast<const uint4 *>(sp + (size_t)(r + h) * I.srow_bytes);
            for (int i = j; i < words; i += lpp) {
                const uint4 x = a[i], y = b[i];
                diff += __builtin_popcount(x.x ^ y.x) + __builtin_popcount(x.y ^ y.y) +
                        __builtin_popcount(x.z ^ y.z) + __builtin_popcount(x.w ^ y.w);
            }
        }
        for (int off = lpp >> 1; off > 0; off >>= 1) diff += __shfl_xor(diff, off);
        if (q < npairs && j == 0) {
            const int bin = (I.N - 2 * diff) + I.N;
            if (local)
                atomicAdd(&qh[bin], 1u);
            else
                atomicAdd(&gh[bin], 1u);
        }
    }
    if (local) {
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += blockDim.x) {
            const uint32_t c = qh[i];
            if (c) atomicAdd(&gh[i], c);
        }
    }
}

__device__ __forceinline__ void clear_lowest(const Inst &I)
{
    if ((int)threadIdx.x < kMinParts) I.emin[threadIdx.x] = kNoEnergy;
}
// What the last workgroup needs of the descriptor, read before the election:
// its acquire empties the L2 of everything, and each read behind it is a trip
// to memory (a chain of three took 5 us).
struct PostEnd {
    int nT, Rcap, real, fam_pow2;
    const uint32_t *loff, *bsum;
    uint32_t *boff, *map, *Rk;
    const double *fpart;
    int32_t *ctl;
};
__device__ __forceinline__ PostEnd post_end(const Inst &I, int buf)
{
    return PostEnd{scalar(I.nT),           scalar(I.Rcap),      scalar(I.real),     scalar(I.fam_pow2),
                   scalar_ptr(row_offsets(I, buf ^ 1)), scalar_ptr(I.bsum),  scalar_ptr(I.boff), scalar_ptr(I.map),
                   scalar_ptr(I.Rk),       scalar_ptr(I.fpart), scalar_ptr(I.k)};
}

// The map of a population of at most kMapRows rows, by one workgroup: every
// row's offset in LDS, four destinations a thread (see k_expand, whose launch
// takes 5 us).  Returns R_{k+1}; no map if that exceeds the capacity.
__device__ uint32_t expand_small(const PostEnd &p, int Rold, uint32_t *off)
{
    constexpr int B = kMapRows / kRowsPerBlock;
    const int nb = (Rold + kRowsPerBlock - 1) / kRowsPerBlock;
    uint32_t l[B], sum[B], total = 0;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int r = b * kRowsPerBlock + (int)threadIdx.x;
        l[b] = r < Rold ? p.loff[r] : 0u;
        sum[b] = b < nb ? p.bsum[b] : 0u;
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if (b < nb) off[b * kRowsPerBlock + (int)threadIdx.x] = total + l[b];
        total += scalar(sum[b]);
    }
    __syncthreads();
    if (total > (uint32_t)p.Rcap) return total;
    int first = 1;
    while (2 * first < Rold) first *= 2;
    for (uint32_t j = threadIdx.x; j < total; j += kRowsPerBlock) {
        int q = 0;  // off[0] = 0 <= j
        for (int step = first; step > 0; step >>= 1)
            if (q + step < Rold && off[q + step] <= j) q += step;
        p.map[j] = (uint32_t)q;
    }
    return total;
}

// Last workgroup of an instance in a post launch.
__device__ void post_finish(const Inst &I, const PostEnd &p, int k, int buf, int Rk, uint32_t *sh, double *a)
{
    const bool resample = k < p.nT - 1;
    bool ok = true;
    if (resample) {
        const int nb = (Rk + kRowsPerBlock - 1) / kRowsPerBlock;
        uint64_t carry = 0;
        if (p.Rcap <= kMapRows) {
            carry = expand_small(p, Rk, reinterpret_cast<uint32_t *>(a));
            if (p.real) clear_lowest(I);
        } else if (nb <= 64) {
            // (every wave: no barrier)
            const int b = (int)threadIdx.x & 63;
            const uint32_t v = b < nb ? p.bsum[b] : 0u, x = wave_scan(v);
            if ((int)threadIdx.x < nb) p.boff[b] = x - v;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        } else {
            for (int b0 = 0; b0 < nb; b0 += blockDim.x) {
                const int b = b0 + (int)threadIdx.x;
                const uint32_t v = b < nb ? p.bsum[b] : 0u;
                uint32_t total;
                const uint32_t off = block_exscan(v, sh, &total);
                if (b < nb) p.boff[b] = (uint32_t)(carry + off);
                carry += total;
            }
        }
        ok = carry > 0 && carry <= (uint64_t)p.Rcap;
        if (threadIdx.x == 0) {
            p.Rk[k + 1] = carry > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)carry;
            if (!ok) {
                I.status[1] = (uint32_t)k;
                I.status[0] |= carry == 0 ? 2u : 1u;
            }
        }
    }
    if (p.fam_pow2 > 2048) {
        __syncthreads();
        const int n = p.fam_pow2 / 2048;  // power of two
        const double s = tree_sum<1024>(n, [&](int i) { return p.fpart[i]; }, a, a + 1024);
        if (threadIdx.x == 0) I.rec[k].T = s;
    }
    if (threadIdx.x == 0) {
        // the population of step k lies where its sweeps left it; rows of the
        // next step live there through the copy map
        p.ctl[1] = buf;
        p.ctl[2] = ok && resample ? 1 : 0;
        if (ok) p.ctl[0] = k + 1;
    }
}

__global__ __launch_bounds__(1024) void k_post(const Inst *insts, const Work *work)
{
    __shared__ uint32_t sh[17];
    __shared__ double pw[40];
    // pairwise-tree scratch, or the LDS overlap histogram
    __shared__ double a[kOvlLdsBins / 2 + 1];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    // (k, cur and mapped in one read)
    const int4 ctl = *reinterpret_cast<const int4 *>(I.k);
    const uint32_t status = I.status[0];
    const int k = scalar(ctl.x), buf = scalar(ctl.y ^ ctl.z);
    if (k >= scalar(I.nT) || scalar(status) != 0u) return;
    const int Rk = (int)scalar(I.Rk[k]);
    const uint32_t row0 = scalar(w.row0), role = scalar(w.role);
    const PostEnd end = post_end(I, buf);
    const int expected = scalar(I.post_blocks);
    uint32_t *const count = scalar_ptr(&I.sync[1]);
    if (role == kRoleCopies) {
        copies_role(I, k, buf, Rk, row0, sh, pw, a);
    } else if (role == kRoleMeasure) {
        measure_role(I, k, buf, Rk);
    } else if (role == kRoleFamilies) {
        families_role(I, k, buf, Rk, row0, a);
    } else {
        overlap_role(I, k, buf, Rk, row0, reinterpret_cast<uint32_t *>(a));
    }
    if (last_workgroup(count, expected)) post_finish(I, end, k, buf, Rk, sh, a);
}

// Copy map of the resampling of step k - 1 (the step index has advanced), more
// than kMapRows rows: source row r owns destination rows [off_r, off_r + n_r).  A few rows can
// own thousands of copies when the temperature step is large, so the
// workgroup of a row block walks the block's destinations instead of its
// rows: destination j belongs to the last row whose local offset is <= j.
__global__ __launch_bounds__(1024) void k_expand(const Inst *insts, const Work *work)
{
    __shared__ uint32_t off[kRowsPerBlock];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = *I.k;
    if (!inst_live(I, k) || k == 0 || !*I.mapped) return;
    const int Rold = (int)I.Rk[k - 1];
    const int row0 = (int)w.row0;
    if (I.real && row0 == 0) clear_lowest(I);
    if (!I.real && I.hist_copies > 0) {
        // every copies workgroup has measured the step: the nblk workgroups
        // clear its energy histogram for the next sweep, a slice each
        const int slice = (int)((int64_t)I.hist_copies * I.nlev + I.nblk - 1) / I.nblk;
        const int first = (row0 / kRowsPerBlock) * slice, last = min(I.hist_copies * I.nlev, first + slice);
        for (int i = first + (int)threadIdx.x; i < last; i += blockDim.x) {
            if (i < I.nlev)
                I.hist[i] = 0u;
            else
                I.loff[i - I.nlev] = 0u;
        }
    }
    if (row0 >= Rold) return;
    const int nrow = min(kRowsPerBlock, Rold - row0);
    const uint32_t total = I.bsum[row0 / kRowsPerBlock];
    const uint32_t base = I.boff[row0 / kRowsPerBlock];
    if (total == 0u) return;
    // (the step has moved on: cur is the buffer of the rows being copied)
    const uint32_t *loff = row_offsets(I, *I.cur ^ 1);
    for (int t = threadIdx.x; t < nrow; t += blockDim.x) off[t] = loff[row0 + t];
    __syncthreads();
    const uint32_t lim = (uint32_t)I.Rcap - min(base, (uint32_t)I.Rcap);
    const uint32_t end = min(total, lim);
    for (uint32_t j = threadIdx.x; j < end; j += blockDim.x) {
        int p = 0;  // off[0] = 0 <= j
        for (int step = kRowsPerBlock / 2; step > 0; step >>= 1)
            if (p + step < nrow && off[p + step] <= j) p += step;
        I.map[base + j] = (uint32_t)(row0 + p);
    }
}

// After a stand-alone gather the population lives in the other buffer.
__global__ void k_flip(const Inst *insts, const uint32_t *list)
{
    const Inst &I = insts[list[blockIdx.x]];
    const int k = *I.k;
    if (threadIdx.x == 0 && inst_live(I, k) && *I.mapped) {
        *I.cur ^= 1;
        *I.mapped = 0;
    }
}

// ---------------------------------------------------------------------------
void launch_weights(const Inst *insts, const Work *work, int nwork, hipStream_t st)
{
    if (nwork) k_weights<<<nwork, 512, 0, st>>>(insts, work);
}
void launch_post(const Inst *insts, const Work *work, int nwork, hipStream_t st)
{
    if (nwork) k_post<<<nwork, 1024, 0, st>>>(insts, work);
}
void launch_expand(const Inst *insts, const Work *work, int nwork, hipStream_t st)
{
    if (nwork) k_expand<<<nwork, 1024, 0, st>>>(insts, work);
}
void launch_flip(const Inst *insts, const uint32_t *list, int n, hipStream_t st)
{
    if (n) k_flip<<<n, 64, 0, st>>>(insts, list);
}

}  // namespace pamc
