// resample.hip -- resampling and the per-step statistics (paper Sec. II.B,
// Eq. (2), Sec. V.A) for gfx950.
//
// After the sweeps, one post launch runs three kinds of workgroups per
// instance:
//   copies    measures the step (energy sums, normaliser) and takes
//             n_r = floor(tau) + [u_r < frac(tau) 2^32] for 1024 rows, with
//             their exclusive scan inside the workgroup;
//   families  n ln n of 2048 family ids, summed by the pairwise tree;
//   overlap   spin overlaps of 2048 replica pairs (at overlap steps).
// The last workgroup of an instance to finish scans the per-workgroup
// totals into offsets, sets R_{k+1} and the capacity / extinction status,
// folds the family partial sums, and advances the step.  An expand launch
// then writes the copy map (destination row -> source row, stable order),
// which the next sweep reads its tile through, and clears the step's energy
// histogram.
#include "launch.h"
#include "pamc_dev.h"
#include "step_common.h"

namespace pamc {

// The moments of a step with real couplings from their parts, by a wave
// (lane = part); every lane returns them.
struct Moments {
    long long emin, emax;
    unsigned long long sum, lo, hi;
};
__device__ __forceinline__ Moments fold_moments(const EMoments *parts)
{
    static_assert(kMomentParts == 64, "one part per lane");
    const EMoments &p = parts[threadIdx.x & 63];
    Moments m{p.emin, p.emax, p.sum, p.sq_lo, p.sq_hi};
    for (int off = 32; off > 0; off >>= 1) {
        const long long a = __shfl_xor(m.emin, off), b = __shfl_xor(m.emax, off);
        const unsigned long long s = __shfl_xor(m.sum, off), l = __shfl_xor(m.lo, off), h = __shfl_xor(m.hi, off);
        m.emin = a < m.emin ? a : m.emin;
        m.emax = b > m.emax ? b : m.emax;
        m.sum += s;
        const unsigned long long nl = m.lo + l;
        m.hi += h + (nl < m.lo ? 1ull : 0ull);
        m.lo = nl;
    }
    return m;
}

// Resampling weights with real couplings (Sec. II.B), for rows
// [row0, row0 + 1024) of one instance after the sweeps of step k:
// w_r = exp(-dbeta (E_r - E_min)) as the product over the set bits b of
// E_r - E_min (units of 2^-20) of exp(-dbeta 2^(b-20)), in ascending b.  The
// block's 1024 leaves (zero beyond R_k) form an aligned subtree of the
// pairwise tree over rows 0 .. P-1 (P the smallest power of two >= R_k); the
// copies workgroups fold the block roots (real_normaliser).  For P < 1024 the
// block tree adds only zeros above the P-leaf subtree, which leaves its sum
// unchanged.  The instance's first workgroup writes the step's energy record.
__global__ __launch_bounds__(512) void k_weights(const Inst *insts, const Work *work)
{
    __shared__ double pw[40];
    __shared__ double a[512];
    __shared__ Moments sh;
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = *I.k;
    if (!inst_live(I, k)) return;
    const bool resample = k < I.nT - 1;
    if (!resample && w.row0 != 0) return;
    const int Rk = (int)I.Rk[k];
    const int t = threadIdx.x;
    if (resample && t < 40) pw[t] = I.gpw[(size_t)k * 40 + t];
    if (t < 64) {
        const Moments m = fold_moments(I.emom);
        if (t == 0) sh = m;
    }
    const int64_t *E = I.Eq[swept_buffer(I)];
    int64_t e[2] = {0, 0};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = (int)w.row0 + 2 * t + j;
        if (resample && r < Rk) e[j] = E[r];
    }
    __syncthreads();
    if (w.row0 == 0 && t == 0) {
        StepRec *rec = I.rec + k;
        rec->R = Rk;
        rec->sumE = (int64_t)sh.sum;
        rec->sumE2 = sh.lo;
        rec->sumE2_hi = (int64_t)sh.hi;
        rec->Emin = sh.emin;
        rec->Emax = sh.emax;
        rec->S = __builtin_nan("");
    }
    if (!resample) return;
    double l[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = (int)w.row0 + 2 * t + j;
        if (r < Rk) {
            const double x = weight64(pw, (uint64_t)(e[j] - sh.emin));
            I.wrep[r] = x;
            l[j] = x;
        }
    }
    a[t] = l[0] + l[1];
    __syncthreads();
    const double root = lds_pairwise(a, 512);
    if (t == 0) I.wpart[w.row0 / kRowsPerBlock] = root;
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

// Exclusive scan over the workgroup (1024 threads, 16 waves).
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t *sh, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        const int nw = blockDim.x >> 6;
        for (int i = 0; i < nw; ++i) {
            const uint32_t t = sh[i];
            sh[i] = acc;
            acc += t;
        }
        sh[16] = acc;
    }
    __syncthreads();
    *total = sh[16];
    const uint32_t r = sh[wave] + x - v;
    __syncthreads();
    return r;
}

// Measurement of step k after its sweeps with +-1 couplings, by a workgroup of
// 1024 threads: E_min, E_max, sum E, sum E^2 (exact integers; written to the
// step's record by `writer`), and for k < nT-1 the level weights
// w[m] = exp(-2 dbeta m) as a fixed product of rho^(2^b) and their normaliser
// S by the pairwise tree over 2^ceil(log2(M+1)) levels.  Every copies
// workgroup measures for itself: its pass over the energies or the histogram
// comes out of the L2 (12 loads a thread at L = 8), where one workgroup at the
// end of the sweep launch kept the whole chip waiting (64 threads at L = 8:
// about 25 us a step) and every other one had to count itself in.
//   Up to kDirectRows rows: the energies themselves, 32 a thread, with the
// histogram built in LDS (a sweep launch then counts nothing: its atomics on
// the few energies of a cold population follow each other about 0.1 us apart
// on each address, 15-50 us a launch at 10^4 rows).
//   Beyond: the histogram that the sweep's workgroups have counted.
// pw: 40 doubles, a: 4096 doubles, of LDS.
struct Levels {
    int lmin;
    double S;
};

struct LevelSums {
    int64_t s1, s2;
    int32_t lmin, lmax;
    __device__ __forceinline__ void add(int m, int64_t c, int N3)
    {
        const int64_t e = 2 * m - N3;
        s1 += c * e;
        s2 += c * e * e;
        lmin = min(lmin, m);
        lmax = max(lmax, m);
    }
    // over the workgroup (two barriers inside)
    __device__ __forceinline__ void reduce()
    {
        __shared__ int64_t sh64[2][16];
        __shared__ int32_t sh32[2][16];
        for (int off = 32; off > 0; off >>= 1) {
            s1 += __shfl_xor(s1, off);
            s2 += __shfl_xor(s2, off);
            lmin = min(lmin, __shfl_xor(lmin, off));
            lmax = max(lmax, __shfl_xor(lmax, off));
        }
        const int wave = threadIdx.x >> 6, nw = ((int)blockDim.x + 63) >> 6;
        if ((threadIdx.x & 63) == 0) {
            sh64[0][wave] = s1;
            sh64[1][wave] = s2;
            sh32[0][wave] = lmin;
            sh32[1][wave] = lmax;
        }
        __syncthreads();
        s1 = sh64[0][0];
        s2 = sh64[1][0];
        lmin = sh32[0][0];
        lmax = sh32[1][0];
        for (int i = 1; i < nw; ++i) {
            s1 += sh64[0][i];
            s2 += sh64[1][i];
            lmin = min(lmin, sh32[0][i]);
            lmax = max(lmax, sh32[1][i]);
        }
        __syncthreads();
    }
};

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

__device__ Levels measure_levels(const Inst &I, int k, int buf, bool writer, double *pw, double *a)
{
    const bool resample = k < I.nT - 1;
    // loaded before the pass over the energies so that its latency overlaps it
    const double rho_k = resample ? I.rho[k] : 1.0;
    const int N3 = 3 * I.N, nlev = I.nlev, copies = I.hist_copies, Rk = (int)I.Rk[k];
    const bool direct = copies == 0;
    LevelSums s{0, 0, 0x7FFFFFFF, -1};
    int lev[32];
    const int groups = (Rk + 8191) / 8192;
    if (threadIdx.x == 0) {
        pw[0] = rho_k;
        for (int b = 1; b < 40; ++b) pw[b] = pw[b - 1] * pw[b - 1];
    }
    // loads eight at a time before any is used: the pass waits for about one
    // memory latency per eight of a thread
    if (direct) {
        const int32_t *E = I.E[buf];
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
                    lev[8 * g + u] = r < Rk ? (e[u] + N3) >> 1 : -1;
                    if (r < Rk) s.add(lev[8 * g + u], 1, N3);
                }
            }
        }
    } else {
        for (int base = threadIdx.x; base < nlev; base += 8 * 1024) {
            uint32_t c[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
            for (int p = 0; p < copies; ++p) {
                const uint32_t *hp = hist_copy(I, p);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int m = base + u * 1024;
                    c[u] += m < nlev ? hp[m] : 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (c[u]) s.add(base + u * 1024, (int64_t)c[u], N3);
        }
    }
    s.reduce();
    double S = __builtin_nan("");
    if (resample) {
        const int lmin = s.lmin, nl = s.lmax - s.lmin + 1;
        if (direct) {
            S = normaliser_direct(lev, groups, lmin, nl, pw, a);
        } else {
            int P = 1;
            while (P < nl) P <<= 1;
            S = tree_sum<1024>(
                P,
                [&](int m) {
                    if (m >= nl) return 0.0;
                    uint32_t h = 0;
                    for (int p = 0; p < copies; ++p) h += hist_copy(I, p)[lmin + m];
                    return (double)h * level_weight(pw, (uint32_t)m);
                },
                a, a + 1024);
        }
    }
    if (writer && threadIdx.x == 0) {
        StepRec *rec = I.rec + k;
        rec->R = Rk;
        rec->sumE = s.s1;
        rec->sumE2 = (uint64_t)s.s2;
        rec->sumE2_hi = 0;
        rec->Emin = 2 * s.lmin - N3;
        rec->Emax = 2 * s.lmax - N3;
        rec->S = S;
    }
    __syncthreads();
    return Levels{s.lmin, S};
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
__device__ void copies_role(const Inst &I, int k, uint32_t row0, uint32_t *sh, double *pw, double *a)
{
    const int buf = swept_buffer(I);
    const int Rk = (int)I.Rk[k];
    const int r = (int)row0 + (int)threadIdx.x;
    const bool resample = k < I.nT - 1;
    Levels lv{0, 0.0};
    // (issued before the measurement, whose latency covers it)
    const int E = !I.real && resample && r < Rk ? I.E[buf][r] : 0;
    if (!I.real && (resample || row0 == 0)) lv = measure_levels(I, k, buf, row0 == 0, pw, a);
    if (!resample) return;
    if (I.real) {
        lv.S = real_normaliser(I, Rk, a);
        if (row0 == 0 && threadIdx.x == 0) I.rec[k].S = lv.S;
    }
    uint32_t n = 0;
    if (r < Rk) {
        const uint32_t u = philox10(make_uint4(0u, (uint32_t)r, (uint32_t)k, kTagResample), I.key0, I.key1).x;
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
// without descendants and beyond R); the counts are cleared for the next
// step.
__device__ void families_role(const Inst &I, int k, uint32_t base, double *a)
{
    const int n = min(2048, I.fam_pow2);
    const int t = threadIdx.x;
    double v = 0.0;
    if (2 * t < n) {
        const int f0 = (int)base + 2 * t, f1 = f0 + 1;
        double l0 = 0.0, l1 = 0.0;
        if (f0 < I.R) {
            l0 = I.nlnn[I.cnt[f0]];
            I.cnt[f0] = 0u;
        }
        if (n >= 2 && f1 < I.R) {
            l1 = I.nlnn[I.cnt[f1]];
            I.cnt[f1] = 0u;
        }
        v = n >= 2 ? l0 + l1 : l0;
    }
    a[t] = v;
    __syncthreads();
    const double s = lds_pairwise(a, n >= 2 ? n / 2 : 1);
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
__device__ void overlap_role(const Inst &I, int k, uint32_t p0, uint32_t *qh)
{
    const int slot = I.ovl_slot[k];
    if (slot < 0) return;
    const int h = (int)I.Rk[k] / 2;
    if ((int)p0 >= h) return;
    const int npairs = min(kOvlPairs, h - (int)p0);
    const int nb = 2 * I.N + 1;
    uint32_t *gh = I.qhist + (size_t)slot * nb;
    const bool local = nb <= kOvlLdsBins;
    if (local) {
        for (int i = threadIdx.x; i < nb; i += blockDim.x) qh[i] = 0u;
        __syncthreads();
    }
    const uint8_t *sp = I.spins[swept_buffer(I)];
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

// Last workgroup of an instance in a post launch.
__device__ void post_finish(const Inst &I, int k, uint32_t *sh, double *a)
{
    if (I.fam_pow2 > 2048) {
        const int n = I.fam_pow2 / 2048;  // power of two
        const double s = tree_sum<1024>(n, [&](int i) { return I.fpart[i]; }, a, a + 1024);
        if (threadIdx.x == 0) I.rec[k].T = s;
    }
    bool ok = true;
    if (k < I.nT - 1) {
        const int nb = ((int)I.Rk[k] + kRowsPerBlock - 1) / kRowsPerBlock;
        uint64_t carry = 0;
        for (int b0 = 0; b0 < nb; b0 += blockDim.x) {
            const int b = b0 + (int)threadIdx.x;
            const uint32_t v = b < nb ? I.bsum[b] : 0u;
            uint32_t total;
            const uint32_t off = block_exscan(v, sh, &total);
            if (b < nb) I.boff[b] = (uint32_t)(carry + off);
            carry += total;
        }
        ok = carry > 0 && carry <= (uint64_t)I.Rcap;
        if (threadIdx.x == 0) {
            I.Rk[k + 1] = carry > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)carry;
            if (!ok) {
                I.status[1] = (uint32_t)k;
                I.status[0] |= carry == 0 ? 2u : 1u;
            }
        }
    }
    if (threadIdx.x == 0) {
        // the population of step k lies where its sweeps left it; rows of the
        // next step live there through the copy map
        *I.cur = swept_buffer(I);
        *I.mapped = ok && k < I.nT - 1 ? 1 : 0;
        if (ok) *I.k = k + 1;
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
    const int k = *I.k;
    if (!inst_live(I, k)) return;
    if (w.role == kRoleCopies) {
        copies_role(I, k, w.row0, sh, pw, a);
    } else if (w.role == kRoleFamilies) {
        families_role(I, k, w.row0, a);
    } else {
        overlap_role(I, k, w.row0, reinterpret_cast<uint32_t *>(a));
    }
    if (last_workgroup(&I.sync[1], I.post_blocks)) post_finish(I, k, sh, a);
}

// Copy map of the resampling of step k - 1 (the step index has advanced):
// source row r owns destination rows [off_r, off_r + n_r).  A few rows can
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
    if (I.real && row0 == 0 && threadIdx.x < kMomentParts) {
        EMoments *m = I.emom + threadIdx.x;
        m->emin = 0x7FFFFFFFFFFFFFFFll;
        m->emax = -0x7FFFFFFFFFFFFFFFll - 1;
        m->sum = 0ull;
        m->sq_lo = 0ull;
        m->sq_hi = 0ull;
    }
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
