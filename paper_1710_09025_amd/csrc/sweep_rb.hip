// sweep_rb.hip -- Metropolis sweeps with +-1 couplings (paper Sec. II.B and
// Sec. III.A) for gfx950: replicas as bits of a word, every lattice size.
//
// Up to 32 replicas (m of them: the rows of a "set") share an LDS word per
// lattice site, bit j the spin of the j-th.  A lane takes Philox block g of a
// colour (four sites) of one set and draws for the m replicas one after
// another.  The local fields of the four sites in all replicas are bit-sliced
// sums of six words (own ^ neighbour ^ [J = -1]), so they cost the lane the
// same number of instructions whatever m is; what is left per attempt is the
// draw and the comparison with the threshold.
//
// What bounds it: instruction issue.  On this chip nearly every VALU
// instruction, v_mad_u64_u32 included, takes a wave 4.4-5.3 cycles of its
// SIMD (2.7-3.8 for XORs and adds with four or more waves resident), so the
// count of instructions per attempt is what matters:
//   draw       rounds 1 and 2 and half of round 3 of Philox4x32-10 depend on
//              (block, sweep) alone or on (replica) alone: computed once per
//              lane and colour step, or on the scalar unit where a wave
//              holds a single set (UNI); 15 multiplies and 17 XORs are left
//              per draw of four words, 8 instructions per attempt;
//   fields     about 150 instructions for 4 m attempts;
//   decision   mode kTable: the threshold by n read from LDS, compared, the
//              result shifted into the flip word: 3.5 per attempt.  Where
//              even the threshold for dE = 8 (kMid) or dE = 4 (kRare) is so
//              low that hardly any draw falls below it, the minimum of eight
//              words is compared once and the exact decision made only where
//              a lane of the wave needs it, 0.6 per attempt; kMid compares
//              every draw with the threshold for dE = 4 besides (2).
#include <algorithm>

#include "launch.h"
#include "pamc_dev.h"
#include "rb_common.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

namespace {

enum RBMode { kAll = 0, kTable = 1, kMid = 2, kRare = 3 };

// Up to this value a threshold is left to the check of the minimum: eight
// words in 64 lanes then call for exact decisions in at most 12% of the
// checks (512 draws, 2^20 / 2^32 each), where they cost about as much as
// the threshold reads and compares of those eight words would.
constexpr uint32_t kRareT = 1u << 20;

// Bit-sliced number of unsatisfied bonds of the four sites of a block in the
// replicas of a set: n = b0 + 2 b1 + 4 b2 per replica.
struct Fields {
    uint32_t own[4], b0[4], b1[4], b2[4], dn[4];  // dn: n >= 3
};

__device__ __forceinline__ void block_fields(const uint32_t *lds, const Record &rec, int own, int plane, Fields &f,
                                             uint32_t &valid)
{
    const u32x4 q0 = rec.q[0], q1 = rec.q[1], q2 = rec.q[2], q3 = rec.q[3];
    const uint32_t e[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
    valid = q3.y;
    uint32_t nb[24];
#pragma unroll
    for (int d = 0; d < 6; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = e[2 * d + (i >> 1)];
            nb[4 * d + i] = lds[(i & 1) ? w >> 16 : w & 0xFFFFu];
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) f.own[i] = lds[own + i * plane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t x[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            // [J = -1] as a full word
            const uint32_t j = (uint32_t)(((int32_t)(q3.x << (31 - (4 * d + i)))) >> 31);
            x[d] = xor3(f.own[i], nb[4 * d + i], j);
        }
        const uint32_t s1 = xor3(x[0], x[1], x[2]), c1 = maj(x[0], x[1], x[2]);
        const uint32_t s2 = xor3(x[3], x[4], x[5]), c2 = maj(x[3], x[4], x[5]);
        const uint32_t c3 = s1 & s2;
        f.b0[i] = s1 ^ s2;
        f.b1[i] = xor3(c1, c2, c3);
        f.b2[i] = maj(c1, c2, c3);
        f.dn[i] = f.b2[i] | (f.b1[i] & f.b0[i]);
    }
}

// One colour step of block g for the m replicas from row rb on (bits past the
// m-th, and rows past the population, hold whatever comes: never stored).
// Lanes without a block (has = false) go along and write nothing.
template <bool UNI, int MODE>
__device__ __forceinline__ void rb_block(const RBInst &X, uint32_t *lds, const uint32_t *tab, uint4 th, int c, int g,
                                         bool has, uint32_t rb, int m, int k, int t, Record &rec, int next_c, int next_g)
{
    const int plane = X.plane, own = pick3(X.base, c) + g;
    const uint32_t k0 = X.k0, k1 = X.k1, ctr = ((uint32_t)c << 24) | (uint32_t)g;
    Fields f;
    uint32_t valid;
    block_fields(lds, rec, own, plane, f, valid);
    // the next block's record is on its way while this one draws
    rec = load_record(X, next_c, next_g);
    uint32_t acc[4] = {0u, 0u, 0u, 0u};
    if constexpr (MODE == kTable) {
        const LaneDraw d = lane_draw(ctr, k, t, k0, k1);
        const uint8_t *tb = reinterpret_cast<const uint8_t *>(tab);
        if (m >= 4) {
            // 4 n (n modulo 4) of replica 4 j + q of site i in nibble j of
            // w[i][q]: the byte offset of its threshold
            uint32_t w[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t l = q < 2 ? f.b0[i] << (2 - q) : f.b0[i] >> (q - 2);
                    const uint32_t h = f.b1[i] << (3 - q);
                    w[i][q] = (l & 0x44444444u) | (h & 0x88888888u);
                }
#pragma unroll 1
            for (int j = (m + 3) / 4 - 1; j >= 0; --j) {
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    uint32_t thr[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        thr[i] = *reinterpret_cast<const uint32_t *>(tb + __builtin_amdgcn_ubfe(w[i][q], 4 * j, 4));
                    const uint4 u = replica_draw<UNI>(d, rb + (uint32_t)(4 * j + q), k, k0, k1);
                    push_lt(acc[0], u.x, thr[0]);
                    push_lt(acc[1], u.y, thr[1]);
                    push_lt(acc[2], u.z, thr[2]);
                    push_lt(acc[3], u.w, thr[3]);
                }
            }
        } else {
            for (int j = m - 1; j >= 0; --j) {
                const uint4 u = replica_draw<UNI>(d, rb + (uint32_t)j, k, k0, k1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t n = __builtin_amdgcn_ubfe(f.b0[i], j, 1) | (__builtin_amdgcn_ubfe(f.b1[i], j, 1) << 1);
                    push_lt(acc[i], word_of(u, i), tab[n]);
                }
            }
        }
    } else if constexpr (MODE == kMid || MODE == kRare) {
        // the flips of n <= LOW + 1 unsatisfied bonds are rare
        const LaneDraw d = lane_draw(ctr, k, t, k0, k1);
        const uint32_t low = MODE == kMid ? th.y : th.x;
        uint32_t up[4] = {0u, 0u, 0u, 0u};  // kMid: [u < T(dE = 4)]
#pragma unroll 2
        for (int j = (m - 1) & ~1; j >= 0; j -= 2) {
            uint4 u[2];
            uint32_t mn = 0xFFFFFFFFu;
#pragma unroll
            for (int p = 1; p >= 0; --p) {
                u[p] = replica_draw<UNI>(d, rb + (uint32_t)(j + p), k, k0, k1);
                mn = min(min(min(min(mn, u[p].x), u[p].y), u[p].z), u[p].w);
                if constexpr (MODE == kMid) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) push_lt(up[i], word_of(u[p], i), th.x);
                }
            }
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(mn < low) != 0ull, 0)) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t l = (f.b0[i] >> (j + p)) & 1u, h = (f.b1[i] >> (j + p)) & 1u;
                        const uint32_t T0 = h ? th.x : l ? th.y : th.z;
                        acc[i] |= (word_of(u[p], i) < T0 ? 1u : 0u) << (j + p);
                    }
            }
        }
        if constexpr (MODE == kMid) {
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] |= up[i] & f.b1[i];  // n = 2 (and 3, which flips anyway)
        }
    }
    const bool whole = __builtin_amdgcn_ballot_w64(has && valid != 15u) == 0ull;
    if (!has) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // n >= 3 (dE <= 0) always flips
        const uint32_t flip = MODE == kAll ? 0xFFFFFFFFu : f.dn[i] | acc[i];
        if (whole || ((valid >> i) & 1u)) lds[own + i * plane] = f.own[i] ^ flip;
    }
}

// UNI: one set per workgroup, so the replica index is uniform; else the
// blocks of all sets are dealt out to the threads in order.
template <bool UNI, int MODE>
__device__ __forceinline__ void rb_sweeps(const RBInst &X, int k, uint32_t *lds, const uint32_t *tab, uint4 th, int r0,
                                          int m, int sets, int t0, int t1, int tid, bool even)
{
    const bool local = UNI && blockDim.x == 64;
    int set = 0, g0 = tid, step = (int)blockDim.x;
    if constexpr (!UNI) {
        set = tid / X.gmax;
        g0 = tid - set * X.gmax;
        step = X.gmax;
    }
    const bool act = UNI || set < sets;
    uint32_t *sp = UNI ? lds : lds + (act ? set : 0) * 4 * X.plane;
    const uint32_t rb = (uint32_t)(UNI ? r0 : r0 + set * m);
    const int last = X.gmax - 1;  // (records past a colour's blocks are zeros)
    const int wave0 = UNI ? scalar(tid & ~63) : 0;
    Record rec = load_record(X, 0, min(g0, last));
    for (int t = t0; t < t1; ++t) {
        if (even) even_progress(t, t0, t1);
        for (int c = 0; c < X.ncol; ++c) {
            const int nc = c + 1 < X.ncol ? c + 1 : 0;
            // (UNI: a wave past the last block draws nothing)
            for (int first = 0; wave0 + first <= last; first += step) {
                const int g = g0 + first;
                const bool more = wave0 + first + step <= last;
                rb_block<UNI, MODE>(X, sp, tab, th, c, min(g, last), act && g < pick3(X.gcs, c), rb, m, k, t, rec, more ? c : nc,
                                    min(more ? g + step : g0, last));
            }
            set_barrier(local);
        }
    }
    if (even) __builtin_amdgcn_s_setprio(3);
}

// Sum over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ uint32_t row16_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);   // quad_perm 1 0 3 2
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);  // row_half_mirror
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);  // row_mirror
    return v;
}

// Unsatisfied bonds of block g of colour c per replica, bit-sliced (at most
// 24: five bits).
__device__ __forceinline__ void block_unsat(const RBInst &X, const uint32_t *sp, int c, int g, uint32_t (&q)[5])
{
    Fields f;
    uint32_t valid;
    block_fields(sp, load_record(X, c, g), pick3(X.base, c) + g, X.plane, f, valid);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (!((valid >> i) & 1u)) f.b0[i] = f.b1[i] = f.b2[i] = 0u;
    // sites 0 + 1 and 2 + 3 (four bits), then all
    uint32_t p[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int a = 2 * h, b = a + 1;
        const uint32_t c0 = f.b0[a] & f.b0[b];
        const uint32_t c1 = maj(f.b1[a], f.b1[b], c0);
        p[h][0] = f.b0[a] ^ f.b0[b];
        p[h][1] = xor3(f.b1[a], f.b1[b], c0);
        p[h][2] = xor3(f.b2[a], f.b2[b], c1);
        p[h][3] = maj(f.b2[a], f.b2[b], c1);
    }
    uint32_t cy = p[0][0] & p[1][0];
    q[0] = p[0][0] ^ p[1][0];
#pragma unroll
    for (int b = 1; b < 4; ++b) {
        q[b] = xor3(p[0][b], p[1][b], cy);
        cy = maj(p[0][b], p[1][b], cy);
    }
    q[4] = cy;
}

// Unsatisfied bonds per replica into unsat (zeroed): every bond is seen from
// both of its ends, except that with two colours the sites of colour 0 see
// each bond exactly once.
//   UNI: each lane adds up its blocks' counts in 16-bit halves (replicas k
// and k + 16, k + 8 and k + 24 of a word), each 16 lanes add up theirs.
//   else: few blocks a set; each lane adds its own replica by replica.
template <bool UNI>
__device__ __forceinline__ void rb_energy(const RBInst &X, const uint32_t *lds, int *unsat, int m, int sets, int tid)
{
    const int nc = X.ncol == 2 ? 1 : X.ncol;
    if constexpr (!UNI) {
        const int s = tid / X.gmax, g = tid - s * X.gmax;
        for (int c = 0; c < nc; ++c)
            if (s < sets && g < pick3(X.gcs, c)) {
                uint32_t q[5];
                block_unsat(X, lds + s * 4 * X.plane, c, g, q);
                for (int r = 0; r < m; ++r) {
                    uint32_t v = 0;
#pragma unroll
                    for (int b = 4; b >= 0; --b) v = 2 * v + __builtin_amdgcn_ubfe(q[b], r, 1);
                    atomicAdd(&unsat[s * m + r], (int)v);
                }
            }
        return;
    }
    uint32_t lo[8], hi[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) lo[r] = hi[r] = 0u;
    for (int c = 0; c < nc; ++c)
        for (int g = tid; g < pick3(X.gcs, c); g += blockDim.x) {
            uint32_t q[5];
            block_unsat(X, lds, c, g, q);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                uint32_t v = 0;
#pragma unroll
                for (int b = 4; b >= 0; --b) v = (v << 1) + ((q[b] >> r) & 0x01010101u);
                lo[r] += v & 0x00FF00FFu;
                hi[r] += (v >> 8) & 0x00FF00FFu;
            }
        }
    // sums over 16 lanes stay within 16 bits (at most 4 blocks of 24 a lane
    // and colour)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        lo[r] = row16_sum(lo[r]);
        hi[r] = row16_sum(hi[r]);
    }
    // lane i of each 16 adds word i (addresses that differ from lane to
    // lane: a uniform one would be serialised lane by lane)
    const int i = tid & 15;
    uint32_t v = lo[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) v = i == r ? (r < 8 ? lo[r & 7] : hi[r & 7]) : v;
    if (i < m) atomicAdd(&unsat[i], (int)(v & 0xFFFFu));
    if (i + 16 < m) atomicAdd(&unsat[i + 16], (int)(v >> 16));
}

// The workgroup's LDS: the sets' words, then the pass's source rows, their
// families and their unsatisfied-bond counts (32 of each a set).
template <bool UNI>
__device__ __forceinline__ void rb_tile(const Inst &I, int k, uint32_t *lds, int r0, int nrows, int m, int sets, int phase,
                                        bool even)
{
    // thresholds by n: T(dE = 12, 8, 4) for n = 0, 1, 2; n = 3 flips whatever
    // the entry
    __shared__ uint32_t tab[4];
    const int pass = m * sets;
    const TileIO io = tile_io(I);
    uint4 th = I.thr[k];
    const RBInst X = rb_inst(I, io);
    uint32_t *src = lds + 4 * X.plane * sets, *fam = src + 32 * sets;
    int *unsat = reinterpret_cast<int *>(fam + 32 * sets);
    th = make_uint4(scalar(th.x), scalar(th.y), scalar(th.z), scalar(th.w));
    const int ns = scalar(I.NS), t0 = phase == 2 ? ns / 2 : 0, t1 = phase == 1 ? ns / 2 : ns;
    if (threadIdx.x < 4)
        tab[threadIdx.x] = threadIdx.x == 0 ? th.z : threadIdx.x == 1 ? th.y : threadIdx.x == 2 ? th.x : 0u;
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
            unsat[q] = 0;
        }
        __syncthreads();
        rb_load<UNI>(X, lds, src, m, sets, tid);
        for (int q = tid; q < nr; q += blockDim.x) fam[q] = io.fsrc[src[q]];
        __syncthreads();
        // (the checks take two draws at a time)
        if (th.w)
            rb_sweeps<UNI, kAll>(X, k, lds, tab, th, row0, m, sets, t0, t1, tid, even);
        else if (th.x <= kRareT && m > 1)
            rb_sweeps<UNI, kRare>(X, k, lds, tab, th, row0, m, sets, t0, t1, tid, even);
        else if (th.y <= kRareT && m > 1)
            rb_sweeps<UNI, kMid>(X, k, lds, tab, th, row0, m, sets, t0, t1, tid, even);
        else
            rb_sweeps<UNI, kTable>(X, k, lds, tab, th, row0, m, sets, t0, t1, tid, even);
        __syncthreads();
        if (phase != 1) rb_energy<UNI>(X, lds, unsat, m, sets, tid);
        rb_store<UNI>(X, lds, row0, nr, m, sets, tid);
        if (io.map)
            for (int q = tid; q < nr; q += blockDim.x) io.fdst[row0 + q] = fam[q];
        if (phase != 1) {
            __syncthreads();
            // U counted twice with three colours
            if (X.ncol == 3)
                for (int q = tid; q < nr; q += blockDim.x) unsat[q] >>= 1;
            tile_energy_out(I, io, unsat, row0, nr);
            tile_family_count(I, fam, nr);
        }
        __syncthreads();
    }
}

}  // namespace

template <bool UNI>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(6))) void k_sweep_rb(
    const Inst *insts, const Work *work, int tile_rows, int m, int sets, int phase, bool even)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = scalar(*I.k);
    if (k >= I.nT || I.status[0]) return;
    const int Rk = (int)I.Rk[k];
    const int r0 = scalar((int)w.row0);
    const int nrows = scalar(min(tile_rows, Rk - r0));
    if (nrows > 0) rb_tile<UNI>(I, k, reinterpret_cast<uint32_t *>(lds), r0, nrows, m, sets, phase, even);
    if (phase == 1) phase1_done(I, w.n);
}

// ---------------------------------------------------------------------------
// Workgroup form of the lattice whose largest colour has G blocks: one set
// whose waves waste few lanes (up to a quarter, or beyond 1024 threads, when
// each thread takes several blocks in turn), else several sets with their
// blocks side by side.  (L = 13, G = 194, R = 10^5: one set in four waves 1072
// us a launch, five sets in 16 waves 1274: a barrier for 16 waves after every
// colour, and the replica's part of the draws per lane.)
// ---------------------------------------------------------------------------
bool rb_uniform(int G)
{
    if (G > 1024) return true;
    const int waves = (G + 63) / 64;
    return G >= 48 && 100 * G >= 75 * 64 * waves;
}

int rb_threads(int G, int sets)
{
    // beyond 1024 blocks 16 waves, four a SIMD, of which the first take one
    // block more than the last: the SIMDs' shares differ by one (L = 24,
    // G = 1728: 7 at most, R = 4000 in 267 us; two blocks for each of 14 waves
    // were 8 and 308 us)
    if (G > 1024) return 1024;
    return (G * sets + 63) / 64 * 64;
}

// The sets' words, source rows and counts.
size_t rb_lds(int plane, int sets) { return (size_t)(16 * plane + 384) * sets; }

hipError_t sweep_rb_init()
{
    for (const void *f : {(const void *)&k_sweep_rb<true>, (const void *)&k_sweep_rb<false>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSweepLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void launch_sweep_rb(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    const int nt = rb_threads(sh.G, sh.sets);
    const size_t lds = rb_lds(sh.plane, sh.sets);
    // all workgroups on the chip at once (256 compute units, 24 waves each):
    // then even progress takes 3-9% off (L = 8, R = 10^5: 255 -> 232 us); in a
    // launch of several rounds it would bring the loads of the later ones
    // together (L = 12, R = 10^5: 725 -> 766 us)
    const bool even = nwork <= 256 * (int)std::min<size_t>(24 / (nt / 64), 160 * 1024 / (lds + 512));
    if (rb_uniform(sh.G) && sh.sets == 1)
        k_sweep_rb<true><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.M, sh.sets, phase, even);
    else
        k_sweep_rb<false><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.M, sh.sets, phase, even);
}

}  // namespace pamc
