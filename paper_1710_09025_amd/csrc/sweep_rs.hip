// sweep_rs.hip -- Metropolis sweeps with +-1 couplings (paper Sec. II.B and
// Sec. III.A) for gfx950, populations too small to fill the chip: up to four
// replicas as bytes of a word.
//
// A lane takes a Philox block (four sites of a colour) as in sweep_rb.hip, but
// with a replica or two a lane the bit-sliced fields there cost three times
// the draws they serve, and the block's record is read and unpacked anew for
// every colour step.  Here a lane keeps its neighbours' LDS addresses (one
// block of every colour, 24 each) through all sweeps; a spin is a byte 0 or 1,
// and each site has a second word with the spins flipped, which the bonds with
// J = -1 read, so that one XOR-add a bond counts its unsatisfied ones (n, at
// most 6) in all four bytes.  With c the number of thresholds
// T(4) >= T(8) >= T(12) that a draw is below, dE = 12 - 4 n is accepted when
// n + c >= 3: the comparisons wait for no field.
//
// What bounds it: the latency of one wave, about 190 instructions and two LDS
// round trips a colour step for one replica a lane (0.55 us), and some 6 us to
// read the tables and rows.  Launches of 10 sweeps at beta = 1.5 against words
// of bits: L = 4, R = 1000: 29.5 -> 21.4 us; L = 10, R = 500: 35.0 -> 28.6
// (L = 8 and 16 have sweep_sw.hip for such populations).  With four
// replicas a lane the two are level (L = 8, R = 8000: 61.1 and 60.9); beyond,
// words of bits win.
#include "launch.h"
#include "pamc_dev.h"
#include "rb_common.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

namespace {

// A lane's block of one colour, as byte addresses in LDS.
struct RSBlock {
    uint32_t nb[24];   // neighbour words, [direction][site]
    uint32_t own;      // word of site 0 (site i: i planes on)
    uint32_t real[4];  // bytes 1 for real sites, 0 for padding
    uint32_t ctr;      // Philox counter word 0
};

// LDS words by address (the kernel's LDS need not start at 0; a pointer and an
// offset would be added for every access).
typedef __attribute__((address_space(3))) uint32_t *LdsWord;
__device__ __forceinline__ uint32_t lds_address(uint32_t *p) { return (uint32_t)(uintptr_t)(LdsWord)p; }
__device__ __forceinline__ uint32_t word_at(uint32_t a) { return *(LdsWord)(uintptr_t)a; }
__device__ __forceinline__ void set_word(uint32_t a, uint32_t v) { *(LdsWord)(uintptr_t)a = v; }

// acc += a ^ b, acc += [u < T] (T the same in all lanes)
__device__ __forceinline__ void xor_add(uint32_t &acc, uint32_t a, uint32_t b)
{
    asm("v_xad_u32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void count_lt(uint32_t &acc, uint32_t u, uint32_t T)
{
    asm("v_cmp_gt_u32 vcc, %2, %1\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(acc) : "v"(u), "s"(T) : "vcc");
}

// Unsatisfied bonds of site i, per byte.
__device__ __forceinline__ uint32_t unsat_of(const RSBlock &b, const uint32_t (&nb)[24], int i, uint32_t own)
{
    uint32_t n = 0;
#pragma unroll
    for (int d = 0; d < 6; ++d) xor_add(n, own, nb[4 * d + i]);
    return n;
}

template <bool UNI, bool ALL, int NCOL>
__device__ __forceinline__ void rs_sweeps(const RBInst &X, int k, const RSBlock (&blk)[NCOL], uint4 th,
                                          uint32_t rb, int m, bool local, int t0, int t1)
{
    const uint32_t plane = 4u * (uint32_t)X.plane, other = 4u * plane;
    for (int t = t0; t < t1; ++t)
#pragma unroll
        for (int c = 0; c < NCOL; ++c) {
            const RSBlock &b = blk[c];
            uint32_t own[4], flip[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) own[i] = word_at(b.own + i * plane);
            if constexpr (ALL) {
#pragma unroll
                for (int i = 0; i < 4; ++i) flip[i] = b.real[i];
            } else {
                uint32_t nb[24], below[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int e = 0; e < 24; ++e) nb[e] = word_at(b.nb[e]);
                // (the draws while the reads are under way)
                __builtin_amdgcn_sched_barrier(0);
                const LaneDraw d = lane_draw(b.ctr, k, t, X.k0, X.k1);
#pragma unroll 1
                for (int r = m - 1; r >= 0; --r) {
                    const uint4 u = replica_draw<UNI>(d, rb + (uint32_t)r, k, X.k0, X.k1);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t w = word_of(u, i);
                        below[i] <<= 8;
                        count_lt(below[i], w, th.x);
                        count_lt(below[i], w, th.y);
                        count_lt(below[i], w, th.z);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    flip[i] = ((unsat_of(b, nb, i, own[i]) + below[i] + 0x05050505u) >> 3) & b.real[i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b.real[i]) {
                    const uint32_t s = own[i] ^ flip[i];
                    set_word(b.own + i * plane, s);
                    set_word(b.own + i * plane + other, s ^ 0x01010101u);
                }
            set_barrier(local);
        }
}

// Rows of a pass into the sets' words and back; src as in rb_load.  Four
// positions a step (rows of bytes) or 32 (of bits).
__device__ __forceinline__ void rs_load(const RBInst &X, uint32_t *lds, int stride, const uint32_t *src, int m, int sets, int tid)
{
    const int plane = X.plane, nb = X.nb;
    const int items = X.packed ? (nb + 7) >> 3 : nb;
    for (int it = tid; it < sets * items; it += blockDim.x) {
        const int s = it / items, b = it - s * items;
        uint32_t *sp = lds + s * stride;
        uint32_t a[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = ((GlobalIn)(X.src + (size_t)src[s * m + min(j, m - 1)] * X.srow))[(uint32_t)b];
        if (!X.packed) {
            uint32_t o[4];
            transpose4(a[0], a[1], a[2], a[3], o);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sp[i * plane + b] = o[i];
                sp[(4 + i) * plane + b] = o[i] ^ 0x01010101u;
            }
        } else {
            const int last = min(8, nb - 8 * b);
            for (int q = 0; q < last; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t v = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v |= __builtin_amdgcn_ubfe(a[j], (uint32_t)(4 * q + i), 1u) << (8 * j);
                    sp[i * plane + 8 * b + q] = v;
                    sp[(4 + i) * plane + 8 * b + q] = v ^ 0x01010101u;
                }
        }
    }
}

__device__ __forceinline__ void rs_store(const RBInst &X, const uint32_t *lds, int stride, int row0, int nrows, int m, int sets,
                                         int tid)
{
    const int plane = X.plane, nb = X.nb;
    const int items = X.packed ? X.srow >> 2 : nb;
    for (int it = tid; it < sets * items; it += blockDim.x) {
        const int s = it / items, b = it - s * items;
        const uint32_t *sp = lds + s * stride;
        uint32_t a[4] = {0u, 0u, 0u, 0u};
        if (!X.packed) {
            transpose4(sp[b], sp[plane + b], sp[2 * plane + b], sp[3 * plane + b], a);
        } else {
            const int last = min(8, nb - 8 * b);
            for (int q = 0; q < last; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t v = sp[i * plane + 8 * b + q];
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[j] |= __builtin_amdgcn_ubfe(v, (uint32_t)(8 * j), 1u) << (4 * q + i);
                }
        }
        const int left = min(m, nrows - s * m);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < left) ((GlobalOut)(X.dst + (size_t)(row0 + s * m + j) * X.srow))[(uint32_t)b] = a[j];
    }
}

// The workgroup's LDS: the sets' words (eight planes each and padding), then
// the pass's source rows, their families and their unsatisfied-bond counts.
template <bool UNI, int NCOL>
__device__ __forceinline__ void rs_tile(const Inst &I, int k, uint32_t *lds, int r0, int nrows, int m, int sets, int stride,
                                        int phase)
{
    const int pass = m * sets, tid = (int)threadIdx.x;
    const TileIO io = tile_io(I);
    uint4 th = I.thr[k];
    const RBInst X = rb_inst(I, io);
    th = make_uint4(scalar(th.x), scalar(th.y), scalar(th.z), scalar(th.w));
    const int ns = scalar(I.NS), t0 = phase == 2 ? ns / 2 : 0, t1 = phase == 1 ? ns / 2 : ns;
    uint32_t *src = lds + sets * stride, *fam = src + 4 * sets;
    int *unsat = reinterpret_cast<int *>(fam + 4 * sets);
    // UNI: a set fills the workgroup's waves; else the sets' blocks side by side
    int set = UNI ? 0 : tid / X.gmax;
    const int g = UNI ? tid : tid - set * X.gmax;
    const bool act = set < sets && g < X.gmax;
    if (!act) set = 0;
    const bool local = blockDim.x == 64;
    RSBlock blk[NCOL];
#pragma unroll
    for (int c = 0; c < NCOL; ++c) {
        const Record rec = load_record(X, c, act ? g : 0);
        const uint32_t e[12] = {rec.q[0].x, rec.q[0].y, rec.q[0].z, rec.q[0].w, rec.q[1].x, rec.q[1].y,
                                rec.q[1].z, rec.q[1].w, rec.q[2].x, rec.q[2].y, rec.q[2].z, rec.q[2].w};
        const uint32_t base = lds_address(lds + set * stride), minus = rec.q[3].x;
        const uint32_t valid = act && g < pick3(X.gcs, c) ? rec.q[3].y : 0u;
#pragma unroll
        for (int d = 0; d < 6; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t v = e[2 * d + (i >> 1)], w = (i & 1) ? v >> 16 : v & 0xFFFFu;
                const uint32_t flipped = (minus >> (4 * d + i)) & 1u ? 4u * (uint32_t)X.plane : 0u;
                blk[c].nb[4 * d + i] = base + 4u * (w + flipped);
            }
        blk[c].own = base + 4u * ((uint32_t)pick3(X.base, c) + (valid ? (uint32_t)g : 0u));
#pragma unroll
        for (int i = 0; i < 4; ++i) blk[c].real[i] = (valid >> i) & 1u ? 0x01010101u : 0u;
        blk[c].ctr = ((uint32_t)c << 24) | (uint32_t)g;
    }
    for (int q0 = 0; q0 < nrows; q0 += pass) {
        const int row0 = r0 + q0, nr = min(pass, nrows - q0);
        // rows past the end are swept as copies of the pass's first row and
        // never stored
        for (int q = tid; q < pass; q += blockDim.x) {
            uint32_t r = (uint32_t)(row0 + (q < nr ? q : 0));
            if (io.map) r = io.map[r];
            src[q] = r;
            unsat[q] = 0;
        }
        __syncthreads();
        rs_load(X, lds, stride, src, m, sets, tid);
        for (int q = tid; q < nr; q += blockDim.x) fam[q] = io.fsrc[src[q]];
        __syncthreads();
        uint32_t rb = (uint32_t)(row0 + set * m);
        if constexpr (UNI) rb = scalar(rb);
        if (th.w)
            rs_sweeps<UNI, true>(X, k, blk, th, rb, m, local, t0, t1);
        else
            rs_sweeps<UNI, false>(X, k, blk, th, rb, m, local, t0, t1);
        __syncthreads();
        if (phase != 1) {
            // two colours: the sites of the first see each bond once; three:
            // all sites see it twice
            uint32_t n = 0;
#pragma unroll
            for (int c = 0; c < (NCOL == 2 ? 1 : NCOL); ++c) {
                uint32_t nb[24];
#pragma unroll
                for (int e = 0; e < 24; ++e) nb[e] = word_at(blk[c].nb[e]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t v = unsat_of(blk[c], nb, i, word_at(blk[c].own + 4u * (uint32_t)(i * X.plane)));
                    n += blk[c].real[i] ? v : 0u;
                }
            }
            if (n)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < m) atomicAdd(&unsat[set * m + j], (int)((n >> (8 * j)) & 0xFFu));
        }
        rs_store(X, lds, stride, row0, nr, m, sets, tid);
        if (io.map)
            for (int q = tid; q < nr; q += blockDim.x) io.fdst[row0 + q] = fam[q];
        if (phase != 1) {
            __syncthreads();
            if (NCOL == 3) {
                for (int q = tid; q < nr; q += blockDim.x) unsat[q] >>= 1;
                __syncthreads();
            }
            tile_energy_out(I, io, unsat, row0, nr);
            tile_family_count(I, fam, nr);
        }
        __syncthreads();
    }
}

}  // namespace

template <bool UNI, int NCOL>
__global__ __launch_bounds__(512) void k_sweep_rs(const Inst *insts, const Work *work, int tile_rows, int m, int sets, int stride,
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
    if (nrows > 0) rs_tile<UNI, NCOL>(I, k, reinterpret_cast<uint32_t *>(lds), r0, nrows, m, sets, stride, phase);
    if (phase == 1) phase1_done(I, w.n);
}

// Few replicas a lane, and a block of every colour for each.
bool rs_small(int G, int m, int sets) { return m <= kSmallWord && G * sets <= 512; }

// Words of a set: eight planes, padded so that the sets whose blocks share a
// wave start G banks apart.
static int rs_stride(int plane, int G)
{
    const int base = 8 * plane;
    return G >= 64 ? base : base + (((G - base) % 64) + 64) % 64;
}
size_t rs_lds(int plane, int G, int sets) { return 4 * (size_t)sets * (size_t)(rs_stride(plane, G) + 12); }

hipError_t sweep_rs_init()
{
    for (const void *f : {(const void *)&k_sweep_rs<true, 2>, (const void *)&k_sweep_rs<true, 3>,
                          (const void *)&k_sweep_rs<false, 2>, (const void *)&k_sweep_rs<false, 3>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSweepLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void launch_sweep_rs(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    const int nt = rb_threads(sh.G, sh.sets), stride = rs_stride(sh.plane, sh.G);
    const size_t lds = rs_lds(sh.plane, sh.G, sh.sets);
#define PAMC_RS(UNI, NCOL) \
    k_sweep_rs<UNI, NCOL><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.M, sh.sets, stride, phase)
    if (rb_uniform(sh.G) && sh.sets == 1) {
        if (sh.ncol == 2)
            PAMC_RS(true, 2);
        else
            PAMC_RS(true, 3);
    } else {
        if (sh.ncol == 2)
            PAMC_RS(false, 2);
        else
            PAMC_RS(false, 3);
    }
#undef PAMC_RS
}

}  // namespace pamc
