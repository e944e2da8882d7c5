// sweep_sw.hip -- Metropolis sweeps with +-1 couplings (paper Sec. II.B and
// Sec. III.A) for gfx950, L = 8 and 16, populations too small to fill words
// with replicas: the four sites of a Philox block as bytes of a word.
//
// With half a row of x a multiple of four, the stored rows are such words
// already: word g of colour c is block g, the sites of colour c in row (y, z)
// with x of parity p = (c + y + z) & 1.  The neighbours of all four are whole
// words of the other colour: the words at the same place of rows y +- 1 and
// z +- 1, the word at the same place of the same row (one x neighbour), and
// that word moved on by a byte (the other).  Seven LDS reads give what 28 do
// where bytes are replicas (sweep_rs.hip), and one lane takes block g of both
// colours in M replicas, so that the lanes of a wave hold one replica at
// L = 8 and the draw's replica part is scalar.  Per byte the six terms
// own ^ neighbour ^ [J = -1] add up to the unsatisfied bonds n; the threshold
// reads go out before the draws, whose arithmetic covers them.
//
// What bounds it: a lone wave's latency, 0.21 us a colour step with one replica
// a lane and 0.31 with two (about 80 and 125 instructions); beyond four waves a
// SIMD instruction issue, 1800 attempts per ns, which words of many replicas
// exceed.  Launches against bytes as replicas and bits (sweep_rs.hip,
// sweep_rb.hip), and against a form that held the rows in byte planes: L = 8,
// 50 sweeps: R = 300: 29 us, 63 and 43; R = 10^4: 126, 233 and 155; 10 sweeps,
// R = 10^4: 35, 56 and 51; L = 16, 50 sweeps, R = 300: 64, 119 and 106.
#include "launch.h"
#include "pamc_dev.h"
#include "rb_common.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

namespace {

template <int L>
struct SWShape {
    static constexpr int N = L * L * L;
    static constexpr int W = N / 4;     // words of a row
    static constexpr int G = N / 8;     // Philox blocks of a colour, and threads of a replica
    static constexpr int GPR = L / 8;   // blocks of half a row of x
    static constexpr bool kWave = G == 64;
};

// A lane's block of one colour: word offsets in the row, [J = -1] per byte.
struct SWBlock {
    uint32_t own, same, next, yp, ym, zp, zm;
    uint32_t shift;  // bytes that the pair (same, next) or (next, same) is moved by
    uint32_t ja, js, j[4];
};

__device__ __forceinline__ uint32_t nibble_to_bytes(uint32_t b) { return (b * 0x00204081u) & 0x01010101u; }

template <int L>
__device__ __forceinline__ SWBlock sw_block(const RBInst &X, int c, int g)
{
    using S = SWShape<L>;
    const int row = g / S::GPR, jb = g % S::GPR, y = row % L, z = row / L, p = (c + y + z) & 1;
    const uint32_t other = (uint32_t)(1 - c) * S::G;
    const uint32_t minus = load_record(X, c, g).q[3].x;  // bit 4 d + i, d: +x, -x, +y, -y, +z, -z
    auto sign = [&](int d) { return nibble_to_bytes((minus >> (4 * d)) & 15u); };
    SWBlock b;
    b.own = (uint32_t)c * S::G + g;
    b.same = other + g;
    // sites at x = 2 i + p: the word at the same place holds x + 1 (p = 0) or
    // x - 1, the other x neighbour is a site further left or right
    b.next = other + row * S::GPR + (jb + (p ? 1 : S::GPR - 1)) % S::GPR;
    b.shift = p ? 1u : 3u;
    b.ja = sign(p);
    b.js = sign(1 - p);
    b.yp = other + (z * L + (y + 1) % L) * S::GPR + jb;
    b.ym = other + (z * L + (y + L - 1) % L) * S::GPR + jb;
    b.zp = other + ((z + 1) % L * L + y) * S::GPR + jb;
    b.zm = other + ((z + L - 1) % L * L + y) * S::GPR + jb;
#pragma unroll
    for (int d = 0; d < 4; ++d) b.j[d] = sign(2 + d);
    return b;
}

// The words around a block.
struct SWWords {
    uint32_t own, same, next, yp, ym, zp, zm;
};
template <int L>
__device__ __forceinline__ SWWords sw_read(const uint32_t *row, const SWBlock &b)
{
    SWWords w;
    w.own = row[b.own];
    w.same = row[b.same];
    w.next = SWShape<L>::GPR == 1 ? w.same : row[b.next];
    w.yp = row[b.yp];
    w.ym = row[b.ym];
    w.zp = row[b.zp];
    w.zm = row[b.zm];
    return w;
}
// Unsatisfied bonds per byte (at most 6).
__device__ __forceinline__ uint32_t sw_unsat(const SWWords &w, const SWBlock &b)
{
    const uint32_t hi = b.shift == 1u ? w.next : w.same, lo = b.shift == 1u ? w.same : w.next;
    const uint32_t moved = __builtin_amdgcn_alignbyte(hi, lo, b.shift);
    return (xor3(w.own, w.same, b.ja) + xor3(w.own, moved, b.js) + xor3(w.own, w.yp, b.j[0])) +
           (xor3(w.own, w.ym, b.j[1]) + xor3(w.own, w.zp, b.j[2]) + xor3(w.own, w.zm, b.j[3]));
}

template <int L, int M, bool ALL>
__device__ __forceinline__ void sw_sweeps(const RBInst &X, int k, uint32_t *lds, const SWBlock (&blk)[2], const uint32_t *tab,
                                          int g, uint32_t rb, int t0, int t1)
{
    using S = SWShape<L>;
    const uint8_t *tb = reinterpret_cast<const uint8_t *>(tab);
    for (int t = t0; t < t1; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const SWBlock &b = blk[c];
            if constexpr (ALL) {
#pragma unroll
                for (int j = 0; j < M; ++j) lds[j * S::W + b.own] ^= 0x01010101u;
            } else {
                SWWords w[M];
#pragma unroll
                for (int j = 0; j < M; ++j) w[j] = sw_read<L>(lds + j * S::W, b);
                __builtin_amdgcn_sched_barrier(0);
                const LaneDraw d = lane_draw(((uint32_t)c << 24) | (uint32_t)g, k, t, X.k0, X.k1);
                uint32_t th[M][4], flip[M];
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    const uint32_t n = sw_unsat(w[j], b), n4 = n << 2;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        th[j][i] = *reinterpret_cast<const uint32_t *>(tb + __builtin_amdgcn_ubfe(n4, 8 * i, 5));
                    // n >= 3 (dE <= 0) always flips
                    flip[j] = ((n + 0x05050505u) >> 3) & 0x01010101u;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    const uint4 u = replica_draw<true>(d, rb + (uint32_t)j, k, X.k0, X.k1);
#pragma unroll
                    for (int i = 0; i < 4; ++i) flip[j] |= word_of(u, i) < th[j][i] ? 1u << (8 * i) : 0u;
                    lds[j * S::W + b.own] = w[j].own ^ flip[j];
                }
            }
            set_barrier(S::kWave);
        }
}

// The workgroup's LDS: the rows' words, then the pass's source rows, their
// families and their unsatisfied-bond counts.
template <int L, int M>
__device__ __forceinline__ void sw_tile(const Inst &I, int k, uint32_t *lds, int r0, int nrows, int sets, int phase)
{
    using S = SWShape<L>;
    // thresholds by n: T(dE = 12, 8, 4) for n = 0, 1, 2; no draw is below the
    // others, which flip anyway
    __shared__ uint32_t tab[8];
    const int pass = M * sets, tid = (int)threadIdx.x, g = tid & (S::G - 1), set = scalar(tid / S::G);
    const TileIO io = tile_io(I);
    uint4 th = I.thr[k];
    const RBInst X = rb_inst(I, io);
    th = make_uint4(scalar(th.x), scalar(th.y), scalar(th.z), scalar(th.w));
    const int ns = scalar(I.NS), t0 = phase == 2 ? ns / 2 : 0, t1 = phase == 1 ? ns / 2 : ns;
    uint32_t *src = lds + pass * S::W, *fam = src + pass;
    int *unsat = reinterpret_cast<int *>(fam + pass);
    const SWBlock blk[2] = {sw_block<L>(X, 0, g), sw_block<L>(X, 1, g)};
    if (tid < 8) tab[tid] = tid == 0 ? th.z : tid == 1 ? th.y : tid == 2 ? th.x : 0u;
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
        for (int it = tid; it < pass * S::W; it += blockDim.x) {
            const int q = it / S::W, w = it % S::W;
            const GlobalIn row = (GlobalIn)(X.src + (size_t)src[q] * X.srow);
            lds[it] = X.packed ? nibble_to_bytes((row[w >> 3] >> (4 * (w & 7))) & 15u) : row[w];
        }
        for (int q = tid; q < nr; q += blockDim.x) fam[q] = io.fsrc[src[q]];
        __syncthreads();
        uint32_t *mine = lds + set * M * S::W;
        const uint32_t rb = scalar((uint32_t)(row0 + set * M));
        if (th.w)
            sw_sweeps<L, M, true>(X, k, mine, blk, tab, g, rb, t0, t1);
        else
            sw_sweeps<L, M, false>(X, k, mine, blk, tab, g, rb, t0, t1);
        if (phase != 1)
            // the sites of colour 0 see each bond once
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const uint32_t n = sw_unsat(sw_read<L>(mine + j * S::W, blk[0]), blk[0]);
                const int sum = wave_fold((int32_t)__builtin_amdgcn_sad_u8(n, 0u, 0u), [](int a, int b) { return a + b; });
                if ((tid & 63) == 0) atomicAdd(&unsat[set * M + j], sum);
            }
        __syncthreads();
        if (!X.packed) {
            for (int it = tid; it < nr * S::W; it += blockDim.x) {
                const int q = it / S::W, w = it % S::W;
                ((GlobalOut)(X.dst + (size_t)(row0 + q) * X.srow))[w] = lds[it];
            }
        } else {
            constexpr int P = S::W / 8;  // stored words of a row
            for (int it = tid; it < nr * P; it += blockDim.x) {
                const int q = it / P, w = it % P;
                uint32_t v = 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) v |= bytes_to_bits4(lds[q * S::W + 8 * w + i]) << (4 * i);
                ((GlobalOut)(X.dst + (size_t)(row0 + q) * X.srow))[w] = v;
            }
        }
        if (io.map)
            for (int q = tid; q < nr; q += blockDim.x) io.fdst[row0 + q] = fam[q];
        if (phase != 1) {
            tile_energy_out(I, io, unsat, row0, nr);
            tile_family_count(I, fam, nr);
        }
        __syncthreads();
    }
}

}  // namespace

template <int L, int M>
__global__ __launch_bounds__(1024) void k_sweep_sw(const Inst *insts, const Work *work, int tile_rows, int sets, int phase)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = scalar(*I.k);
    if (k >= I.nT || I.status[0]) return;
    const int Rk = (int)I.Rk[k];
    const int r0 = scalar((int)w.row0);
    const int nrows = scalar(min(tile_rows, Rk - r0));
    if (nrows > 0) sw_tile<L, M>(I, k, reinterpret_cast<uint32_t *>(lds), r0, nrows, sets, phase);
    if (phase == 1) phase1_done(I, w.n);
}

// Stored rows are words of blocks where half a row of x is whole blocks; up to
// two replicas a lane.
bool sw_form(int L, int m) { return (L == 8 || L == 16) && (m == kSiteWord + 1 || m == kSiteWord + 2); }
int sw_threads(int G, int sets) { return G * sets; }
size_t sw_lds(int row_bytes, int m, int sets) { return (size_t)(m - kSiteWord) * sets * (size_t)(row_bytes + 12); }

hipError_t sweep_sw_init()
{
    for (const void *f : {(const void *)&k_sweep_sw<8, 1>, (const void *)&k_sweep_sw<8, 2>, (const void *)&k_sweep_sw<16, 1>,
                          (const void *)&k_sweep_sw<16, 2>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSweepLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void launch_sweep_sw(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    const int nt = sw_threads(sh.G, sh.sets), m = sh.M - kSiteWord;
    const size_t lds = sw_lds(sh.row_bytes, sh.M, sh.sets);
#define PAMC_SW(LL, MM)                                                                                 \
    if (sh.G == SWShape<LL>::G && m == MM) k_sweep_sw<LL, MM><<<nwork, nt, lds, st>>>(insts, work, sh.tile_rows, sh.sets, phase)
    PAMC_SW(8, 1);
    PAMC_SW(8, 2);
    PAMC_SW(16, 1);
    PAMC_SW(16, 2);
#undef PAMC_SW
}

}  // namespace pamc
