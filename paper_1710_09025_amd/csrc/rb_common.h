// rb_common.h -- device routines shared by the replica-word sweeps (+-1
// couplings in sweep_rb.hip, real couplings in sweep_rq.hip): the draws split
// by what they depend on, what a tile reads of its instance, and the rows of a
// pass to and from words that hold one site of up to 32 replicas.
#pragma once
#include "pamc_dev.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;

// Row memory and tables are global (the descriptor's pointers would make flat
// accesses).
typedef __attribute__((address_space(1))) const uint32_t *GlobalIn;
typedef __attribute__((address_space(1))) uint32_t *GlobalOut;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 *GlobalRec;

// What the passes of a tile read of the instance, in scalar registers
// (values read through pointers would stay in vector registers).
struct RBInst {
    const uint8_t *src;
    uint8_t *dst;
    int srow, packed;
    int plane, nb;        // LDS words per site plane, four-site blocks of a row
    int ncol, gmax;
    int gcs[3], base[3];  // Philox blocks of each colour, first block of each in a row
    GlobalRec tab;        // records of four 16-byte words
    uint32_t k0, k1;
};
__device__ __forceinline__ RBInst rb_inst(const Inst &I, const TileIO &io)
{
    RBInst x;
    x.src = scalar_ptr(io.src);
    x.dst = scalar_ptr(io.dst);
    x.srow = scalar(io.srow);
    x.packed = scalar(io.packed);
    x.plane = scalar(I.rb_plane);
    x.nb = scalar(I.row_bytes) >> 2;
    x.ncol = scalar(I.ncol);
    x.gmax = scalar(I.gmax);
    for (int c = 0; c < 3; ++c) {
        x.gcs[c] = scalar(I.gcs[c]);
        x.base[c] = scalar(I.cbase[c]) >> 2;
    }
    x.tab = (GlobalRec)scalar_ptr(I.rbtab);
    x.k0 = scalar(I.key0);
    x.k1 = scalar(I.key1);
    return x;
}
__device__ __forceinline__ int pick3(const int (&a)[3], int c) { return c == 0 ? a[0] : c == 1 ? a[1] : a[2]; }

__device__ __forceinline__ uint32_t hi32(uint64_t v) { return (uint32_t)(v >> 32); }
__device__ __forceinline__ uint32_t maj(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Philox state after the rounds that do not mix (block, sweep) with the
// replica: lane part of rounds 1-3 of the block at counter
// (ctr, r, k, tag | t).
struct LaneDraw {
    uint32_t w1;   // round 1 word w, round 2 key mixed in
    uint32_t y2;   // round 2 word y, round 3 key mixed in
    uint32_t z3;   // round 3 word z without the replica's part
    uint32_t w3;   // round 3 word w
};
__device__ __forceinline__ LaneDraw lane_draw(uint32_t ctr, int k, int t, uint32_t k0, uint32_t k1)
{
    const uint64_t a = (uint64_t)kM0 * ctr;
    const uint32_t z1 = xor3(hi32(a), kTagSweep | (uint32_t)t, k1);
    const uint64_t b = (uint64_t)kM1 * z1;
    const uint32_t x2 = xor3(hi32(b), kM1 * (uint32_t)k, k0 + kW0);
    const uint64_t q = (uint64_t)kM0 * x2;
    LaneDraw d;
    d.w1 = (uint32_t)a ^ (k1 + kW1);
    d.y2 = (uint32_t)b ^ (k0 + 2u * kW0);
    d.z3 = hi32(q) ^ (k1 + 2u * kW1);
    d.w3 = (uint32_t)q;
    return d;
}
// The replica's part of rounds 1 and 2, the same in every lane and sweep: on
// the scalar unit when a wave holds one set (UNI, r uniform); then rounds
// 3-10.
template <bool UNI>
__device__ __forceinline__ uint4 replica_draw(const LaneDraw &d, uint32_t r, int k, uint32_t k0, uint32_t k1)
{
    const uint32_t x1 = __umulhi(kM1, (uint32_t)k) ^ r ^ k0;
    uint32_t ph, pl;
    if constexpr (UNI) {
        ph = __umulhi(kM0, x1);
        pl = kM0 * x1;
    } else {
        const uint64_t p = (uint64_t)kM0 * x1;
        ph = hi32(p);
        pl = (uint32_t)p;
    }
    const uint64_t m = (uint64_t)kM1 * (ph ^ d.w1);
    uint4 c = make_uint4(hi32(m) ^ d.y2, (uint32_t)m, pl ^ d.z3, d.w3);
#pragma unroll
    for (int i = 3; i < 10; ++i) {
        const uint64_t a = (uint64_t)kM0 * c.x, b = (uint64_t)kM1 * c.z;
        c = make_uint4(xor3(hi32(b), c.y, k0 + (uint32_t)i * kW0), (uint32_t)b,
                       xor3(hi32(a), c.w, k1 + (uint32_t)i * kW1), (uint32_t)a);
    }
    return c;
}

// acc = 2 acc + [u < T]
__device__ __forceinline__ void push_lt(uint32_t &acc, uint32_t u, uint32_t T)
{
    asm("v_cmp_lt_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(acc) : "v"(u), "v"(T) : "vcc");
}

// A block's record: 16-bit LDS word indices of the six neighbours of its four
// sites ([direction][site]), then the sign bits (J = -1, bit 4 d + i) and the
// mask of real sites.
struct Record {
    u32x4 q[4];
};
__device__ __forceinline__ Record load_record(const RBInst &X, int c, int g)
{
    const GlobalRec p = X.tab + (size_t)(uint32_t)(c * X.gmax + g) * 4;
    return Record{{p[0], p[1], p[2], p[3]}};
}
// Issue priority by progress: sweep t of [t0, t1) in quarters, the waves that
// are behind first.  A SIMD serves its oldest wave first, so of waves that
// start together (a launch that the chip holds at once) one after another
// finishes early and the last run alone, at half the rate of instructions:
// L = 8, R = 10^5, five waves a SIMD, finished after 73 to 200 us.
__device__ __forceinline__ void even_progress(int t, int t0, int t1)
{
    const int q = 4 * (t - t0) / (t1 - t0);
    if (q == 0)
        __builtin_amdgcn_s_setprio(3);
    else if (q == 1)
        __builtin_amdgcn_s_setprio(2);
    else if (q == 2)
        __builtin_amdgcn_s_setprio(1);
    else
        __builtin_amdgcn_s_setprio(0);
}

// LDS order between the lanes of a set: a wave's LDS operations complete in
// issue order, so sets inside one wave need only a compiler fence.
__device__ __forceinline__ void set_barrier(bool wave_local)
{
    if (wave_local) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// 32 x 32 bit transpose: bit i of a[j] <-> bit j of a[i].
__device__ __forceinline__ void transpose32(uint32_t (&a)[32])
{
    constexpr uint32_t mask[5] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu, 0x00FF00FFu, 0x0000FFFFu};
#pragma unroll
    for (int b = 4; b >= 0; --b) {
        const int s = 1 << b;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            if (k & s) continue;
            const uint32_t x = ((a[k] >> s) ^ a[k + s]) & mask[b];
            a[k + s] ^= x;
            a[k] ^= x << s;
        }
    }
}

// Rows of a pass into the sets' words (rows stored one byte or one bit per
// position) and back.  src[q]: stored row of the pass's row q.  A lane takes
// four positions (bytes) or 32 (bits) of the m rows of a set; UNI: row
// addresses are uniform, lane j holding row j's.
template <bool UNI>
__device__ __forceinline__ GlobalIn row_in(const RBInst &X, const uint32_t *src, uint64_t mine, int j, int m)
{
    if constexpr (UNI)
        return (GlobalIn)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, j) |
                          ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), j) << 32));
    else
        return (GlobalIn)(X.src + (size_t)src[min(j, m - 1)] * X.srow);
}

template <bool UNI>
__device__ __forceinline__ void rb_load(const RBInst &X, uint32_t *lds, const uint32_t *src, int m, int sets, int tid)
{
    const int plane = X.plane, nb = X.nb, lane = tid & 63;
    // (rows past the m-th: the last one again)
    const uint64_t mine = UNI ? (uint64_t)(X.src + (size_t)src[min(lane, m - 1)] * X.srow) : 0ull;
    // eight loads in flight before the first is used (a CU holds many waves;
    // more would cost registers)
    if (!X.packed) {
        for (int it = tid; it < sets * nb; it += blockDim.x) {
            const int s = UNI ? 0 : it / nb, b = UNI ? it : it - s * nb;
            uint32_t a[4] = {0u, 0u, 0u, 0u}, o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (8 * q >= m) break;
                uint32_t v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = row_in<UNI>(X, src + s * m, mine, 8 * q + j, m)[(uint32_t)b];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j) a[q] |= v[j] << j;
            }
            transpose4(a[0], a[1], a[2], a[3], o);
            uint32_t *sp = lds + s * 4 * plane + b;
#pragma unroll
            for (int i = 0; i < 4; ++i) sp[i * plane] = o[i];
        }
        return;
    }
    const int nd = (nb + 7) >> 3;
    for (int it = tid; it < sets * nd; it += blockDim.x) {
        const int s = UNI ? 0 : it / nd, d = UNI ? it : it - s * nd;
        uint32_t a[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            a[j] = row_in<UNI>(X, src + s * m, mine, j, m)[(uint32_t)d];
            if ((j & 7) == 7) __builtin_amdgcn_sched_barrier(0);
        }
        transpose32(a);
        uint32_t *sp = lds + s * 4 * plane;
#pragma unroll
        for (int p = 0; p < 32; ++p) {
            const int b = 8 * d + (p >> 2);
            if (b < nb) sp[(p & 3) * plane + b] = a[p];
        }
    }
}

template <bool UNI>
__device__ __forceinline__ void rb_store(const RBInst &X, const uint32_t *lds, int row0, int nrows, int m, int sets, int tid)
{
    const int plane = X.plane, nb = X.nb;
    if (!X.packed) {
        for (int it = tid; it < sets * nb; it += blockDim.x) {
            const int s = UNI ? 0 : it / nb, b = UNI ? it : it - s * nb;
            const uint32_t *sp = lds + s * 4 * plane + b;
            uint32_t a[4];
            transpose4(sp[0], sp[plane], sp[2 * plane], sp[3 * plane], a);
            uint8_t *p = X.dst + (size_t)(row0 + s * m) * X.srow;
            int left = min(m, nrows - s * m);  // rows of this set
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = min(8, left);
#pragma unroll 1
                for (int j = 0; j < n; ++j) {
                    ((GlobalOut)p)[(uint32_t)b] = (a[q] >> j) & 0x01010101u;
                    p += X.srow;
                }
                left -= n;
            }
        }
        return;
    }
    // (every word of a stored row, zeros past the blocks: the overlap reads
    // whole rows, and a buffer that staged a stored state holds its bytes)
    // (opaque: the reciprocal to divide by it would be held through the sweeps)
    int nd = X.srow >> 2;
    asm volatile("" : "+s"(nd));
    for (int it = tid; it < sets * nd; it += blockDim.x) {
        const int s = UNI ? 0 : it / nd, d = UNI ? it : it - s * nd;
        const uint32_t *sp = lds + s * 4 * plane;
        uint32_t a[32];
#pragma unroll
        for (int p = 0; p < 32; ++p) {
            const int b = 8 * d + (p >> 2);
            a[p] = b < nb ? sp[(p & 3) * plane + b] : 0u;
        }
        transpose32(a);
        uint8_t *p = X.dst + (size_t)(row0 + s * m) * X.srow;
        int left = min(m, nrows - s * m);
        // (opaque: the comparisons with the row count would otherwise be
        // hoisted out of the loop, 32 masks in scalar registers)
        if constexpr (UNI)
            asm volatile("" : "+s"(left));
        else
            asm volatile("" : "+v"(left));
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            if (j >= left) break;
            ((GlobalOut)p)[(uint32_t)d] = a[j];
            p += X.srow;
        }
    }
}

}  // namespace pamc
