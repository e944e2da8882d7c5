// step_common.h -- device routines shared by the sweep and resampling
// kernels: the Philox4x32-10 generator, block reductions, the fixed pairwise
// summation tree, the level weights, counting with few atomics per wave and
// the end-of-launch detection of the last workgroup of an instance.
#pragma once
#include "pamc_dev.h"

#pragma clang fp contract(off)

namespace pamc {

// a ^ b ^ c in one instruction: gfx950's three-input bitwise operation with
// the truth table of a three-way exclusive or.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  Each round multiplies
// counter words 0 and 2 by the round multipliers, the high halves mixed with
// words 1 and 3 and the round key; the key advances by the Weyl constants.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * (uint64_t)c.x;
        const uint64_t b = (uint64_t)0xCD9E8D57u * (uint64_t)c.z;
        uint4 n;
        n.x = xor3((uint32_t)(b >> 32), c.y, k0);
        n.y = (uint32_t)b;
        n.z = xor3((uint32_t)(a >> 32), c.w, k1);
        n.w = (uint32_t)a;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ uint32_t word_of(uint4 v, int i)
{
    return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

__device__ __forceinline__ bool inst_live(const Inst &I, int k) { return k < I.nT && I.status[0] == 0; }

// A value or pointer known to be the same in all lanes, in scalar registers
// (values read through pointers would stay in vector registers, and branches
// on them mask lanes).
template <typename V>
__device__ __forceinline__ V scalar(V v)
{
    return (V)__builtin_amdgcn_readfirstlane((int)v);
}
template <typename P>
__device__ __forceinline__ P *scalar_ptr(P *p)
{
    const uint64_t a = (uint64_t)p;
    return (P *)((uint64_t)scalar((uint32_t)a) | ((uint64_t)scalar((uint32_t)(a >> 32)) << 32));
}

// v of the lane that the DPP control names, and folds over a wave from it:
// lanes 1, 2, 4 and 8 away by DPP (half mirror and mirror stand for 4 and 8:
// by then the lanes of a quad, of eight, agree), 16 and 32 away by the row
// swaps.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, ((uint64_t)dpp32<CTRL>((uint32_t)(b >> 32)) << 32) | dpp32<CTRL>((uint32_t)b));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor4 = 0x141, kXor8 = 0x140;
// both values that a lane and the one 16 or 32 away hold, the lower lane's first
struct Pair32 {
    uint32_t lo, hi;
};
__device__ __forceinline__ Pair32 both16(uint32_t v)
{
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return Pair32{p[0], p[1]};
}
__device__ __forceinline__ Pair32 both32(uint32_t v)
{
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return Pair32{p[0], p[1]};
}
template <typename Op>
__device__ __forceinline__ int32_t wave_fold(int32_t v, Op op)
{
    v = op(v, (int32_t)dpp32<kXor1>((uint32_t)v));
    v = op(v, (int32_t)dpp32<kXor2>((uint32_t)v));
    v = op(v, (int32_t)dpp32<kXor4>((uint32_t)v));
    v = op(v, (int32_t)dpp32<kXor8>((uint32_t)v));
    Pair32 p = both16((uint32_t)v);
    v = op((int32_t)p.lo, (int32_t)p.hi);
    p = both32((uint32_t)v);
    return op((int32_t)p.lo, (int32_t)p.hi);
}

// Pairwise tree sum of the values of each aligned group of n = 2^p <= 64
// lanes: node i of the next level is node 2i + node 2i+1 (the sum of two
// values is the same in either order, so both lanes of a pair compute it).
__device__ __forceinline__ double wave_tree(double v, int n)
{
    if (n > 1) v = v + dpp64<kXor1>(v);
    if (n > 2) v = v + dpp64<kXor2>(v);
    if (n > 4) v = v + dpp64<kXor4>(v);
    if (n > 8) v = v + dpp64<kXor8>(v);
    if (n > 16) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const Pair32 l = both16((uint32_t)b), h = both16((uint32_t)(b >> 32));
        v = __builtin_bit_cast(double, ((uint64_t)h.lo << 32) | l.lo) + __builtin_bit_cast(double, ((uint64_t)h.hi << 32) | l.hi);
    }
    if (n > 32) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const Pair32 l = both32((uint32_t)b), h = both32((uint32_t)(b >> 32));
        v = __builtin_bit_cast(double, ((uint64_t)h.lo << 32) | l.lo) + __builtin_bit_cast(double, ((uint64_t)h.hi << 32) | l.hi);
    }
    return v;
}

// Pairwise tree sum of the values of threads 0 .. n-1, n = 2^p <= blockDim
// (at most 1024): the waves' subtrees in registers, their roots through
// roots[16] in LDS.  Two barriers (a level at a time through LDS took two
// each, 20 for 1024 values).
__device__ __forceinline__ double wg_tree(double v, int n, double *roots)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = n > 64 ? n >> 6 : 1;
    v = wave_tree(v, n < 64 ? n : 64);
    if (lane == 0 && wave < nw) roots[wave] = v;
    __syncthreads();
    v = wave_tree(roots[lane & (nw - 1)], nw);
    __syncthreads();
    return v;
}

// The same of the n values a[0..n) held in LDS (after a barrier).
__device__ __forceinline__ double lds_pairwise(double *a, int n)
{
    const double v = (int)threadIdx.x < n ? a[threadIdx.x] : 0.0;
    __syncthreads();
    return wg_tree(v, n, a);
}

// Pairwise tree sum of n = 2^p leaves leaf(0..n).  T = the largest power of
// two <= min(blockDim, NT) threads take part: aligned chunks of 2T leaves
// are subtrees of the global tree; each is folded, then the chunk roots are.
// a holds 16 doubles, roots one per chunk; n <= 2 T blockDim.
template <int NT, typename Leaf>
__device__ __forceinline__ double tree_sum(int n, Leaf leaf, double *a, double *roots)
{
    const int t = threadIdx.x;
    int T = 1;
    while (2 * T <= (int)blockDim.x && 2 * T <= NT) T <<= 1;
    if (n == 1) return wg_tree(t == 0 ? leaf(0) : 0.0, 1, a);
    const int chunk = 2 * T;
    if (n <= chunk) return wg_tree(2 * t < n ? leaf(2 * t) + leaf(2 * t + 1) : 0.0, n / 2, a);
    const int nchunks = n / chunk;
    for (int c = 0; c < nchunks; ++c) {
        const double r = wg_tree(t < T ? leaf(c * chunk + 2 * t) + leaf(c * chunk + 2 * t + 1) : 0.0, T, a);
        if (t == 0) roots[c] = r;
    }
    __syncthreads();
    return lds_pairwise(roots, nchunks);
}

// w[m] = product over the set bits b of m < 2^17, ascending, of
// pw[b] = rho^(2^b).  The first nine factors are read at once (a loop over the
// set bits waited for LDS at each).
constexpr int kLevelBits = 17;
__device__ __forceinline__ double level_weight(const double *pw, uint32_t m)
{
    double x = 1.0, f[9];
#pragma unroll
    for (int b = 0; b < 9; ++b) f[b] = pw[b];
#pragma unroll
    for (int b = 0; b < 9; ++b) x = (m >> b) & 1u ? x * f[b] : x;
    for (int b = 9; (m >> b) != 0; ++b)
        if ((m >> b) & 1u) x = x * pw[b];
    return x;
}

// w = product over the set bits b of D (< 2^40), ascending, of pw[b].
__device__ __forceinline__ double weight64(const double *pw, uint64_t D)
{
    double x = 1.0;
    for (int b = 0; D != 0; ++b, D >>= 1)
        if (D & 1u) x = x * pw[b];
    return x;
}

// ---------------------------------------------------------------------------
// Metropolis acceptance with real couplings.  exp(x) in binary32 for
// -23 <= x <= 0 by a fixed recipe of correctly rounded steps: Cody-Waite
// reduction x = n ln 2 + r, n = rint(x log2 e), with ln 2 split into a head
// of 16 significant bits (n times it is exact) and a tail; the Taylor
// polynomial of degree 7 in r (|r| <= ln(2)/2) by Horner's rule with fused
// multiply-adds; scaling by 2^n.  Any IEEE implementation of the same steps
// returns the same bits, so decisions are reproducible.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float exp_recipe(float x)
{
    const float n = __builtin_rintf(x * 1.44269504f);
    float r = __builtin_fmaf(-n, 0.693145751953125f, x);
    r = __builtin_fmaf(-n, 1.42860677e-06f, r);
    float p = 1.0f / 5040.0f;
    p = __builtin_fmaf(p, r, 1.0f / 720.0f);
    p = __builtin_fmaf(p, r, 1.0f / 120.0f);
    p = __builtin_fmaf(p, r, 1.0f / 24.0f);
    p = __builtin_fmaf(p, r, 1.0f / 6.0f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    return __builtin_ldexpf(p, (int)n);
}

// A move with dE > 0 (units of 2^-20) at bq = beta 2^-20 (binary32) is
// accepted when x = -(bq dE) >= -23 and e = exp(x) >= 1 or u < floor(e 2^32).
// The recipe's argument is x clamped to [-24, 0] (dE <= 0 taken as 0): every
// decision is unchanged and its conversions stay in range for any dE.
__device__ __forceinline__ bool real_accept(float bq, int32_t dE, uint32_t u)
{
    const float x = -(bq * (float)max(dE, 0));
    const float e = exp_recipe(__builtin_fmaxf(x, -24.0f));
    const uint32_t T = (uint32_t)((e < 1.0f ? e : 0.0f) * 4294967296.0f);
    return x >= -23.0f && (e >= 1.0f || u < T);
}

// threadIdx.x for the end of a sweep workgroup, opaque: lane masks and
// addresses that follow from it are made there, not hoisted before the sweeps
// and spilled for them.
__device__ __forceinline__ int late_thread()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Adds one count per valid lane to arr[idx], one atomic per distinct index of
// the wave: at low temperature most replicas share a few energies, and per-lane
// atomics on one address would serialise.  Every lane of the wave must call it.
__device__ __forceinline__ void count_wave(uint32_t *arr, uint32_t idx, bool valid)
{
    const int lane = late_thread() & 63;
    uint64_t pending = __ballot(valid);
    while (pending) {
        const int leader = __builtin_ctzll(pending);
        const uint32_t li = __builtin_amdgcn_readlane(idx, leader);
        const uint64_t same = __ballot(valid && idx == li) & pending;
        if (lane == leader) atomicAdd(&arr[li], (uint32_t)__builtin_popcountll(same));
        pending &= ~same;
    }
}

// The same where equal indices come in runs of consecutive lanes: one count
// per run, all in one instruction.
__device__ __forceinline__ void count_runs(uint32_t *arr, uint32_t idx, bool valid)
{
    const int lane = late_thread() & 63;
    const uint32_t left = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (lane - 1), (int)idx);
    const uint64_t on = __ballot(valid);
    const bool head = valid && (lane == 0 || !((on >> (lane - 1)) & 1u) || left != idx);
    // a run ends at the next head or the next lane without a row
    const uint64_t stop = (__ballot(head) | ~on) & ~(((uint64_t)2 << lane) - 1);
    if (head) atomicAdd(&arr[idx], (uint32_t)((stop ? __builtin_ctzll(stop) : 64) - lane));
}

// Called by every workgroup of an instance at the end of its work in a
// launch: returns true in exactly one workgroup, the last to finish, after
// which the writes of all the others are visible to it.
//   kStores: the last workgroup reads plain stores of the others.  Each
// workgroup releases its writes (device scope: an L2 write-back, the L2s of
// the XCDs not being coherent) before it counts itself in.
//   else: it reads only what the others changed with device-scope atomics,
// which are performed at the memory the XCDs share; each wave waits for its
// own to complete, and no cache is written back (the write-backs of a sweep
// launch's thousands of workgroups, each with its tile of spins dirty in the
// L2, took longer than its sweeps at L = 8).
// Only the last workgroup acquires (an L2 invalidate); a full fence in every
// workgroup would also invalidate the L2 under all the workgroups still
// running.
template <bool kStores = true>
__device__ __forceinline__ bool last_workgroup(uint32_t *counter, int expected)
{
    __shared__ int is_last;
    if constexpr (!kStores) __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        if constexpr (kStores) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        is_last = atomicAdd(counter, 1u) == (uint32_t)(expected - 1);
    }
    __syncthreads();
    if (!is_last) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x == 0) *counter = 0u;
    return true;
}

// Part c of the energy histogram.
__device__ __forceinline__ uint32_t *hist_copy(const Inst &I, int c)
{
    return c == 0 ? I.hist : I.loff + (size_t)(c - 1) * I.nlev;
}

// The buffer that holds the population once the sweeps of the step are done:
// a sweep through the copy map wrote the other one, and the roles move on
// when the post launch finishes.
__device__ __forceinline__ int swept_buffer(const Inst &I) { return *I.cur ^ *I.mapped; }

}  // namespace pamc
