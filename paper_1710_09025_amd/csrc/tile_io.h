// tile_io.h -- device routines shared by the sweep kernels: the rows of a tile
// (through the copy map or in place, one byte or one bit per spin), the byte
// transpose between rows and replica words, and the end of a sweep workgroup
// (energies, family counts).
#pragma once
#include "pamc_dev.h"
#include "step_common.h"

namespace pamc {

// Packed spin rows: bit p of a row (bit p & 7 of byte p >> 3) is the spin at
// storage position p.
__device__ __forceinline__ uint32_t bytes_to_bits4(uint32_t w)
{
    // byte i (0 or 1) lands on bit 24 + i of w * (2^24 + 2^17 + 2^10 + 2^3)
    return (uint32_t)(((uint64_t)w * 0x01020408ull) >> 24) & 15u;
}
__device__ __forceinline__ uint32_t bytes_to_bits16(uint4 v)
{
    return bytes_to_bits4(v.x) | (bytes_to_bits4(v.y) << 4) | (bytes_to_bits4(v.z) << 8) | (bytes_to_bits4(v.w) << 12);
}
// ---------------------------------------------------------------------------
// Shared tile load / store.  Rows of the tile come from buffer `cur`, either
// directly (in place) or through the copy map (then they go to the other
// buffer, with their family ids).
// ---------------------------------------------------------------------------
struct TileIO {
    const uint8_t *src;
    uint8_t *dst;
    const uint32_t *map;  // nullptr: identity
    const uint32_t *fsrc;
    uint32_t *fdst;
    int32_t *Edst;
    int64_t *Eqdst;       // real couplings: 64-bit energies
    int packed;           // stored rows hold one bit per position
    int srow;             // bytes per stored row
};

__device__ __forceinline__ TileIO tile_io(const Inst &I)
{
    TileIO io;
    // (both buffers' pointers are read at once, not the one that cur picks
    // after it has arrived)
    uint8_t *const s0 = I.spins[0], *const s1 = I.spins[1];
    uint32_t *const f0 = I.fam[0], *const f1 = I.fam[1], *const map = I.map;
    int32_t *const e0 = I.E[0], *const e1 = I.E[1];
    int64_t *const q0 = I.Eq[0], *const q1 = I.Eq[1];
    io.packed = I.packed;
    io.srow = I.srow_bytes;
    const int cur = *I.cur, mapped = *I.mapped, out = cur ^ mapped;
    // (uniform, but the compiler cannot know: as lane values the pointers were
    // spilled to memory for the sweeps.  With late_thread at the workgroup's
    // end 20 bytes a thread instead of 76, 0.5 GB a launch at L = 16,
    // R = 5 10^5; L = 8, R = 10^5, 201 temperatures 47.1 -> 46.3 ms)
    io.src = scalar_ptr(cur ? s1 : s0);
    io.dst = scalar_ptr(out ? s1 : s0);
    io.map = scalar_ptr(mapped ? map : nullptr);
    io.fsrc = scalar_ptr(cur ? f1 : f0);
    io.fdst = scalar_ptr(mapped ? (out ? f1 : f0) : nullptr);
    io.Edst = scalar_ptr(out ? e1 : e0);
    io.Eqdst = scalar_ptr(out ? q1 : q0);
    return io;
}

// Energies of the tile's rows, stored and (populations too large for the
// measurement to read them all) counted.  The workgroups count into
// hist_copies histograms in turn: a launch's atomics fall on the same hundred
// bins or less, and those on one address follow each other about 0.1 us apart.
__device__ __forceinline__ void tile_energy_out(const Inst &I, const TileIO &io, const int *unsat, int r0, int nrows)
{
    const int copies = I.hist_copies;
    uint32_t *hist = copies > 0 ? hist_copy(I, (int)blockIdx.x % copies) : nullptr;
    for (int base = 0; base < nrows; base += blockDim.x) {
        const int q = base + late_thread();
        const bool valid = q < nrows;
        int E = 0;
        if (valid) {
            E = 2 * unsat[q] - 3 * I.N;
            io.Edst[r0 + q] = E;
        }
        if (copies > 0) count_wave(hist, (uint32_t)((E + 3 * I.N) >> 1), valid);
    }
}

// Descendants per family: a tile's rows counted under their family ids fam[]
// (sorted, unless a caller's imported state is not: then the runs are short),
// where the population is too large for the statistics to count them all.
__device__ __forceinline__ void tile_family_count(const Inst &I, const uint32_t *fam, int nrows)
{
    if (I.Rcap <= kDirectRows) return;
    for (int base = 0; base < nrows; base += blockDim.x) {
        const int q = base + late_thread();
        const bool valid = q < nrows;
        count_runs(I.cnt, valid ? fam[q] : 0u, valid);
    }
}

// Energies of the tile's rows (real couplings), and the lowest of them; the other moments are taken with the weights.
// (All of them here, with 128-bit sums through LDS and five atomics a
// workgroup, took 7 us of a workgroup's 170 at L = 8, R = 10^5.)
__device__ __forceinline__ void tile_energies_real(const Inst &I, const TileIO &io, const unsigned long long *eacc,
                                                   int r0, int nrows)
{
    const int t = late_thread();
    for (int q0 = scalar(t & ~63); q0 < nrows; q0 += blockDim.x) {
        const int q = q0 + (t & 63);
        long long e = kNoEnergy;
        if (q < nrows) {
            e = (long long)eacc[q];
            io.Eqdst[r0 + q] = e;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const long long o = __shfl_xor(e, off);
            e = o < e ? o : e;
        }
        if (q == q0) atomicMin(I.emin + blockIdx.x % kMinParts, e);
    }
}

// A sweep launch runs the whole step (phase 0) or, for runs with cluster
// moves, the first floor(N_S/2) sweeps (phase 1: through the copy map, no
// energies) and later the remaining ones (phase 2: in place, with energies
// and the measurement).

// End of phase 1 in the last workgroup: the population now lives in the
// buffer the tiles were written to.
__device__ __forceinline__ void phase1_done(const Inst &I, uint32_t tiles)
{
    const bool last = last_workgroup<false>(&I.sync[0], (int)tiles);
    if (last && threadIdx.x == 0 && *I.mapped) {
        *I.cur ^= 1;
        *I.mapped = 0;
    }
}

// 4 x 4 byte transpose: word k of the result holds byte k of w0, w1, w2, w3
// (v_perm selectors: bytes 0-3 of the second operand, 4-7 of the first).
// It is its own inverse.
__device__ __forceinline__ void transpose4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t (&o)[4])
{
    const uint32_t a_lo = __builtin_amdgcn_perm(w1, w0, 0x05010400u);  // [w0.0 w1.0 w0.1 w1.1]
    const uint32_t a_hi = __builtin_amdgcn_perm(w1, w0, 0x07030602u);  // [w0.2 w1.2 w0.3 w1.3]
    const uint32_t b_lo = __builtin_amdgcn_perm(w3, w2, 0x05010400u);
    const uint32_t b_hi = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(b_lo, a_lo, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(b_lo, a_lo, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(b_hi, a_hi, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(b_hi, a_hi, 0x07060302u);
}

}  // namespace pamc
