// gather.hip -- stand-alone copy of the surviving replicas into the other
// population buffer (the gather step of the resampling, paper Sec. II.B), for
// gfx950.  The default path fuses this copy into the next sweep's tile load;
// this kernel serves runs with the fusion off and the export of a population,
// whose rows the last two kernels convert.
#include <algorithm>

#include "launch.h"
#include "pamc_dev.h"

namespace pamc {

// ---------------------------------------------------------------------------
// Stand-alone gather of surviving replicas: destination row d of the other
// buffer receives source row map[d] (spins, energy, family).  Used when the
// gather is not fused into the next sweep and to materialise a population
// for export.  Runs after the step index has moved to the new population;
// a one-workgroup launch then moves the buffer roles on.  (Having the last
// workgroup of the gather do that instead costs a device-scope release fence
// in every one of its many short workgroups, which slowed the gather about
// five-fold.)
// A work item is a block of w.n destination rows (about 32 KB of spins);
// each thread keeps four 16-byte loads in flight before its stores.  The
// rows are written with nontemporal (streaming) stores: the new population
// is not read again before the next sweep, and ordinary stores let it evict
// the source rows from the caches, which costs a third to half of the
// bandwidth at these sizes.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void store_streaming(uint4 *p, uint4 v)
{
    const u32x4 x = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(p));
}

__global__ __launch_bounds__(256) void k_gather(const Inst *insts, const Work *work)
{
    const Work w = work[blockIdx.x];
    const Inst &I = insts[w.inst];
    const int k = *I.k;
    if (k >= I.nT || I.status[0] || !*I.mapped) return;
    const int Rn = (int)I.Rk[k];
    const int row0 = (int)w.row0;
    const int rows = min((int)w.n, Rn - row0);
    if (rows <= 0) return;
    const int cur = *I.cur;
    const int per_row = I.srow_bytes >> 4;
    const int total = rows * per_row;
    const uint4 *src = reinterpret_cast<const uint4 *>(I.spins[cur]);
    uint4 *dst = reinterpret_cast<uint4 *>(I.spins[cur ^ 1]);
    const int nt = (int)blockDim.x;
    for (int base = threadIdx.x; base < total; base += 4 * nt) {
        uint4 v[4];
        size_t to[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int it = base + u * nt;
            if (it < total) {
                const int q = it / per_row, c = it - q * per_row;
                const uint32_t d = (uint32_t)(row0 + q);
                v[u] = src[(size_t)I.map[d] * per_row + c];
                to[u] = (size_t)d * per_row + c;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (base + u * nt < total) store_streaming(dst + to[u], v[u]);
    }
    for (int q = threadIdx.x; q < rows; q += nt) {
        const uint32_t d = (uint32_t)(row0 + q), s = I.map[d];
        if (I.real)
            I.Eq[cur ^ 1][d] = I.Eq[cur][s];
        else
            I.E[cur ^ 1][d] = I.E[cur][s];
        I.fam[cur ^ 1][d] = I.fam[cur][s];
    }
}

// ---------------------------------------------------------------------------
// Rows of the current population as a caller holds them (+-1 per site, sites
// in lexicographic order) and back, for stored states.  A thread writes four
// bytes (k_export) or 32 storage positions (k_import); the reads within a row
// are scattered but stay in the caches, and both kernels take less time than
// the copy to or from the host (20000 rows of L = 10: below 0.1 ms, where the
// host took 20 ms).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_export(const Inst *inst, int8_t *out, int row0, int rows)
{
    const Inst &I = *inst;
    const uint32_t N = (uint32_t)I.N;
    const uint8_t *src = I.spins[*I.cur] + (size_t)row0 * I.srow_bytes;
    const uint64_t total = (uint64_t)rows * N;
    for (uint64_t at = 4 * ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x); at < total;
         at += 4 * (uint64_t)gridDim.x * blockDim.x) {
        uint32_t r = (uint32_t)(at / N), s = (uint32_t)(at - (uint64_t)r * N), v = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (at + j >= total) break;
            const uint8_t *row = src + (size_t)r * I.srow_bytes;
            const uint32_t p = I.pos[s];
            const uint32_t up = I.packed ? (row[p >> 3] >> (p & 7)) & 1u : row[p];
            v |= (up ? 0x01u : 0xFFu) << (8 * j);
            if (++s == N) s = 0, ++r;
        }
        if (at + 4 <= total) {
            *reinterpret_cast<uint32_t *>(out + at) = v;
        } else {
            for (int j = 0; at + j < total; ++j) out[at + j] = (int8_t)(v >> (8 * j));
        }
    }
}

__global__ __launch_bounds__(256) void k_import(const Inst *inst, const int8_t *in, int row0, int rows)
{
    const Inst &I = *inst;
    const int nw = I.srow_bytes >> 2, per = I.packed ? 32 : 4;  // words of a stored row, positions of a word
    uint32_t *dst = reinterpret_cast<uint32_t *>(I.spins[0] + (size_t)row0 * I.srow_bytes);
    const uint64_t total = (uint64_t)rows * nw;
    for (uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; at < total; at += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t r = (uint32_t)(at / nw), w = (uint32_t)(at - (uint64_t)r * nw);
        const int8_t *row = in + (size_t)r * I.N;
        uint32_t v = 0;
        for (int j = 0; j < per; ++j) {
            const int p = (int)w * per + j;
            const uint32_t s = p < I.row_bytes ? I.lexof[p] : 0xFFFFu;
            if (s != 0xFFFFu && row[s] > 0) v |= 1u << (I.packed ? j : 8 * j);
        }
        dst[at] = v;
    }
}

static unsigned state_blocks(int64_t threads) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(8192, (threads + 255) / 256)); }
void launch_export(const Inst *inst, int N, int8_t *out, int row0, int rows, hipStream_t st)
{
    if (rows) k_export<<<state_blocks(((int64_t)rows * N + 3) / 4), 256, 0, st>>>(inst, out, row0, rows);
}
void launch_import(const Inst *inst, int srow_bytes, const int8_t *in, int row0, int rows, hipStream_t st)
{
    if (rows) k_import<<<state_blocks((int64_t)rows * srow_bytes / 4), 256, 0, st>>>(inst, in, row0, rows);
}

void launch_gather(const Inst *insts, const Work *work, int nwork, hipStream_t st)
{
    if (nwork) k_gather<<<nwork, 256, 0, st>>>(insts, work);
}

}  // namespace pamc
