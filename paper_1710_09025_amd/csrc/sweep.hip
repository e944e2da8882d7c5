// sweep.hip -- initial population and energies (paper Sec. II.B) for gfx950,
// and the choice of the kernel that runs the checkerboard Metropolis sweeps
// (Sec. III.A): +-1 couplings in sweep_rb.hip, sweep_rs.hip and sweep_sw.hip
// (few replicas a lane), real couplings in sweep_rq.hip.
//
// A sweep workgroup loads replica rows into LDS, runs all N_S sweeps of the
// current temperature on chip, recomputes each replica's energy (Eq. (1))
// from the final spins, and writes the rows back once.  When the previous
// resampling left a copy map, the rows are read through it, so the gather of
// surviving replicas costs no separate pass over HBM.
//
// Random numbers: the draw for a site of colour c whose rank among the
// sites of that colour is i, in replica row r, step k and sweep t, is word
// (i & 3) of Philox4x32-10 at counter ((c << 24) | (i >> 2), r, k,
// TAG_SWEEP | t) under the run's key.
#include "launch.h"
#include "pamc_dev.h"
#include "step_common.h"
#include "tile_io.h"

namespace pamc {

__device__ __forceinline__ const Inst &inst_ref(const Inst *insts, uint32_t i) { return insts[i]; }

// Storage position of lexicographic site s in a replica row.
__device__ __forceinline__ int storage_pos(const Inst &I, int s) { return I.pos[s]; }

// Spin (0/1) at storage position p of a stored row.
__device__ __forceinline__ int stored_spin(const Inst &I, const uint8_t *row, int p)
{
    return I.packed ? (row[p >> 3] >> (p & 7)) & 1 : row[p];
}

// ---------------------------------------------------------------------------
// Initial replicas (Sec. II.B: random configurations at beta = 0).  Site s
// of row r takes S = +1 when bit 31 of word (s & 3) of Philox at counter
// (s >> 2, r, 0, TAG_INIT) is set.  One thread per Philox block; gridDim.y
// workgroups share the 1024 rows of a work item.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init(const Inst *insts, const Work *work)
{
    extern __shared__ __align__(16) uint8_t stage[];
    Work w = work[blockIdx.x];
    const Inst &I = inst_ref(insts, w.inst);
    const int nq = (I.N + 3) >> 2;
    const int per = kRowsPerBlock / (int)gridDim.y;
    w.row0 += blockIdx.y * per;
    const int rows = min(per, I.R - (int)w.row0);
    if (!I.packed) {
        uint8_t *sp = I.spins[0];
        for (int it = threadIdx.x; it < rows * nq; it += blockDim.x) {
            const int q = it / nq, b = it - q * nq;
            const uint32_t r = w.row0 + q;
            const uint4 v = philox10(make_uint4((uint32_t)b, r, 0u, kTagInit), I.key0, I.key1);
            for (int j = 0; j < 4; ++j) {
                const int s = 4 * b + j;
                if (s >= I.N) break;
                sp[(size_t)r * I.row_bytes + storage_pos(I, s)] = (uint8_t)(word_of(v, j) >> 31);
            }
        }
    } else {
        // rows staged as bytes in LDS (16 KB, or one row), then packed
        const int nvec = I.row_bytes >> 4;
        const int rpi = max(1, 16384 / I.row_bytes);
        uint4 *st16 = reinterpret_cast<uint4 *>(stage);
        for (int q0 = 0; q0 < rows; q0 += rpi) {
            const int nr = min(rpi, rows - q0);
            for (int i = threadIdx.x; i < nr * nvec; i += blockDim.x) st16[i] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            for (int it = threadIdx.x; it < nr * nq; it += blockDim.x) {
                const int q = it / nq, b = it - q * nq;
                const uint32_t r = w.row0 + q0 + q;
                const uint4 v = philox10(make_uint4((uint32_t)b, r, 0u, kTagInit), I.key0, I.key1);
                for (int j = 0; j < 4; ++j) {
                    const int s = 4 * b + j;
                    if (s >= I.N) break;
                    stage[q * I.row_bytes + storage_pos(I, s)] = (uint8_t)(word_of(v, j) >> 31);
                }
            }
            __syncthreads();
            for (int i = threadIdx.x; i < nr * nvec; i += blockDim.x) {
                const int q = i / nvec, c = i - q * nvec;
                uint16_t *dst = reinterpret_cast<uint16_t *>(I.spins[0] + (size_t)(w.row0 + q0 + q) * I.srow_bytes);
                dst[c] = (uint16_t)bytes_to_bits16(st16[i]);
            }
            __syncthreads();
        }
    }
    for (int q = threadIdx.x; q < rows; q += blockDim.x) I.fam[0][w.row0 + q] = w.row0 + q;
}

// ---------------------------------------------------------------------------
// Energies of the rows of the current buffer, Eq. (1): E = -sum over the
// D N bonds (s, s + e_d) of J S_s S_{s+e_d} (D = 3, or 2 on the square
// lattice, real couplings only).  One wave per row; gridDim.y workgroups
// share the 1024 rows of a work item.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_energy(const Inst *insts, const Work *work, const int8_t *const *Jraw)
{
    Work w = work[blockIdx.x];
    const Inst &I = inst_ref(insts, w.inst);
    const int k = *I.k;
    if (k >= I.nT) return;
    const int per = kRowsPerBlock / (int)gridDim.y;
    w.row0 += blockIdx.y * per;
    const int Rk = (int)I.Rk[k];
    const int cur = *I.cur;
    const int8_t *J = Jraw[w.inst];
    const int L = I.L, N = I.N;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (I.real) {
        // real couplings: int32 [D][N] in units of 2^-20, 64-bit sums; on
        // the square lattice z = 0 and the z bond is absent
        const int32_t *Jq = reinterpret_cast<const int32_t *>(J);
        const int Lz = I.dim == 3 ? L : 1;
        for (int q = wave; q < per; q += 4) {
            const int r = (int)w.row0 + q;
            if (r >= Rk) break;
            const uint8_t *S = I.spins[cur] + (size_t)r * I.srow_bytes;
            long long e = 0;
            for (int s = lane; s < N; s += 64) {
                const int x = s % L, y = (s / L) % L, z = s / (L * L);
                const int ss = 2 * stored_spin(I, S, storage_pos(I, s)) - 1;
                const int nb[3] = {(x + 1) % L + L * (y + L * z), x + L * ((y + 1) % L + L * z),
                                   x + L * (y + L * ((z + 1) % Lz))};
                for (int d = 0; d < I.dim; ++d)
                    e -= (long long)Jq[d * N + s] * (ss * (2 * stored_spin(I, S, storage_pos(I, nb[d])) - 1));
            }
            for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
            if (lane == 0) I.Eq[cur][r] = e;
        }
        return;
    }
    for (int q = wave; q < per; q += 4) {
        const int r = (int)w.row0 + q;
        if (r >= Rk) break;
        const uint8_t *S = I.spins[cur] + (size_t)r * I.srow_bytes;
        int e = 0;
        for (int s = lane; s < N; s += 64) {
            const int x = s % L, y = (s / L) % L, z = s / (L * L);
            const int ss = 2 * stored_spin(I, S, storage_pos(I, s)) - 1;
            const int nb[3] = {(x + 1) % L + L * (y + L * z), x + L * ((y + 1) % L + L * z),
                               x + L * (y + L * ((z + 1) % L))};
            for (int d = 0; d < 3; ++d)
                e -= J[d * N + s] * ss * (2 * stored_spin(I, S, storage_pos(I, nb[d])) - 1);
        }
        for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off);
        if (lane == 0) I.E[cur][r] = e;
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t sweep_kernels_init()
{
    hipError_t r = sweep_rb_init();
    if (r == hipSuccess) r = sweep_rs_init();
    if (r == hipSuccess) r = sweep_sw_init();
    if (r == hipSuccess) r = sweep_rq_init();
    return r;
}

// Workgroups per work item of 1024 rows: down to 8 rows each where there are
// few items (whole items in one workgroup left most of the chip idle: 70 ms
// for the 4000 rows of an L = 24 run).
static unsigned row_slices(int nwork)
{
    unsigned s = 1;
    while (s < 128 && s * (unsigned)nwork < 4096) s *= 2;
    return s;
}

void launch_init(const Inst *insts, const Work *work, int nwork, size_t lds_bytes, hipStream_t st)
{
    if (nwork) k_init<<<dim3(nwork, row_slices(nwork)), 256, lds_bytes, st>>>(insts, work);
}

void launch_energy(const Inst *insts, const Work *work, int nwork, const int8_t *const *Jraw, hipStream_t st)
{
    if (nwork) k_energy<<<dim3(nwork, row_slices(nwork)), 256, 0, st>>>(insts, work, Jraw);
}

void launch_sweep(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    if (!nwork) return;
    if (sh.variant != kSweepRB)
        launch_sweep_rq(sh, insts, work, nwork, phase, st);
    else if (sh.M > kSiteWord)
        launch_sweep_sw(sh, insts, work, nwork, phase, st);
    else if (rs_small(sh.G, sh.M, sh.sets))
        launch_sweep_rs(sh, insts, work, nwork, phase, st);
    else
        launch_sweep_rb(sh, insts, work, nwork, phase, st);
}

}  // namespace pamc
