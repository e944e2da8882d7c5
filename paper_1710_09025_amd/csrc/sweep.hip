// sweep.hip -- initial population, energies and the checkerboard Metropolis
// sweeps with real couplings (paper Sec. II.B and Sec. III.A) for gfx950; the
// sweeps with +-1 couplings are in sweep_rb.hip.
//
// A block loads a tile of replica rows into LDS, runs all N_S sweeps of the
// current temperature on chip, recomputes each replica's energy (Eq. (1))
// from the final spins, and writes the rows back once.  When the previous
// resampling left a copy map, the tile is read through it, so the gather of
// surviving replicas costs no separate pass over HBM.  The epilogue adds the
// tile to the step's energy moments and the family counts.
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

__device__ __forceinline__ void replica_barrier(int tpr)
{
    if (tpr <= 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Byte offset, in a replica-quad slot, of storage position p (p < row_bytes;
// the complement's positions follow at 4 plane_bytes).
__device__ __forceinline__ uint32_t quad_pos(uint32_t p, uint32_t plane_bytes)
{
    return (p & 3u) * plane_bytes + 4u * (p >> 2);
}

__device__ __forceinline__ uint32_t lds_word(const uint8_t *lds, uint32_t a)
{
    return *reinterpret_cast<const uint32_t *>(lds + a);
}

// ---------------------------------------------------------------------------
// Colour-major sweep with real couplings (Sec. II.A: Gaussian J in fixed
// point, J = j 2^-20).  A thread group sweeps four replicas at once from one
// LDS slot in which the byte lanes of a word are the replicas: storage
// position p of the four is the word at plane(p) plane_bytes + 4 (p >> 2),
// plane(p) = p & 3, each spin a byte 0x00 / 0xFF (converted on load and
// store): one 32-bit read of a neighbour word returns
// that neighbour's spin in all four replicas, and its XOR with the site's own
// word is, per byte, 0 or -1 for sigma = [S != S_nb] = 0 or 1.  With
// S S_nb = 1 - 2 sigma,
//   dE = 2 S sum_d J_d S_d = 2 sum_d J_d - 4 sum_d sigma_d J_d,
// where sigma_d J_d is the sign-extended byte ANDed with j.  Each
// thread keeps the 24 neighbour addresses and couplings of its block of every
// colour in registers.  Energy: every bond is seen from both of its sites, so E = -sum_b J_b + sum over sites of sum_d sigma_d J_d.
// ---------------------------------------------------------------------------
struct CQBlock {
    uint32_t nb[24];  // LDS offsets of the neighbour words, [direction][site]
    int32_t j[24];    // coupling of each of those bonds (units of 2^-20)
    int32_t j2[4];        // twice the sum of the couplings of each site
    uint32_t own;     // LDS offset of site 0's word (site i at + i plane_bytes)
    uint32_t vbits;   // bit i set when site i of the block is a real site
    uint32_t ctr;     // Philox counter word 0
    bool has;
};

// sum_d sigma_d J_d of site i of block b for the four replicas (bytes of the
// XOR words, 0x00 or 0xFF), given the site's own word.
__device__ __forceinline__ void cq_field(const uint8_t *lds, const CQBlock &b, int i, uint32_t own,
                                         int32_t (&a)[4])
{
    a[0] = a[1] = a[2] = a[3] = 0;
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const uint32_t x = own ^ lds_word(lds, b.nb[4 * d + i]);
        const int32_t jj = b.j[4 * d + i];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] += (int32_t)(int8_t)(uint8_t)(x >> (8 * r)) & jj;
    }
}

// 0/1 spin bytes to 0x00/0xFF (255 b per byte, no carries) and back.
__device__ __forceinline__ uint32_t spin_ff(uint32_t w) { return (w << 8) - w; }
__device__ __forceinline__ uint4 spin_ff4(uint4 v)
{
    return make_uint4(spin_ff(v.x), spin_ff(v.y), spin_ff(v.z), spin_ff(v.w));
}
__device__ __forceinline__ uint4 spin_01(uint4 v)
{
    return make_uint4(v.x & 0x01010101u, v.y & 0x01010101u, v.z & 0x01010101u, v.w & 0x01010101u);
}

template <int NCOL, bool ALL>
__device__ __forceinline__ void cq_passes(const Inst &I, int k, uint8_t *lds, const CQBlock (&blk)[NCOL], float bq,
                                          unsigned long long *eacc, const TileIO &io, int r0, int nrows, int phase)
{
    const int tpr = I.tpr;
    const int RPG = (int)blockDim.x / tpr;
    const int ps = I.plane_bytes;
    const int lane_r = (int)threadIdx.x % tpr, qsub = (int)threadIdx.x / tpr;
    uint8_t *slot = lds + qsub * I.slot_bytes;
    const int nvec = I.row_bytes >> 4, pvec = ps >> 4;
    const uint32_t key0 = I.key0, key1 = I.key1;
    for (int qb = 0; qb < nrows; qb += 4 * RPG) {
        const int q0 = qb + 4 * qsub;
        const bool act = qsub < RPG && q0 < nrows;  // the last wave's spare lanes idle
        const uint32_t r0q = (uint32_t)(r0 + q0);
        if (act) {
            const uint8_t *src[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t r = r0q + j;
                src[j] = q0 + j < nrows ? io.src + (size_t)(io.map ? io.map[r] : r) * io.srow : nullptr;
            }
            uint4 *sp = reinterpret_cast<uint4 *>(slot);
            for (int i = lane_r; i < nvec; i += tpr) {
                uint4 v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = src[j] ? stored_vec(io, src[j], i) : make_uint4(0u, 0u, 0u, 0u);
                uint32_t ox[4], oy[4], oz[4], ow[4];
                transpose4(v[0].x, v[1].x, v[2].x, v[3].x, ox);
                transpose4(v[0].y, v[1].y, v[2].y, v[3].y, oy);
                transpose4(v[0].z, v[1].z, v[2].z, v[3].z, oz);
                transpose4(v[0].w, v[1].w, v[2].w, v[3].w, ow);
#pragma unroll
                for (int pl = 0; pl < 4; ++pl) sp[pl * pvec + i] = spin_ff4(make_uint4(ox[pl], oy[pl], oz[pl], ow[pl]));
            }
        }
        replica_barrier(tpr);
        const int t1 = phase_t1(I, phase);
        for (int t = phase_t0(I, phase); t < t1; ++t) {
#pragma unroll
            for (int c = 0; c < NCOL; ++c) {
                const CQBlock &b = blk[c];
                if (act && b.has) {
                    // raised issue priority for the field reads: a wave whose
                    // reads are due goes ahead of the others' multiply chains
                    if constexpr (!ALL) __builtin_amdgcn_s_setprio(1);
                    uint32_t own[4], flip[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        own[i] = lds_word(lds, b.own + i * ps);
                        flip[i] = (b.vbits >> i) & 1u ? 0xFFFFFFFFu : 0u;
                    }
                    if constexpr (!ALL) {
                        // the fields (24 neighbour reads) before the draws,
                        // whose arithmetic then covers the reads' latency
                        int32_t aa[4][4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) cq_field(lds, b, i, own[i], aa[i]);
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_setprio(0);
                        uint4 u[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            u[j] = philox10(make_uint4(b.ctr, r0q + j, (uint32_t)k, kTagSweep | (uint32_t)t), key0, key1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int32_t *a = aa[i];
                            uint32_t acc = 0;
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int32_t dE = b.j2[i] - 4 * a[r];
                                const bool ok = dE <= 0 || real_accept(bq, dE, word_of(u[r], i));
                                acc |= (ok ? 0xFFu : 0u) << (8 * r);
                            }
                            flip[i] &= acc;
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *reinterpret_cast<uint32_t *>(lds + b.own + i * ps) = own[i] ^ flip[i];
                }
                replica_barrier(tpr);
            }
        }
        if (act && phase != 1) {
            // per replica, sum over the thread's sites of sum_d sigma_d J_d:
            // at most 12 sites x 6 bonds x 2^23 < 2^30
            int32_t e[4] = {0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < NCOL; ++c) {
                if (!blk[c].has) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int32_t a[4];
                    cq_field(lds, blk[c], i, lds_word(lds, blk[c].own + i * ps), a);
#pragma unroll
                    for (int r = 0; r < 4; ++r) e[r] += a[r];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (q0 + j < nrows) atomicAdd(&eacc[q0 + j], (unsigned long long)(long long)e[j]);
        }
        if (act) {
            const uint4 *sp = reinterpret_cast<const uint4 *>(slot);
            for (int i = lane_r; i < nvec; i += tpr) {
                uint4 w[4];
#pragma unroll
                for (int pl = 0; pl < 4; ++pl) w[pl] = spin_01(sp[pl * pvec + i]);
                uint32_t ox[4], oy[4], oz[4], ow[4];
                transpose4(w[0].x, w[1].x, w[2].x, w[3].x, ox);
                transpose4(w[0].y, w[1].y, w[2].y, w[3].y, oy);
                transpose4(w[0].z, w[1].z, w[2].z, w[3].z, oz);
                transpose4(w[0].w, w[1].w, w[2].w, w[3].w, ow);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (q0 + j < nrows)
                        store_vec(io, io.dst + (size_t)(r0q + j) * io.srow, i, make_uint4(ox[j], oy[j], oz[j], ow[j]));
            }
        }
        replica_barrier(tpr);
    }
}

template <int NCOL>
__device__ __forceinline__ void sweep_tile_cq(const Inst &I, int k, uint8_t *lds, int r0, int nrows, int tile_rows,
                                              int phase)
{
    const int tpr = I.tpr;
    const int RPG = (int)blockDim.x / tpr;
    const int ps = I.plane_bytes;
    unsigned long long *eacc = reinterpret_cast<unsigned long long *>(lds + RPG * I.slot_bytes + 32);
    const TileIO io = tile_io(I);
    const int lane_r = (int)threadIdx.x % tpr, qsub = (int)threadIdx.x / tpr;
    const uint32_t slot = (uint32_t)(qsub * I.slot_bytes);
    CQBlock blk[NCOL];
#pragma unroll
    for (int c = 0; c < NCOL; ++c) {
        const int g = lane_r;
        blk[c].has = g < I.gcs[c];
        blk[c].ctr = ((uint32_t)c << 24) | (uint32_t)g;
        const int gg = blk[c].has ? g : 0;
        const uint16_t *d = I.cmdesc + ((size_t)c * I.gmax + gg) * 32;
        const int32_t *jd = I.cmj + ((size_t)c * I.gmax + gg) * 24;
#pragma unroll
        for (int i = 0; i < 24; ++i) {
            blk[c].nb[i] = slot + quad_pos((uint32_t)d[i], (uint32_t)ps);
            blk[c].j[i] = jd[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int32_t s2 = 0;
#pragma unroll
            for (int dd = 0; dd < 6; ++dd) s2 += blk[c].j[4 * dd + i];
            blk[c].j2[i] = 2 * s2;
        }
        const uint32_t vm = blk[c].has ? (uint32_t)d[24] | ((uint32_t)d[25] << 16) : 0u;
        blk[c].vbits = (vm & 1u) | ((vm >> 7) & 2u) | ((vm >> 14) & 4u) | ((vm >> 21) & 8u);
        blk[c].own = slot + (uint32_t)(I.cbase[c] + 4 * gg);
    }
    const float bq = I.bq[k];
    const bool all = I.thr[k].w != 0;
    for (int q = threadIdx.x; q < tile_rows; q += blockDim.x) eacc[q] = 0ull;
    __syncthreads();
    if (all)
        cq_passes<NCOL, true>(I, k, lds, blk, bq, eacc, io, r0, nrows, phase);
    else
        cq_passes<NCOL, false>(I, k, lds, blk, bq, eacc, io, r0, nrows, phase);
    __syncthreads();
    if (io.map)
        for (int q = threadIdx.x; q < nrows; q += blockDim.x) io.fdst[r0 + q] = io.fsrc[io.map[r0 + q]];
    if (phase == 1) return;
    tile_energies_real(I, io, eacc, r0, nrows, I.Jtot);
    __syncthreads();
    uint32_t *fam = reinterpret_cast<uint32_t *>(eacc);  // (the energies are out)
    for (int q = threadIdx.x; q < nrows; q += blockDim.x) fam[q] = io.fsrc[io.map ? io.map[r0 + q] : r0 + q];
    __syncthreads();
    tile_family_count(I, fam, nrows);
}

template <int NCOL, int MAXT>
__global__ __launch_bounds__(MAXT, 2) void k_sweep_cq(const Inst *insts, const Work *work, int tile_rows, int phase)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const Work w = work[blockIdx.x];
    const Inst &I = inst_ref(insts, w.inst);
    const int k = *I.k;
    if (k >= I.nT || I.status[0]) return;
    const int Rk = (int)I.Rk[k];
    const int r0 = (int)w.row0;
    const int nrows = min(tile_rows, Rk - r0);
    if (nrows > 0) sweep_tile_cq<NCOL>(I, k, lds, r0, nrows, tile_rows, phase);
    if (phase == 1) phase1_done(I, w.n);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t sweep_kernels_init()
{
    hipError_t r = sweep_rb_init();
    if (r == hipSuccess) r = sweep_rs_init();
    if (r == hipSuccess) r = sweep_rq_init();
    if (r != hipSuccess) return r;
    const void *fns[] = {
        reinterpret_cast<const void *>(&k_sweep_cq<2, 512>), reinterpret_cast<const void *>(&k_sweep_cq<2, 1024>),
        reinterpret_cast<const void *>(&k_sweep_cq<3, 512>), reinterpret_cast<const void *>(&k_sweep_cq<3, 1024>),
    };
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSweepLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
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

// Default workgroup shape of the colour-major sweep: 256 / tpr quads for
// quads of at most 64 threads; above, the number of quads (of at most 512
// threads together) that leaves the fewest idle lanes in the last wave, the
// one nearest 256 threads among equals.
int cm_replicas_per_block(int tpr)
{
    if (tpr <= 64) return 256 / tpr;
    int best = 1;
    double best_use = 0.0;
    for (int rp = 1; rp * tpr <= 512 || rp == 1; ++rp) {
        const int nt = rp * tpr;
        const double use = (double)nt / (double)cm_launch_threads(tpr, rp);
        const bool nearer = std::abs(nt - 256) < std::abs(best * tpr - 256);
        if (use > best_use + 1e-9 || (use > best_use - 1e-9 && nearer)) {
            best = rp;
            best_use = use;
        }
    }
    return best;
}

void launch_sweep(const SweepShape &sh, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st)
{
    if (!nwork) return;
    const int variant = sh.variant, tile_rows = sh.tile_rows, row_bytes = sh.row_bytes, tpr = sh.tpr, rp = sh.rp;
    if (variant == kSweepRB) {
        if (rs_small(sh.G, sh.M, sh.sets))
            launch_sweep_rs(sh, insts, work, nwork, phase, st);
        else
            launch_sweep_rb(sh, insts, work, nwork, phase, st);
        return;
    }
    if (is_rq(variant)) {
        launch_sweep_rq(sh, insts, work, nwork, phase, st);
        return;
    }
    if (variant == kSweepCQ2 || variant == kSweepCQ3) {
        // rp replica quads of four planes, and a 64-bit energy per tile row
        const size_t lds = (size_t)cm_slot_bytes(row_bytes, tpr, 4) * rp + 32 + 8 * (size_t)tile_rows;
        const int nt = cm_launch_threads(tpr, rp);
        if (variant == kSweepCQ2) {
            if (nt <= 512)
                k_sweep_cq<2, 512><<<nwork, nt, lds, st>>>(insts, work, tile_rows, phase);
            else
                k_sweep_cq<2, 1024><<<nwork, nt, lds, st>>>(insts, work, tile_rows, phase);
        } else {
            if (nt <= 512)
                k_sweep_cq<3, 512><<<nwork, nt, lds, st>>>(insts, work, tile_rows, phase);
            else
                k_sweep_cq<3, 1024><<<nwork, nt, lds, st>>>(insts, work, tile_rows, phase);
        }
        return;
    }
}

}  // namespace pamc
