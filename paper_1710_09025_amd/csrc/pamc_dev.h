// pamc_dev.h -- data layout shared by the host orchestrator and the gfx950
// kernels of the population annealing library.
//
// Every kernel is segmented by instance: it reads the instance descriptor
// `Inst` from device memory, so one run, a batch of mixed-size instances and
// the serving loop all use the same kernels.  The current temperature step
// k of each instance lives on the device, so a step can be captured once in
// a hipGraph and replayed.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// (Device arithmetic shared by the kernels -- Philox, the three-way xor --
// lives in step_common.h, which only the kernel sources include.)

namespace pamc {

// Philox stream tags, the top four bits of counter word 3.
constexpr uint32_t kTagInit = 0x10000000u;
constexpr uint32_t kTagSweep = 0x20000000u;
constexpr uint32_t kTagResample = 0x30000000u;
constexpr uint32_t kTagIcm = 0x40000000u;

// Spin storage inside one replica row: colour-major, one position per site
// (0: S = -1, 1: S = +1).  The sites of colour 0 in lexicographic order, then
// colour 1 (and 2 for odd L), each colour padded to a multiple of four, so
// that the four sites of one Philox block are positions 4 b ... 4 b + 3 for
// every L.

constexpr int kRowsPerBlock = 1024;  // rows handled per block by row kernels
constexpr int kDirectRows = 32768;    // populations (capacity) up to this size are measured (+-1 couplings) and their families counted row by row
constexpr int kMapRows = 4096;        // populations (capacity) up to this size get their copy map in the post launch
constexpr int kOvlPairs = 2048;      // replica pairs per overlap workgroup (few workgroups: most steps measure no overlap)
constexpr int kOvlLdsBins = 8194;    // overlap histograms up to this many bins (L <= 16) are built in LDS

// Per-step integer record written on the device.  Energies are in units of
// 2^-20 for real couplings.
struct StepRec {
    int64_t R;        // R_k
    int64_t sumE;     // sum of E
    uint64_t sumE2;   // sum of E^2: low 64 bits of the exact 128-bit sum
    int64_t sumE2_hi; //   and its high 64 bits
    int64_t Emin, Emax;
    double S;         // resampling normaliser (NaN at the last step)
    double T;         // family term sum n ln n
};

// Real couplings: the lowest energy of the step being swept, in kMinParts
// parts (one atomic of a sweep wave each; atomics on one address follow each
// other about 0.1 us apart), and the other moments of a block of 1024 rows
// (the squares' sum as two 64-bit halves).
constexpr int kMinParts = 64;
constexpr long long kNoEnergy = 0x7FFFFFFFFFFFFFFFll;
struct BlockMoments {
    long long emax;
    unsigned long long sum, sq_lo, sq_hi;
};

struct Inst {
    // problem
    int32_t L, N, ncol;
    int32_t dim;        // lattice dimension: 3 (cubic, N = L^3) or 2 (square, N = L^2; real couplings only)
    int32_t row_bytes;  // bytes per replica row in LDS, one byte per storage position (>= N, multiple of 16)
    int32_t packed;     // 1: the spin buffers hold one bit per storage position
    int32_t srow_bytes; // bytes per replica row in the spin buffers (row_bytes, or row_bytes / 8 rounded up to 16)
    int32_t nT, NS;
    uint32_t key0, key1;
    int32_t R;          // nominal population
    int32_t Rcap;       // rows per buffer
    int32_t nblk;       // ceil(Rcap / kRowsPerBlock)
    int32_t nlev;       // 3N + 1 energy levels
    int32_t fam_pow2;   // smallest power of two >= R (family tree leaves)
    int32_t ovl_n;      // number of overlap steps
    int32_t real;       // 1: real couplings in fixed point, J = j 2^-20 (int32 j, |J| < 8)
    int32_t icm;        // cluster-move rounds per step (0: none)
    double icm_bmin;    // cluster moves only at steps with beta_k >= icm_bmin
    // double-buffered population
    uint8_t *spins[2];
    int32_t *E[2];
    uint32_t *fam[2];
    // resampling scratch
    uint32_t *map;      // [Rcap] destination row -> source row
    uint32_t *loff;     // [Rcap] real couplings: first destination of each row inside its row block (+-1 couplings
                        //    keep those in the idle energy buffer); +-1 couplings: parts of the energy histogram
    uint32_t *bsum;     // [nblk]
    uint32_t *boff;     // [nblk]
    uint32_t *sync;     // [4] workgroups finished: 0 in the first sweep launch of a step with cluster moves, 1 in the post launch
    int32_t post_blocks;  // workgroups of this instance in a post launch
    uint32_t *hist;     // [nlev] energy histogram, (E + 3N)/2
    int32_t hist_copies;  // parts the sweep's workgroups count into: hist, and more in loff (cleared by k_expand);
                          //    0: at most kDirectRows rows, measured from their energies
    uint32_t *cnt;      // [R] descendants per family
    double *fpart;      // [max(1, fam_pow2 / 2048)] family tree partial sums
    // tables
    const uint4 *thr;   // [nT] (T(dE=4), T(8), T(12), accept_all)
    const double *beta; // [nT]
    const double *rho;  // [nT] exp(-2 (beta_{k+1} - beta_k)), host libm
    const double *Rt;   // [nT] nominal population R(beta_k) the resampling targets
    const double *nlnn; // [>= Rcap + 1] n ln n, host libm (shared)
    // per colour and Philox block 64 bytes: the LDS word indices (16 bits)
    // within a set of the six neighbours of its four sites
    // ([direction][site]), the sign bits (+-1 couplings, J = -1: bit 4 d + i)
    // and the mask of real sites
    const uint4 *rbtab; // [ncol][gmax][4]
    int32_t rb_plane;   // LDS words per site plane (rb_plane())
    const uint16_t *pos;// [N] storage position of each lexicographic site
    const uint16_t *lexof; // [row_bytes] lexicographic site at each storage position (0xFFFF: padding)
    int32_t cbase[3];   // first storage position of each colour
    int32_t gcs[3];     // Philox blocks of each colour
    int32_t gmax;       // ... of the largest
    // real couplings
    int64_t *Eq[2];     // energies, units of 2^-20
    double *wrep;       // [Rcap] resampling weight of each row
    double *wpart;      // [nblk] pairwise-tree roots of the 1024-row blocks
    long long *emin;    // [kMinParts], lowest energies of the step being swept
    const int32_t *cmj; // [ncol][gmax][24] couplings of a block's bonds, [direction][site]
    const float *bq;    // [nT] beta_k 2^-20 rounded to binary32
    const double *gpw;  // [nT][40] exp(-(beta_{k+1} - beta_k) 2^(b-20)), host libm
    // progress and records
    int32_t *k;         // current step (device scalar)
    int32_t *cur;       // buffer holding the current population (0/1)
    int32_t *mapped;    // 1: rows of the current step still live in buffer
                        //    cur through `map` (gather pending)
    uint32_t *Rk;       // [nT + 1]
    StepRec *rec;       // [nT]
    int32_t *ovl_slot;  // [nT] slot in qhist or -1
    uint32_t *qhist;    // [ovl_n][2N + 1]
    uint32_t *status;   // bit 0 capacity, bit 1 extinct; word 1: failing step
};

// Work item of the row-parallel kernels and of the sweep: instance index,
// first row (or first family id), and the role of a post-kernel workgroup.
enum PostRole : uint32_t { kRoleCopies = 0, kRoleFamilies = 1, kRoleOverlap = 2, kRoleMeasure = 3 };
struct Work {
    uint32_t inst;
    uint32_t row0;
    uint32_t role;   // k_post: what to do
    uint32_t n;      // sweeps: workgroups of the instance in the launch; gather: rows
};

}  // namespace pamc
