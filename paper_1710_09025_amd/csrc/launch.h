// launch.h -- host-side launchers of the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "pamc_dev.h"

namespace pamc {

// RB: +-1 couplings, replicas as bits of an LDS word; RQ: the same with real
// couplings, on the cubic (3) or square (2) lattice, with thresholds per site
// in LDS where they fit and pay, else bond sums, else couplings.
enum SweepVariant {
    kSweepRB = 64,
    kSweepRQ3Thr = 128,
    kSweepRQ3Field = 192,
    kSweepRQ2Thr = 256,
    kSweepRQ2Field = 320,
    kSweepRQ3Bonds = 384
};
enum RQKind { kRQThr, kRQField, kRQBonds };  // a table of thresholds, of bond sums, or of couplings

// What a sweep launch needs to know of its instances' lattice and shape.
struct SweepShape {
    int variant = 0, tile_rows = 0, row_bytes = 0;
    int G = 0, plane = 0; // Philox blocks of the largest colour, words per site plane
    int ncol = 0;         // colours
    int M = 0, sets = 0;  // replicas per word (or kSiteWord + replicas per lane), sets of them per pass of a workgroup
};

// Dynamic LDS that every kernel may be launched with: gfx950 gives one
// workgroup up to 160 KB, of which 12 KB stay for static LDS.
constexpr int kMaxSweepLds = 160 * 1024 - 12 * 1024;
// Lets every sweep kernel launch with its dynamic LDS (above the default of
// 64 KB); returns the HIP status.
hipError_t sweep_kernels_init();

// What the options tile_rows and group_replicas may ask for, and which
// lattices real couplings cover, is laid down in quads of replicas: rp quads
// of four (eight, +-1 couplings) byte planes in the workgroup's LDS, tpr
// threads each (one per Philox block of the largest colour, up to 64 a power
// of two).  Plane stride, threads, and stride of a quad in LDS:
inline int cm_plane_bytes(int row_bytes) { return row_bytes <= 64 ? row_bytes : (row_bytes + 255) & ~255; }
inline int cm_launch_threads(int tpr, int rp) { return (tpr * rp + 63) / 64 * 64; }
inline int cm_slot_bytes(int row_bytes, int tpr, int planes)
{
    const int base = planes * cm_plane_bytes(row_bytes);
    if (tpr >= 64) return base;
    const int want = 4 * (tpr < 4 ? 4 : tpr);  // bytes, modulo 256
    return base + (((want - base) % 256) + 256) % 256;
}
// quads of a workgroup that asks for none
int cm_replicas_per_block(int tpr);

// The replica-word sweep: LDS words of a set's site plane (plane i holds
// site i of every four-site block of a row; a multiple of 64 words for rows
// of more than 128 bytes, so that every plane starts at bank 0), whether a
// workgroup sweeps one set, its threads and dynamic LDS for `sets` sets.
inline int rb_plane(int row_bytes) { return row_bytes <= 128 ? row_bytes / 4 : (row_bytes / 4 + 63) & ~63; }
bool rb_uniform(int G);
int rb_threads(int G, int sets);
size_t rb_lds(int plane, int sets);
// Its form for up to kSmallWord replicas a word (and at most 512 threads), in
// the same workgroups of threads: whether a shape takes it, and its LDS.
constexpr int kSmallWord = 4;
bool rs_small(int G, int m, int sets);
size_t rs_lds(int plane, int G, int sets);
// The form whose words are the four sites of a block of one replica (L = 8 and
// 16): M = kSiteWord + replicas per lane, one thread per block and set.
constexpr int kSiteWord = 32;
bool sw_form(int L, int m);
int sw_threads(int G, int sets);
size_t sw_lds(int row_bytes, int m, int sets);
// The same with real couplings, the tables included (thresholds or bond sums
// by the rows of a pass).  These kernels have
// little LDS of their own.
constexpr int64_t kMaxWordLds = 160 * 1024 - 2048;
bool rq_uniform(int G);
int rq_threads(int G, int sets);
int rq_kind(int variant, int rows);
int64_t rq_lds(int variant, int plane, int m, int sets);

// LDS of one cluster-move pair (the island search of one lane group): the
// sector flags of every lexicographic site (a byte: bit 0 where the replicas
// differ, bit 1 where they agree), the visited bits, the
// island queue (16-bit site indices; an island lies in the smaller sector,
// so it holds at most (N + 1) / 2 sites) and its tail, each part a multiple
// of 16 bytes, so that every pair's slice starts 16-byte aligned.
constexpr int icm_pair_bytes(int N)
{
    return ((N + 15) & ~15) + ((4 * ((N + 31) / 32) + 15) & ~15) + ((2 * ((N + 1) / 2) + 15) & ~15) + 16;
}
// the largest lattice the library accepts (L = 32) fits one pair per workgroup
static_assert(icm_pair_bytes(32 * 32 * 32) <= kMaxSweepLds, "cluster-move pair exceeds the LDS of a workgroup");

// lds_bytes: staging for packed rows (max(16384, row_bytes) when any instance
// of the launch is packed, else 0)
void launch_init(const Inst *insts, const Work *work, int nwork, size_t lds_bytes, hipStream_t st);
void launch_energy(const Inst *insts, const Work *work, int nwork, const int8_t *const *Jraw, hipStream_t st);
// sweeps of one temperature step and energies (phase 0: all N_S sweeps; with
// cluster moves, phase 1: the first floor(N_S/2) sweeps without energies,
// phase 2: the rest with them)
void launch_sweep(const SweepShape &shape, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st);
void launch_sweep_rb(const SweepShape &shape, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st);
hipError_t sweep_rb_init();
void launch_sweep_rs(const SweepShape &shape, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st);
hipError_t sweep_rs_init();
void launch_sweep_sw(const SweepShape &shape, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st);
hipError_t sweep_sw_init();
void launch_sweep_rq(const SweepShape &shape, const Inst *insts, const Work *work, int nwork, int phase, hipStream_t st);
hipError_t sweep_rq_init();
// resampling weights and their normaliser (instances with real couplings;
// work items are 1024-row blocks)
void launch_weights(const Inst *insts, const Work *work, int nwork, hipStream_t st);
// one round of isoenergetic cluster moves (work items: instance, pair
// index); N: the largest lattice of the launch (sizes the LDS)
void launch_icm(const Inst *insts, const Work *work, int nwork, int N, int round, hipStream_t st);
hipError_t icm_kernels_init();
// copy counts, family entropy, overlap; the last workgroup of each instance
// finishes the prefix sum and advances the step
void launch_post(const Inst *insts, const Work *work, int nwork, hipStream_t st);
// copy map of the resampling just done
void launch_expand(const Inst *insts, const Work *work, int nwork, hipStream_t st);
void launch_gather(const Inst *insts, const Work *work, int nwork, hipStream_t st);
// rows [row0, row0 + rows) of the current buffer as +-1 bytes in lexicographic
// order (4-byte aligned `out`), and such rows into buffer 0
void launch_export(const Inst *inst, int N, int8_t *out, int row0, int rows, hipStream_t st);
void launch_import(const Inst *inst, int srow_bytes, const int8_t *in, int row0, int rows, hipStream_t st);
void launch_flip(const Inst *insts, const uint32_t *list, int n, hipStream_t st);

}  // namespace pamc
