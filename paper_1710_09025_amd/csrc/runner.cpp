// runner.cpp -- host orchestration: validation results are assumed, this
// file builds the host tables (thresholds, weights' rho, n ln n), lays out
// each instance's device memory, builds the work lists of the segmented
// kernels and enqueues the per-step launch sequence.
#include "runner.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <set>

namespace pamc {

static thread_local std::string g_last_error;
void set_error(const std::string &msg) { g_last_error = msg; }
const char *last_error_cstr() { return g_last_error.c_str(); }

void *Allocator::get(size_t bytes)
{
    if (bytes == 0) bytes = 256;
    if (alloc) return alloc(bytes, user);
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) return nullptr;
    return p;
}

void Allocator::put(void *p)
{
    if (!p) return;
    if (free)
        free(p, user);
    else
        (void)hipFree(p);
}

int64_t default_capacity(int64_t R) { return R + (int64_t)std::ceil(8.0 * std::sqrt((double)R)) + 64; }


// Colour of site (x, y, z): checkerboard for even L; for odd L the proper
// three-colouring (g(x) + g(y) + g(z)) mod 3 with g(v) = v mod 2 below L-1
// and g(L-1) = 2.
static int colour_of(int L, int x, int y, int z)
{
    if ((L & 1) == 0) return (x + y + z) & 1;
    auto g = [L](int v) { return v == L - 1 ? 2 : (v & 1); };
    return (g(x) + g(y) + g(z)) % 3;
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Colour-major rows for every lattice.  Real couplings need a replica quad's
// slot of four byte planes in the workgroup's LDS and its largest colour in
// 1024 threads (even L up to 20, odd L up to 21); no kernel beyond it.  The
// square lattice (dim = 2) runs only with real couplings.  The replica-word
// kernels sweep what their tables of the sites' thresholds or bond sums leave
// LDS for: thresholds on cubic lattices up to L = 8 and square ones up to 45,
// bond sums up to L = 12 and on all other square ones, couplings beyond.
// (Thresholds that leave room for one set only are slower than bond sums, 879
// attempts per ns against 1017 at L = 48 on the square lattice, and bond sums
// than couplings, 490 against 783 at L = 13.)
LayoutInfo layout_for(int L, bool real, int dim)
{
    LayoutInfo li{};
    const int Lz = dim == 3 ? L : 1;
    const int N = L * L * Lz;
    li.ncol = (L & 1) ? 3 : 2;
    for (int z = 0; z < Lz; ++z)
        for (int y = 0; y < L; ++y)
            for (int x = 0; x < L; ++x) li.ncs[colour_of(L, x, y, z)]++;
    li.gmax = 1;
    for (int c = 0; c < 3; ++c) li.gmax = std::max(li.gmax, (li.ncs[c] + 3) / 4);
    int cb = 0;
    for (int c = 0; c < li.ncol; ++c) {
        li.cbase[c] = cb;
        cb += (li.ncs[c] + 3) & ~3;
    }
    li.row_bytes = (cb + 15) & ~15;
    // threads per replica quad: one per Philox block of the largest colour;
    // up to 64 blocks rounded up to a power of two, so that whole quads fit
    // in a wave and sync with wave barriers
    li.tpr = 1;
    if (li.gmax <= 64) {
        while (li.tpr < li.gmax) li.tpr <<= 1;
    } else {
        li.tpr = li.gmax;
    }
    li.valid = true;
    if (!real) {
        li.valid = dim == 3;
        li.variant = kSweepRB;
    } else if (li.tpr <= 1024 && 2 * li.row_bytes <= 65535 &&
               (size_t)cm_slot_bytes(li.row_bytes, li.tpr, 4) * cm_replicas_per_block(li.tpr) + 32 + 8 * 64 <= kMaxSweepLds) {
        const int thr = dim == 3 ? kSweepRQ3Thr : kSweepRQ2Thr, field = dim == 3 ? kSweepRQ3Field : kSweepRQ2Field;
        const int plane = rb_plane(li.row_bytes);
        li.variant = rq_lds(thr, plane, 32, 2) <= kMaxWordLds     ? thr
                     : rq_lds(field, plane, 32, dim == 3 ? 4 : 1) <= kMaxWordLds ? field
                     : kSweepRQ3Bonds;
    } else {
        li.valid = false;
    }
    return li;
}

namespace {
struct Carve {
    size_t off = 0;
    size_t take(size_t bytes)
    {
        const size_t o = off;
        off += align256(bytes);
        return o;
    }
};

struct InstLayout {
    size_t ctl, status, sync, spins0, spins1, E0, E1, f0, f1, map, loff, bsum, boff, hist, cnt, fpart, thr,
        beta, rho, Rt, rbtab, J, pos, lexof, Rk, rec, ovl_slot, qhist, Eq0, Eq1, wrep, wpart, emin, cmj,
        bq, gpw, total;
};

InstLayout layout_of(int L, int64_t R, int64_t Rcap, int nT, int n_ovl, bool packed, bool real, int dim)
{
    const int N = dim == 3 ? L * L * L : L * L;
    const LayoutInfo li = layout_for(L, real, dim);
    const int row_bytes = stored_row_bytes(li.row_bytes, packed);
    const int ncol = li.ncol;
    const int nblk = (int)((Rcap + kRowsPerBlock - 1) / kRowsPerBlock);
    const int nlev = 3 * N + 1;
    int64_t fp2 = 1;
    while (fp2 < R) fp2 <<= 1;
    const int gmax = li.gmax;
    Carve c;
    InstLayout l{};
    l.ctl = c.take(16);
    l.status = c.take(8);
    l.sync = c.take(16);
    l.spins0 = c.take((size_t)Rcap * row_bytes);
    l.spins1 = c.take((size_t)Rcap * row_bytes);
    l.E0 = c.take(real ? 16 : (size_t)Rcap * 4);
    l.E1 = c.take(real ? 16 : (size_t)Rcap * 4);
    l.f0 = c.take((size_t)Rcap * 4);
    l.f1 = c.take((size_t)Rcap * 4);
    l.map = c.take((size_t)Rcap * 4);
    l.loff = c.take((size_t)Rcap * 4);
    l.bsum = c.take((size_t)nblk * 4);
    l.boff = c.take((size_t)nblk * 4);
    l.hist = c.take(real ? 16 : (size_t)nlev * 4);
    l.cnt = c.take((size_t)R * 4);
    l.fpart = c.take((size_t)std::max<int64_t>(1, fp2 / 2048) * 8);
    l.thr = c.take((size_t)nT * 16);
    l.beta = c.take((size_t)nT * 8);
    l.rho = c.take((size_t)nT * 8);
    l.Rt = c.take((size_t)nT * 8);
    l.rbtab = c.take((size_t)ncol * gmax * 64);
    l.J = c.take((size_t)dim * N * (real ? 4 : 1));
    l.pos = c.take((size_t)N * 2);
    l.lexof = c.take((size_t)li.row_bytes * 2);
    l.Rk = c.take((size_t)(nT + 1) * 4);
    l.rec = c.take((size_t)nT * sizeof(StepRec));
    l.ovl_slot = c.take((size_t)nT * 4);
    l.qhist = c.take((size_t)std::max(1, n_ovl) * (2 * N + 1) * 4);
    // real couplings: 64-bit energies, per-row weights, block roots, moments,
    // couplings per neighbour word and the per-step scalars
    l.Eq0 = c.take(real ? (size_t)Rcap * 8 : 16);
    l.Eq1 = c.take(real ? (size_t)Rcap * 8 : 16);
    l.wrep = c.take(real ? (size_t)Rcap * 8 : 16);
    l.wpart = c.take(real ? (size_t)nblk * 8 : 16);
    l.emin = c.take(real ? kMinParts * 8 : 16);
    l.cmj = c.take(real ? (size_t)ncol * gmax * 24 * 4 : 16);
    l.bq = c.take((size_t)nT * 4);
    l.gpw = c.take(real ? (size_t)nT * 40 * 8 : 16);
    l.total = c.off;
    return l;
}
}  // namespace

int stored_row_bytes(int row_bytes, bool packed) { return packed ? (row_bytes + 127) / 128 * 16 : row_bytes; }

size_t inst_device_bytes(int L, int64_t Rcap, int nT, int n_ovl, bool packed, bool real, int dim)
{
    // R <= Rcap; use Rcap for the family counters as an upper bound
    return layout_of(L, Rcap, Rcap, nT, n_ovl, packed, real, dim).total;
}

Runner::~Runner()
{
    if (stream_) (void)hipStreamSynchronize(stream_);
    if (side_) (void)hipStreamSynchronize(side_);
    for (hipStream_t s : aux_) (void)hipStreamSynchronize(s);
    (void)release_fenced(true);
    for (size_t i = 0; i < inst_.size(); ++i)
        if (used_[i]) alloc_.put(inst_[i].block);
    for (void *p : work_allocs_) alloc_.put(p);
    for (hipEvent_t e : ev_pool_) (void)hipEventDestroy(e);
    for (hipEvent_t e : fence_pool_) (void)hipEventDestroy(e);
    if (stage_) (void)hipHostFree(stage_);
    if (side_) (void)hipStreamDestroy(side_);
    drop_graph();
    alloc_.put(d_insts_);
    alloc_.put(d_nlnn_);
    alloc_.put(d_Jptr_);
    for (hipEvent_t e : ev_join_) (void)hipEventDestroy(e);
    if (ev_fork_) (void)hipEventDestroy(ev_fork_);
    for (hipStream_t s : aux_) (void)hipStreamDestroy(s);
    if (own_stream_ && stream_) (void)hipStreamDestroy(stream_);
}

int Runner::dev_fail(hipError_t e, const char *what)
{
    poisoned_ = true;
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return PAMC_ERR_DEVICE;
}

#define HIPCHK(call, what)                                   \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return dev_fail(e_, what);     \
    } while (0)

int Runner::setup(const pamc_options &opt, int max_slots, bool external_stream)
{
    alloc_.alloc = opt.alloc;
    alloc_.free = opt.free;
    alloc_.user = opt.alloc_user;
    fuse_ = opt.fuse_gather != 0;
    timing_ = opt.timing != 0;
    graphs_ = opt.graphs != 0 && !timing_;
    max_slots_ = max_slots;
    if (opt.device >= 0) HIPCHK(hipSetDevice(opt.device), "hipSetDevice");
    HIPCHK(hipGetDevice(&device_), "hipGetDevice");
    HIPCHK(sweep_kernels_init(), "hipFuncSetAttribute (sweep LDS)");
    HIPCHK(icm_kernels_init(), "hipFuncSetAttribute (cluster-move LDS)");
    if (opt.stream || external_stream) {
        stream_ = (hipStream_t)opt.stream;
    } else {
        HIPCHK(hipStreamCreateWithFlags(&stream_, hipStreamNonBlocking), "hipStreamCreate");
        own_stream_ = true;
    }
    if (max_slots > 1) {
        for (int a = 0; a < kAuxStreams; ++a) {
            hipStream_t s = nullptr;
            hipEvent_t e = nullptr;
            HIPCHK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "hipStreamCreate (sweep groups)");
            aux_.push_back(s);
            HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming), "hipEventCreate (sweep groups)");
            ev_join_.push_back(e);
        }
        HIPCHK(hipEventCreateWithFlags(&ev_fork_, hipEventDisableTiming), "hipEventCreate (sweep groups)");
    }
    inst_.resize((size_t)max_slots);
    used_.assign((size_t)max_slots, 0);
    held_.assign((size_t)max_slots, 0);
    d_insts_ = (Inst *)alloc_.get(sizeof(Inst) * (size_t)max_slots);
    d_Jptr_ = (const int8_t **)alloc_.get(sizeof(void *) * (size_t)max_slots);
    if (!d_insts_ || !d_Jptr_) {
        set_error("device allocation failed (instance table)");
        return PAMC_ERR_NOMEM;
    }
    return PAMC_OK;
}

int Runner::enable_async(size_t staging_bytes)
{
    if (async_) return PAMC_OK;
    HIPCHK(hipStreamCreateWithFlags(&side_, hipStreamNonBlocking), "hipStreamCreate (uploads)");
    HIPCHK(hipHostMalloc((void **)&stage_, staging_bytes, hipHostMallocDefault), "hipHostMalloc (staging)");
    stage_cap_ = staging_bytes;
    stage_used_ = 0;
    async_ = true;
    return PAMC_OK;
}

int Runner::h2d(void *dst, const void *src, size_t bytes)
{
    if (bytes == 0) return PAMC_OK;
    if (!async_) {
        HIPCHK(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, stream_), "upload");
        return PAMC_OK;
    }
    const uint8_t *s = static_cast<const uint8_t *>(src);
    uint8_t *d = static_cast<uint8_t *>(dst);
    while (bytes > 0) {
        // the staging is reused once the copies issued from it have landed
        if (stage_used_ == stage_cap_) {
            HIPCHK(hipStreamSynchronize(side_), "staging sync");
            stage_used_ = 0;
        }
        const size_t n = std::min(bytes, stage_cap_ - stage_used_);
        std::memcpy(stage_ + stage_used_, s, n);
        HIPCHK(hipMemcpyAsync(d, stage_ + stage_used_, n, hipMemcpyHostToDevice, side_), "staged upload");
        stage_used_ = std::min(stage_cap_, stage_used_ + ((n + 63) & ~size_t(63)));
        s += n;
        d += n;
        bytes -= n;
    }
    return PAMC_OK;
}

int Runner::upload_sync()
{
    HIPCHK(hipStreamSynchronize(up_stream()), "upload sync");
    stage_used_ = 0;
    return PAMC_OK;
}

int Runner::d2h(void *dst, const void *src, size_t bytes)
{
    if (bytes == 0) return PAMC_OK;
    HIPCHK(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, up_stream()), "read back");
    HIPCHK(hipStreamSynchronize(up_stream()), "read back sync");
    return PAMC_OK;
}

int Runner::fence(std::vector<void *> ptrs, std::vector<int> slots)
{
    hipEvent_t e = nullptr;
    if (!fence_pool_.empty()) {
        e = fence_pool_.back();
        fence_pool_.pop_back();
    } else {
        HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming), "hipEventCreate (fence)");
    }
    HIPCHK(hipEventRecord(e, stream_), "hipEventRecord (fence)");
    for (int i : slots) held_[(size_t)i] = 1;
    fenced_.push_back(Fenced{e, std::move(ptrs), std::move(slots)});
    return PAMC_OK;
}

int Runner::release_fenced(bool wait)
{
    for (size_t j = 0; j < fenced_.size();) {
        Fenced &f = fenced_[j];
        hipError_t q = wait ? hipEventSynchronize(f.ev) : hipEventQuery(f.ev);
        if (q == hipErrorNotReady) {
            ++j;
            continue;
        }
        if (q != hipSuccess) return dev_fail(q, "fence");
        for (void *p : f.ptrs) alloc_.put(p);
        for (int i : f.slots) held_[(size_t)i] = 0;
        fence_pool_.push_back(f.ev);
        fenced_.erase(fenced_.begin() + (long)j);
    }
    return PAMC_OK;
}

int Runner::free_slots() const
{
    int n = 0;
    for (int i = 0; i < max_slots_; ++i)
        if (!used_[i] && !held_[i]) ++n;
    return n;
}

// n ln n for n = 0 .. len-1 (host libm), shared by all instances; grows when
// an instance with a larger capacity arrives.
int Runner::ensure_nlnn(int64_t len)
{
    if (len <= nlnn_len_) return PAMC_OK;
    // every queued step reads the table that is replaced
    HIPCHK(hipStreamSynchronize(stream_), "nlnn sync");
    if (side_) HIPCHK(hipStreamSynchronize(side_), "nlnn sync");
    const int64_t n = std::max(len, 2 * nlnn_len_);
    std::vector<double> nl((size_t)n);
    nl[0] = 0.0;
    for (int64_t q = 1; q < n; ++q) nl[(size_t)q] = (double)q * std::log((double)q);
    double *d = (double *)alloc_.get(nl.size() * 8);
    if (!d) {
        set_error("device allocation failed (n ln n table)");
        return PAMC_ERR_NOMEM;
    }
    HIPCHK(hipMemcpy(d, nl.data(), nl.size() * 8, hipMemcpyHostToDevice), "upload nlnn");
    for (size_t i = 0; i < inst_.size(); ++i) {
        if (!used_[i]) continue;
        inst_[i].dev.nlnn = d;
        HIPCHK(hipMemcpy(d_insts_ + i, &inst_[i].dev, sizeof(Inst), hipMemcpyHostToDevice), "update instance");
    }
    alloc_.put(d_nlnn_);
    d_nlnn_ = d;
    nlnn_len_ = n;
    return PAMC_OK;
}

int Runner::add_instance(HostInst &&h)
{
    int slot = -1;
    for (int i = 0; i < max_slots_; ++i)
        if (!used_[i] && !held_[i]) {
            slot = i;
            break;
        }
    if (slot < 0) {
        set_error("no free instance slot");
        return PAMC_ERR_BUSY;
    }
    int st = ensure_nlnn(h.Rcap + 1);
    if (st != PAMC_OK) return st;
    inst_[slot] = std::move(h);
    st = upload_inst(slot);
    if (st != PAMC_OK) {
        alloc_.put(inst_[slot].block);
        inst_[slot].block = nullptr;
        return st;
    }
    used_[slot] = 1;
    const int8_t *jp = inst_[slot].Jdev;
    st = h2d(d_insts_ + slot, &inst_[slot].dev, sizeof(Inst));
    if (st == PAMC_OK) st = h2d(d_Jptr_ + slot, &jp, sizeof(void *));
    if (st == PAMC_OK) st = upload_sync();
    if (st != PAMC_OK) return st;
    return slot;
}

void Runner::remove_instance(int slot)
{
    if (slot < 0 || slot >= max_slots_ || !used_[slot]) return;
    if (async_) {
        // queued steps may still read the instance: release it behind them
        (void)fence({inst_[slot].block}, {slot});
    } else {
        (void)hipStreamSynchronize(stream_);
        alloc_.put(inst_[slot].block);
    }
    inst_[slot] = HostInst();
    used_[slot] = 0;
}

int Runner::upload_inst(int i)
{
    HostInst &h = inst_[i];
    const int L = h.L, N = h.N;
    const InstLayout lay = layout_of(L, h.R, h.Rcap, h.nT, h.ovl_n, h.packed != 0, h.real != 0, h.dim);
    h.bytes = lay.total;
    h.block = alloc_.get(lay.total);
    if (!h.block) {
        set_error("device allocation of " + std::to_string(lay.total) + " bytes failed");
        return PAMC_ERR_NOMEM;
    }
    uint8_t *b = (uint8_t *)h.block;
    HIPCHK(hipMemsetAsync(b, 0, lay.total, up_stream()), "clear instance memory");
    Inst &d = h.dev;
    std::memset(&d, 0, sizeof(d));
    d.L = L;
    d.N = N;
    d.dim = h.dim;
    d.ncol = h.ncol;
    d.row_bytes = h.row_bytes;
    d.packed = h.packed;
    d.srow_bytes = h.srow_bytes;
    d.nT = h.nT;
    d.NS = h.NS;
    d.key0 = (uint32_t)h.seed;
    d.key1 = (uint32_t)(h.seed >> 32);
    d.R = (int32_t)h.R;
    d.Rcap = (int32_t)h.Rcap;
    d.nblk = (int32_t)((h.Rcap + kRowsPerBlock - 1) / kRowsPerBlock);
    d.nlev = 3 * N + 1;
    int64_t fp2 = 1;
    while (fp2 < h.R) fp2 <<= 1;
    d.fam_pow2 = (int32_t)fp2;
    d.ovl_n = h.ovl_n;
    d.spins[0] = b + lay.spins0;
    d.spins[1] = b + lay.spins1;
    d.E[0] = (int32_t *)(b + lay.E0);
    d.E[1] = (int32_t *)(b + lay.E1);
    d.fam[0] = (uint32_t *)(b + lay.f0);
    d.fam[1] = (uint32_t *)(b + lay.f1);
    d.map = (uint32_t *)(b + lay.map);
    d.loff = (uint32_t *)(b + lay.loff);
    d.bsum = (uint32_t *)(b + lay.bsum);
    d.boff = (uint32_t *)(b + lay.boff);
    d.hist = (uint32_t *)(b + lay.hist);
    // more histogram parts where the rows make hundreds of updates, as far as
    // loff holds them and the measurement (1024 threads) reads them in a few
    // microseconds
    d.hist_copies =
        h.real || h.Rcap <= kDirectRows ? 0 : (int32_t)(1 + std::min({(int64_t)63, h.Rcap / d.nlev, (int64_t)32768 / d.nlev, h.Rcap / 512}));
    d.cnt = (uint32_t *)(b + lay.cnt);
    d.fpart = (double *)(b + lay.fpart);
    d.thr = (const uint4 *)(b + lay.thr);
    d.beta = (const double *)(b + lay.beta);
    d.rho = (const double *)(b + lay.rho);
    d.Rt = (const double *)(b + lay.Rt);
    d.nlnn = d_nlnn_;
    d.rbtab = (const uint4 *)(b + lay.rbtab);
    d.rb_plane = rb_plane(h.row_bytes);
    d.pos = (const uint16_t *)(b + lay.pos);
    d.lexof = (const uint16_t *)(b + lay.lexof);
    d.k = (int32_t *)(b + lay.ctl);
    d.cur = d.k + 1;
    d.mapped = d.k + 2;
    d.Rk = (uint32_t *)(b + lay.Rk);
    d.rec = (StepRec *)(b + lay.rec);
    d.ovl_slot = (int32_t *)(b + lay.ovl_slot);
    d.qhist = (uint32_t *)(b + lay.qhist);
    d.status = (uint32_t *)(b + lay.status);
    d.sync = (uint32_t *)(b + lay.sync);
    d.real = h.real;
    d.icm = h.icm;
    d.icm_bmin = h.icm_bmin;
    d.Eq[0] = (int64_t *)(b + lay.Eq0);
    d.Eq[1] = (int64_t *)(b + lay.Eq1);
    d.wrep = (double *)(b + lay.wrep);
    d.wpart = (double *)(b + lay.wpart);
    d.emin = (long long *)(b + lay.emin);
    d.cmj = (const int32_t *)(b + lay.cmj);
    d.bq = (const float *)(b + lay.bq);
    d.gpw = (const double *)(b + lay.gpw);
    {
        const int64_t nchunks = std::max<int64_t>(1, fp2 / 2048);
        const int64_t novl = (h.Rcap / 2 + kOvlPairs - 1) / kOvlPairs;
        d.post_blocks = (int32_t)(d.nblk + nchunks + novl + 1);
    }
    h.ctl = d.k;
    h.Jdev = (int8_t *)(b + lay.J);

    // --- thresholds: T_k(dE) = floor(exp(-beta_k dE) 2^32), capped; beta = 0
    // accepts every move
    std::vector<uint32_t> thr((size_t)h.nT * 4);
    for (int k = 0; k < h.nT; ++k) {
        const double bk = h.beta[k];
        for (int j = 0; j < 3; ++j) {
            const double p = std::exp(-bk * (4.0 * (j + 1)));
            const double x = std::floor(p * 4294967296.0);
            thr[4 * k + j] = x >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)x;
        }
        thr[4 * k + 3] = bk == 0.0 ? 1u : 0u;
    }
    // --- rho_k = exp(-2 (beta_{k+1} - beta_k)): weight ratio of adjacent levels
    std::vector<double> rho((size_t)h.nT, 1.0);
    for (int k = 0; k + 1 < h.nT; ++k) {
        const double db = h.beta[k + 1] - h.beta[k];
        rho[k] = std::exp(-2.0 * db);
    }
    // --- colours and colour ranks
    const int Lz = h.dim == 3 ? L : 1;
    std::vector<int> col(N), rank(N);
    int ncs[3] = {0, 0, 0};
    for (int z = 0; z < Lz; ++z)
        for (int y = 0; y < L; ++y)
            for (int x = 0; x < L; ++x) {
                const int s = x + L * (y + L * z);
                col[s] = colour_of(L, x, y, z);
                rank[s] = ncs[col[s]]++;
            }
    for (int c = 0; c < 3; ++c) d.gcs[c] = (ncs[c] + 3) / 4;
    d.gmax = std::max(d.gcs[0], std::max(d.gcs[1], d.gcs[2]));
    // coupling of bond (dir, s): +-1, or j (units of 2^-20) for real couplings
    auto J = [&](int dir, int s) { return h.real ? (int)h.Jq[(size_t)dir * N + s] : (int)h.J[(size_t)dir * N + s]; };
    auto site_of = [L, Lz](int x, int y, int z) {
        return ((x % L + L) % L) + L * (((y % L + L) % L) + L * ((z % Lz + Lz) % Lz));
    };
    const LayoutInfo li = layout_for(L, h.real != 0, h.dim);
    for (int c = 0; c < 3; ++c) d.cbase[c] = li.cbase[c];
    // storage position of each site
    std::vector<int> lex_pos((size_t)N);
    std::vector<uint16_t> pos16((size_t)N);
    for (int s = 0; s < N; ++s) {
        lex_pos[s] = li.cbase[col[s]] + rank[s];
        pos16[s] = (uint16_t)lex_pos[s];
    }
    // its inverse over the storage positions of a row (cluster moves read
    // rows in storage order)
    std::vector<uint16_t> lexof16((size_t)h.row_bytes, (uint16_t)0xFFFF);
    for (int s = 0; s < N; ++s) lexof16[(size_t)lex_pos[s]] = (uint16_t)s;
    // per colour, Philox block and site: its six neighbours and couplings.
    // On the square lattice the two z entries of a site point at the site
    // itself with coupling 0 and are not read.  Padding sites point at
    // themselves.
    std::vector<int32_t> cmj;
    std::vector<uint32_t> rbtab;
    std::vector<int> site_at((size_t)3 * N, -1);
    for (int s = 0; s < N; ++s) site_at[(size_t)col[s] * N + rank[s]] = s;
    rbtab.assign((size_t)h.ncol * d.gmax * 16, 0u);
    if (h.real) cmj.assign((size_t)h.ncol * d.gmax * 24, 0);
    const bool sq = h.dim == 2;
    for (int c = 0; c < h.ncol; ++c)
        for (int g = 0; g < d.gcs[c]; ++g) {
            const size_t blk = (size_t)c * d.gmax + g;
            uint32_t vmask = 0;
            for (int bb = 0; bb < 4; ++bb) {
                const int i = 4 * g + bb;
                int nbp[6], jv[6] = {0, 0, 0, 0, 0, 0};
                if (i >= ncs[c]) {
                    for (int dd = 0; dd < 6; ++dd) nbp[dd] = li.cbase[c] + i;
                } else {
                    vmask |= 1u << (8 * bb);
                    const int s = site_at[(size_t)c * N + i];
                    const int x = s % L, y = (s / L) % L, z = s / (L * L);
                    // the bond to s - e_d is stored at the lower site
                    const int nb[6] = {site_of(x + 1, y, z), site_of(x - 1, y, z), site_of(x, y + 1, z),
                                       site_of(x, y - 1, z), sq ? s : site_of(x, y, z + 1),
                                       sq ? s : site_of(x, y, z - 1)};
                    for (int dd = 0; dd < 6; ++dd) {
                        nbp[dd] = lex_pos[nb[dd]];
                        jv[dd] = sq && dd >= 4 ? 0 : J(dd >> 1, dd & 1 ? nb[dd] : s);
                    }
                }
                for (int dd = 0; dd < 6; ++dd) {
                    const int e = 4 * dd + bb;
                    const uint32_t word = (uint32_t)((nbp[dd] & 3) * d.rb_plane + (nbp[dd] >> 2));
                    rbtab[blk * 16 + (e >> 1)] |= word << (16 * (e & 1));
                    if (h.real)
                        cmj[blk * 24 + e] = jv[dd];
                    else if (jv[dd] < 0)
                        rbtab[blk * 16 + 12] |= 1u << e;
                }
            }
            for (int bb = 0; bb < 4; ++bb)
                if ((vmask >> (8 * bb)) & 1u) rbtab[blk * 16 + 13] |= 1u << bb;
        }
    // real couplings: beta_k 2^-20 in binary32 and the weight factors
    // exp(-(beta_{k+1} - beta_k) 2^(b-20)), b < 40, host libm
    std::vector<float> bq((size_t)h.nT);
    for (int k = 0; k < h.nT; ++k) bq[(size_t)k] = (float)(h.beta[k] * 0x1p-20);
    std::vector<double> gpw;
    if (h.real) {
        gpw.assign((size_t)h.nT * 40, 1.0);
        for (int k = 0; k + 1 < h.nT; ++k) {
            const double db = h.beta[k + 1] - h.beta[k];
            for (int bb = 0; bb < 40; ++bb) gpw[(size_t)k * 40 + bb] = std::exp(-db * std::ldexp(1.0, bb - 20));
        }
    }
    const std::vector<long long> emin(h.real ? kMinParts : 0, kNoEnergy);
    std::vector<uint32_t> Rk0((size_t)h.nT + 1, 0u);
    Rk0[0] = (uint32_t)h.R;
    int32_t ctl[4] = {0, 0, 0, 0};
    int st = PAMC_OK;
    auto put = [&](size_t off, const void *src, size_t bytes) {
        if (st == PAMC_OK) st = h2d(b + off, src, bytes);
    };
    put(lay.ctl, ctl, 16);
    put(lay.thr, thr.data(), thr.size() * 4);
    put(lay.beta, h.beta.data(), h.beta.size() * 8);
    put(lay.rho, rho.data(), rho.size() * 8);
    put(lay.Rt, h.pop.data(), h.pop.size() * 8);
    put(lay.rbtab, rbtab.data(), rbtab.size() * 4);
    if (h.real)
        put(lay.J, h.Jq.data(), h.Jq.size() * 4);
    else
        put(lay.J, h.J.data(), h.J.size());
    put(lay.bq, bq.data(), bq.size() * 4);
    if (!emin.empty()) put(lay.emin, emin.data(), emin.size() * 8);
    if (!gpw.empty()) put(lay.gpw, gpw.data(), gpw.size() * 8);
    if (!cmj.empty()) put(lay.cmj, cmj.data(), cmj.size() * 4);
    put(lay.pos, pos16.data(), pos16.size() * 2);
    put(lay.lexof, lexof16.data(), lexof16.size() * 2);
    put(lay.Rk, Rk0.data(), Rk0.size() * 4);
    put(lay.ovl_slot, h.ovl_slot.data(), h.ovl_slot.size() * 4);
    // host vectors must outlive the async copies
    if (st == PAMC_OK) st = upload_sync();
    if (st != PAMC_OK) return st;
    h.k_enq = 0;
    h.k_base = 0;
    h.lnZ_base = (double)N * std::log(2.0);
    return PAMC_OK;
}

std::vector<Work> gather_items(uint32_t slot, int64_t Rcap, int row_bytes)
{
    const int g = std::max(1, std::min(1024, 32768 / row_bytes));
    std::vector<Work> v;
    for (int64_t r = 0; r < Rcap; r += g) v.push_back(Work{slot, (uint32_t)r, 0u, (uint32_t)g});
    return v;
}

int Runner::set_shape(int i, const HostInst &shape)
{
    if (i < 0 || i >= max_slots_ || !used_[i]) return PAMC_ERR_STATE;
    HostInst &h = inst_[i];
    take_shape(h, shape);
    return build_work(active_);
}

int Runner::build_work(const std::vector<int> &active)
{
    if (async_) {
        // the lists being replaced serve the steps already queued
        if (!work_allocs_.empty()) {
            const int st = fence(std::move(work_allocs_), {});
            if (st != PAMC_OK) return st;
        }
    } else {
        HIPCHK(hipStreamSynchronize(stream_), "build_work sync");
        drop_graph();
        for (void *p : work_allocs_) alloc_.put(p);
    }
    work_allocs_.clear();
    sweep_groups_.clear();
    active_ = active;
    auto upload = [&](const void *src, size_t bytes) -> void * {
        void *p = alloc_.get(bytes);
        if (!p) return nullptr;
        work_allocs_.push_back(p);
        if (h2d(p, src, bytes) != PAMC_OK) return nullptr;
        return p;
    };
    // by what a launch's instances share: the lattice, the shape, and
    // whether the launch is split around cluster moves
    std::map<std::tuple<int, int, int, int, int, int, int, int, int>, std::vector<Work>> groups;
    std::map<std::tuple<int, int, int, int, int, int, int, int, int>, SweepShape> shapes;
    std::vector<Work> rows, post, gath, wblk, icm;
    icm_rounds_ = 0;
    icm_N_ = 0;
    std::vector<uint32_t> list;
    // instances of one lattice without a shape of their own sweep in the
    // shape that suits their populations together (each its own: small words
    // that fill the chip alone; a launch of 36 real-coupled instances of
    // L = 4 ... 8 with 5000 rows each took 1.6 times as long)
    std::map<std::tuple<int, int, int>, std::vector<int64_t>> pops;
    std::map<std::tuple<int, int, int>, HostInst> joint;
    auto lattice = [](const HostInst &h) { return std::make_tuple(h.icm > 0 ? 1 : 0, h.variant, h.L); };
    std::set<std::tuple<int, int, int>> launches;
    for (int i : active) {
        if (!inst_[i].own_shape) pops[lattice(inst_[i])].push_back(inst_[i].R);
        launches.insert(lattice(inst_[i]));
    }
    const int beside = (int)std::min(launches.size(), aux_.size() + 1);
    for (int i : active) {
        HostInst &h = inst_[i];
        const uint32_t ii = (uint32_t)i;
        if (!h.own_shape) {
            HostInst &s = joint[lattice(h)];
            if (s.L == 0) {
                s.dim = h.dim;
                s.L = h.L;
                s.N = h.N;
                s.NS = h.NS;
                s.ncol = h.ncol;
                s.variant = h.variant;
                s.gmax = h.gmax;
                s.row_bytes = h.row_bytes;
                s.real = h.real;
                s.tpr = h.tpr;
                s.Rcap = h.Rcap;
                default_shape(s, pops[lattice(h)], beside);
            }
            h.tile_rows = s.tile_rows;
            h.rp = s.rp;
            h.mrep = s.mrep;
            h.sets = s.sets;
        }
        const auto key = std::make_tuple(h.icm > 0 ? 1 : 0, h.variant, h.L, h.tile_rows, h.row_bytes, h.tpr, h.rp, h.mrep,
                                         h.sets);
        auto &g = groups[key];
        SweepShape &sh = shapes[key];
        sh.variant = h.variant;
        sh.tile_rows = h.tile_rows;
        sh.row_bytes = h.row_bytes;
        sh.G = h.dev.gmax;
        sh.plane = h.dev.rb_plane;
        sh.ncol = h.ncol;
        sh.M = h.mrep;
        sh.sets = h.sets;
        if (h.icm > 0) {
            for (int64_t j = 0; j < h.Rcap / 2; ++j) icm.push_back(Work{ii, (uint32_t)j, 0u, 0u});
            icm_rounds_ = std::max(icm_rounds_, h.icm);
            icm_N_ = std::max(icm_N_, h.N);
        }
        const uint32_t tiles = (uint32_t)((h.Rcap + h.tile_rows - 1) / h.tile_rows);
        for (int64_t r = 0; r < h.Rcap; r += h.tile_rows) g.push_back(Work{ii, (uint32_t)r, 0u, tiles});
        for (int64_t r = 0; r < h.Rcap; r += kRowsPerBlock) {
            if (h.Rcap > kMapRows) rows.push_back(Work{ii, (uint32_t)r, 0u, 0u});
            post.push_back(Work{ii, (uint32_t)r, kRoleCopies, 0u});
            if (h.real) wblk.push_back(Work{ii, (uint32_t)r, 0u, 0u});
        }
        for (const Work &w : gather_items(ii, h.Rcap, h.srow_bytes)) gath.push_back(w);
        post.push_back(Work{ii, 0u, kRoleMeasure, 0u});
        int64_t fp2 = 1;
        while (fp2 < h.R) fp2 <<= 1;
        for (int64_t f = 0; f < fp2; f += 2048) post.push_back(Work{ii, (uint32_t)f, kRoleFamilies, 0u});
        for (int64_t r = 0; r < h.Rcap / 2; r += kOvlPairs) post.push_back(Work{ii, (uint32_t)r, kRoleOverlap, 0u});
        list.push_back(ii);
    }
    for (auto &kv : groups) {
        SweepGroup sg;
        sg.shape = shapes[kv.first];
        sg.icm = std::get<0>(kv.first);
        sg.nwork = (int)kv.second.size();
        sg.work = (Work *)upload(kv.second.data(), kv.second.size() * sizeof(Work));
        if (!sg.work) return dev_fail(hipErrorOutOfMemory, "upload sweep work");
        sweep_groups_.push_back(sg);
    }
    d_rows_ = nullptr;
    if (!rows.empty()) {
        d_rows_ = (Work *)upload(rows.data(), rows.size() * sizeof(Work));
        if (!d_rows_) return dev_fail(hipErrorOutOfMemory, "upload map work");
    }
    d_gather_ = (Work *)upload(gath.data(), gath.size() * sizeof(Work));
    ngather_ = (int)gath.size();
    d_post_ = (Work *)upload(post.data(), post.size() * sizeof(Work));
    d_list_ = (uint32_t *)upload(list.data(), list.size() * 4);
    d_icm_ = nullptr;
    nicm_ = (int)icm.size();
    if (nicm_) {
        d_icm_ = (Work *)upload(icm.data(), icm.size() * sizeof(Work));
        if (!d_icm_) return dev_fail(hipErrorOutOfMemory, "upload pair work");
    }
    d_wblk_ = nullptr;
    nwblk_ = (int)wblk.size();
    if (nwblk_) {
        d_wblk_ = (Work *)upload(wblk.data(), wblk.size() * sizeof(Work));
        if (!d_wblk_) return dev_fail(hipErrorOutOfMemory, "upload weight work");
    }
    if (!d_post_ || !d_list_ || !d_gather_) return dev_fail(hipErrorOutOfMemory, "upload work lists");
    const int ust = upload_sync();
    if (ust != PAMC_OK) return ust;
    nrows_work_ = (int)rows.size();
    npost_ = (int)post.size();
    nlist_ = (int)list.size();
    return PAMC_OK;
}

int Runner::init_instances(const std::vector<int> &slots)
{
    std::vector<Work> w;
    for (int i : slots)
        for (int64_t r = 0; r < inst_[i].R; r += kRowsPerBlock) w.push_back(Work{(uint32_t)i, (uint32_t)r, 0u, 0u});
    if (w.empty()) return PAMC_OK;
    Work *d = (Work *)alloc_.get(w.size() * sizeof(Work));
    if (!d) return PAMC_ERR_NOMEM;
    int st = h2d(d, w.data(), w.size() * sizeof(Work));
    if (st != PAMC_OK) return st;
    size_t lds = 0;
    for (int i : slots)
        if (inst_[i].packed) lds = std::max(lds, (size_t)std::max(16384, inst_[i].row_bytes));
    launch_init(d_insts_, d, (int)w.size(), lds, up_stream());
    launch_energy(d_insts_, d, (int)w.size(), d_Jptr_, up_stream());
    HIPCHK(hipGetLastError(), "init launch");
    st = upload_sync();
    if (st != PAMC_OK) return st;
    alloc_.put(d);
    return PAMC_OK;
}

void Runner::drop_graph()
{
    if (graph_exec_) (void)hipGraphExecDestroy(graph_exec_);
    if (graph_) (void)hipGraphDestroy(graph_);
    if (chunk_exec_) (void)hipGraphExecDestroy(chunk_exec_);
    if (chunk_graph_) (void)hipGraphDestroy(chunk_graph_);
    graph_exec_ = nullptr;
    graph_ = nullptr;
    chunk_exec_ = nullptr;
    chunk_graph_ = nullptr;
}

// The kernels of one temperature step, for every active instance.  Their
// arguments do not change from step to step (the step index and the
// population size live on the device), so the sequence can be captured once.
int Runner::launch_step_kernels()
{
    // the shape groups touch disjoint instances: with several of them, fork
    // them onto the auxiliary streams, the largest first, and join before
    // the resampling (a launch's last workgroups then share the chip with
    // the next group's first ones)
    std::vector<const SweepGroup *> plain;
    for (auto &g : sweep_groups_)
        if (!g.icm) plain.push_back(&g);
    const int ns = std::min((int)aux_.size(), (int)plain.size() - 1);
    if (ns <= 0) {
        for (const SweepGroup *g : plain)
            launch_sweep(g->shape, d_insts_, g->work, g->nwork, 0, stream_);
    } else {
        std::stable_sort(plain.begin(), plain.end(), [](const SweepGroup *a, const SweepGroup *b) {
            return (double)a->nwork * a->shape.tile_rows * a->shape.row_bytes >
                   (double)b->nwork * b->shape.tile_rows * b->shape.row_bytes;
        });
        HIPCHK(hipEventRecord(ev_fork_, stream_), "hipEventRecord (fork)");
        for (int a = 0; a < ns; ++a) HIPCHK(hipStreamWaitEvent(aux_[a], ev_fork_, 0), "hipStreamWaitEvent (fork)");
        for (size_t j = 0; j < plain.size(); ++j) {
            const int lane = (int)(j % (size_t)(ns + 1));
            const SweepGroup *g = plain[j];
            launch_sweep(g->shape, d_insts_, g->work, g->nwork, 0, lane == 0 ? stream_ : aux_[lane - 1]);
        }
        for (int a = 0; a < ns; ++a) {
            HIPCHK(hipEventRecord(ev_join_[a], aux_[a]), "hipEventRecord (join)");
            HIPCHK(hipStreamWaitEvent(stream_, ev_join_[a], 0), "hipStreamWaitEvent (join)");
        }
    }
    // runs with cluster moves split their sweeps around the ICM rounds
    if (nicm_) {
        for (auto &g : sweep_groups_)
            if (g.icm)
                launch_sweep(g.shape, d_insts_, g.work, g.nwork, 1, stream_);
        for (int rd = 0; rd < icm_rounds_; ++rd) launch_icm(d_insts_, d_icm_, nicm_, icm_N_, rd, stream_);
        for (auto &g : sweep_groups_)
            if (g.icm)
                launch_sweep(g.shape, d_insts_, g.work, g.nwork, 2, stream_);
    }
    if (timing_) HIPCHK(hipEventRecord(ev_pool_[ev_used_ - 3], stream_), "hipEventRecord");
    launch_weights(d_insts_, d_wblk_, nwblk_, stream_);
    launch_post(d_insts_, d_post_, npost_, stream_);
    launch_expand(d_insts_, d_rows_, nrows_work_, stream_);
    if (timing_) HIPCHK(hipEventRecord(ev_pool_[ev_used_ - 2], stream_), "hipEventRecord");
    if (!fuse_) {
        launch_gather(d_insts_, d_gather_, ngather_, stream_);
        launch_flip(d_insts_, d_list_, nlist_, stream_);
    }
    return PAMC_OK;
}

int Runner::enqueue_step()
{
    if (poisoned_) return PAMC_ERR_DEVICE;
    if (timing_) {
        while (ev_pool_.size() < ev_used_ + 4) {
            hipEvent_t e;
            HIPCHK(hipEventCreate(&e), "hipEventCreate");
            ev_pool_.push_back(e);
        }
        ev_used_ += 4;
        HIPCHK(hipEventRecord(ev_pool_[ev_used_ - 4], stream_), "hipEventRecord");
    }
    if (graphs_) {
        if (!graph_exec_) {
            HIPCHK(hipStreamBeginCapture(stream_, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
            launch_step_kernels();
            hipGraph_t g = nullptr;
            HIPCHK(hipStreamEndCapture(stream_, &g), "hipStreamEndCapture");
            graph_ = g;
            HIPCHK(hipGraphInstantiate(&graph_exec_, graph_, nullptr, nullptr, 0), "hipGraphInstantiate");
        }
        HIPCHK(hipGraphLaunch(graph_exec_, stream_), "hipGraphLaunch");
    } else {
        int st = launch_step_kernels();
        if (st != PAMC_OK) return st;
    }
    if (timing_) HIPCHK(hipEventRecord(ev_pool_[ev_used_ - 1], stream_), "hipEventRecord");
    HIPCHK(hipGetLastError(), "step launch");
    count_enqueued(1);
    return PAMC_OK;
}

void Runner::count_enqueued(int steps)
{
    for (int i : active_) {
        HostInst &h = inst_[i];
        h.k_enq = std::min(h.nT, h.k_enq + steps);
    }
}

// kChunkSteps steps as one graph launch (the step kernels read the step
// index from the device, so consecutive steps are the same kernel
// sequence; steps past an instance's last temperature do nothing).
int Runner::enqueue_chunk()
{
    if (poisoned_) return PAMC_ERR_DEVICE;
    if (!chunk_exec_) {
        HIPCHK(hipStreamBeginCapture(stream_, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
        for (int s = 0; s < kChunkSteps; ++s) launch_step_kernels();
        hipGraph_t g = nullptr;
        HIPCHK(hipStreamEndCapture(stream_, &g), "hipStreamEndCapture");
        chunk_graph_ = g;
        HIPCHK(hipGraphInstantiate(&chunk_exec_, chunk_graph_, nullptr, nullptr, 0), "hipGraphInstantiate");
    }
    HIPCHK(hipGraphLaunch(chunk_exec_, stream_), "hipGraphLaunch");
    HIPCHK(hipGetLastError(), "chunk launch");
    count_enqueued(kChunkSteps);
    return PAMC_OK;
}

int Runner::phase_times(double *sweep_ms, double *resample_ms, double *gather_ms, int64_t *n_steps)
{
    if (!timing_) {
        set_error("timing is off for this run");
        return PAMC_ERR_STATE;
    }
    HIPCHK(hipStreamSynchronize(stream_), "timing sync");
    double t[3] = {0.0, 0.0, 0.0};
    for (size_t j = 0; j + 4 <= ev_used_; j += 4)
        for (int p = 0; p < 3; ++p) {
            float ms = 0.f;
            HIPCHK(hipEventElapsedTime(&ms, ev_pool_[j + p], ev_pool_[j + p + 1]), "hipEventElapsedTime");
            t[p] += ms;
        }
    if (sweep_ms) *sweep_ms = t[0];
    if (resample_ms) *resample_ms = t[1];
    if (gather_ms) *gather_ms = t[2];
    if (n_steps) *n_steps = (int64_t)(ev_used_ / 4);
    ev_used_ = 0;
    return PAMC_OK;
}

int Runner::enqueue_steps(int n)
{
    // steps left for the active instance that is furthest from its end
    int left = 0;
    for (int i : active_) left = std::max(left, inst_[i].nT - inst_[i].k_enq);
    n = std::min(n, left);
    while (n > 0) {
        int st;
        if (graphs_ && n >= kChunkSteps) {
            st = enqueue_chunk();
            n -= kChunkSteps;
        } else {
            st = enqueue_step();
            --n;
        }
        if (st != PAMC_OK) return st;
    }
    return PAMC_OK;
}

int Runner::sync()
{
    if (poisoned_) return PAMC_ERR_DEVICE;
    HIPCHK(hipStreamSynchronize(stream_), "hipStreamSynchronize");
    return PAMC_OK;
}

int Runner::read_ctl(int i, int32_t ctl[3], uint32_t status[2])
{
    const HostInst &h = inst_[i];
    // in serving mode the instance's steps have completed: read on the
    // upload path, without waiting for the steps queued behind them
    const hipStream_t s = async_ ? side_ : stream_;
    HIPCHK(hipMemcpyAsync(ctl, h.ctl, 12, hipMemcpyDeviceToHost, s), "read ctl");
    HIPCHK(hipMemcpyAsync(status, h.dev.status, 8, hipMemcpyDeviceToHost, s), "read status");
    HIPCHK(hipStreamSynchronize(s), "read ctl sync");
    return PAMC_OK;
}

int Runner::inst_status(int i, int *step, int64_t *Rk)
{
    int32_t ctl[3];
    uint32_t status[2];
    int st = read_ctl(i, ctl, status);
    if (st != PAMC_OK) return st;
    const HostInst &h = inst_[i];
    uint32_t r = 0;
    const int k = ctl[0];
    // after the last step the population is that of step nT - 1
    st = d2h(&r, h.dev.Rk + std::min(k, h.nT - 1), 4);
    if (st != PAMC_OK) return st;
    if (step) *step = k;
    if (Rk) *Rk = r;
    if (status[0] & 1u) {
        set_error("resampling at step " + std::to_string(status[1]) + " exceeded the capacity");
        return PAMC_ERR_CAPACITY;
    }
    if (status[0] & 2u) {
        set_error("resampling at step " + std::to_string(status[1]) + " left no replica");
        return PAMC_ERR_EXTINCT;
    }
    return PAMC_OK;
}

int Runner::observables(int i, pamc_step_obs *out, int n)
{
    const HostInst &h = inst_[i];
    if (n < 0 || n > h.nT) {
        set_error("observables: n out of range");
        return PAMC_ERR_INVALID;
    }
    int32_t ctl[3];
    uint32_t status[2];
    int st = read_ctl(i, ctl, status);
    if (st != PAMC_OK) return st;
    std::vector<StepRec> rec((size_t)h.nT);
    std::vector<uint32_t> q((size_t)std::max(1, h.ovl_n) * (2 * h.N + 1));
    st = d2h(rec.data(), h.dev.rec, rec.size() * sizeof(StepRec));
    if (st == PAMC_OK) st = d2h(q.data(), h.dev.qhist, q.size() * 4);
    if (st != PAMC_OK) return st;
    // steps measured: those below the device step, plus the failing step
    int kdone = ctl[0];
    if (status[0]) kdone = (int)status[1] + 1;
    const double nan = std::numeric_limits<double>::quiet_NaN();
    const int N = h.N;
    double lnZ = h.lnZ_base;
    for (int k = 0; k < n; ++k) {
        pamc_step_obs &o = out[k];
        std::memset(&o, 0, sizeof(o));
        o.beta = h.beta[k];
        o.mean_E = o.e = o.C_V = o.lnQ = o.lnZ = o.betaF = o.f = o.S_f = o.rho_s = nan;
        o.q_abs = o.q2 = o.q4 = o.g_SG = nan;
        if (k < h.k_base || k >= kdone) continue;
        const StepRec &r = rec[k];
        o.measured = 1;
        o.R = r.R;
        o.sum_E = r.sumE;
        o.sum_E2 = (int64_t)r.sumE2;
        o.sum_E2_hi = r.sumE2_hi;
        o.E_min = r.Emin;
        o.E_max = r.Emax;
        const double Rd = (double)r.R;
        // energies in units of 2^-20 for real couplings (exact scalings)
        const double sc = h.real ? 0x1p-20 : 1.0;
        o.mean_E = ((double)r.sumE * sc) / Rd;
        o.e = o.mean_E / (double)N;
        const __int128 sum2 = (__int128)(((unsigned __int128)(uint64_t)r.sumE2_hi << 64) | r.sumE2);
        const __int128 num = (__int128)r.R * sum2 - (__int128)r.sumE * (__int128)r.sumE;
        const double var = ((double)num / (Rd * Rd)) * (sc * sc);
        o.C_V = (o.beta * o.beta) * var / (double)N;
        o.lnZ = lnZ;
        o.betaF = -lnZ;
        o.f = o.beta > 0.0 ? -lnZ / (o.beta * (double)N) : nan;
        o.S_f = std::log(Rd) - r.T / Rd;
        o.rho_s = Rd / std::exp(o.S_f);
        if (k < h.nT - 1 && k + 1 < kdone + (status[0] ? 0 : 1)) {
            const double db = h.beta[k + 1] - h.beta[k];
            o.lnQ = (-db * ((double)r.Emin * sc)) + std::log(r.S) - std::log(Rd);
            lnZ = lnZ + o.lnQ;
        }
        const int slot = h.ovl_slot[k];
        if (slot >= 0) {
            const uint32_t *hq = q.data() + (size_t)slot * (2 * N + 1);
            int64_t cnt = 0;
            double m1 = 0.0, m2 = 0.0, m4 = 0.0;
            for (int Q = -N; Q <= N; ++Q) {
                const int64_t c = hq[Q + N];
                if (c == 0) continue;
                const double qq = (double)Q / (double)N;
                cnt += c;
                m1 += (double)c * std::fabs(qq);
                m2 += (double)c * (qq * qq);
                m4 += (double)c * ((qq * qq) * (qq * qq));
            }
            if (cnt > 0) {
                o.q_abs = m1 / (double)cnt;
                o.q2 = m2 / (double)cnt;
                o.q4 = m4 / (double)cnt;
                o.g_SG = 0.5 * (3.0 - o.q4 / (o.q2 * o.q2));
            }
        }
    }
    return PAMC_OK;
}

int Runner::overlap_hist(int i, int step, int64_t *hist)
{
    const HostInst &h = inst_[i];
    if (step < 0 || step >= h.nT || h.ovl_slot[step] < 0) {
        set_error("not an overlap step");
        return PAMC_ERR_STATE;
    }
    int32_t ctl[3];
    uint32_t status[2];
    int st = read_ctl(i, ctl, status);
    if (st != PAMC_OK) return st;
    if (step >= ctl[0]) {
        set_error("overlap step has not run");
        return PAMC_ERR_STATE;
    }
    std::vector<uint32_t> q((size_t)(2 * h.N + 1));
    HIPCHK(hipMemcpy(q.data(), h.dev.qhist + (size_t)h.ovl_slot[step] * (2 * h.N + 1), q.size() * 4,
                     hipMemcpyDeviceToHost),
           "read qhist");
    for (size_t j = 0; j < q.size(); ++j) hist[j] = q[j];
    return PAMC_OK;
}

int Runner::step_sums(int i, double *S, double *T, int n)
{
    const HostInst &h = inst_[i];
    if (n < 0 || n > h.nT) return PAMC_ERR_INVALID;
    std::vector<StepRec> rec((size_t)h.nT);
    HIPCHK(hipStreamSynchronize(stream_), "sync");
    HIPCHK(hipMemcpy(rec.data(), h.dev.rec, rec.size() * sizeof(StepRec), hipMemcpyDeviceToHost), "read rec");
    for (int k = 0; k < n; ++k) {
        if (S) S[k] = rec[k].S;
        if (T) T[k] = rec[k].T;
    }
    return PAMC_OK;
}

// Bring a pending copy map into the other buffer so that rows are stored
// in order (used before export).
int Runner::materialise(int i)
{
    HostInst &h = inst_[i];
    int32_t ctl[3];
    uint32_t status[2];
    int st = read_ctl(i, ctl, status);
    if (st != PAMC_OK) return st;
    if (!ctl[2]) return PAMC_OK;
    const std::vector<Work> rows = gather_items((uint32_t)i, h.Rcap, h.srow_bytes);
    Work *d = (Work *)alloc_.get(rows.size() * sizeof(Work));
    uint32_t *l = (uint32_t *)alloc_.get(4);
    if (!d || !l) {
        alloc_.put(d);
        alloc_.put(l);
        return PAMC_ERR_NOMEM;
    }
    const uint32_t idx = (uint32_t)i;
    HIPCHK(hipMemcpy(d, rows.data(), rows.size() * sizeof(Work), hipMemcpyHostToDevice), "upload rows");
    HIPCHK(hipMemcpy(l, &idx, 4, hipMemcpyHostToDevice), "upload list");
    launch_gather(d_insts_, d, (int)rows.size(), stream_);
    launch_flip(d_insts_, l, 1, stream_);
    HIPCHK(hipGetLastError(), "gather launch");
    HIPCHK(hipStreamSynchronize(stream_), "gather sync");
    alloc_.put(d);
    alloc_.put(l);
    return PAMC_OK;
}

// Where rows of +-1 bytes pass between the caller and population buffer b
// (idle): the buffer itself, or memory for one row where it does not hold one
// (a few packed rows).
Runner::StateStage Runner::state_stage(const HostInst &h, int b)
{
    StateStage s{(int8_t *)h.dev.spins[b], nullptr, h.Rcap * h.srow_bytes / h.N};
    if (s.rows == 0) {
        s.own = alloc_.get((size_t)h.N);
        s.p = (int8_t *)s.own;
        s.rows = 1;
        if (!s.p) set_error("state staging allocation failed");
    }
    return s;
}

int Runner::get_state(int i, pamc_state *stt)
{
    HostInst &h = inst_[i];
    int st = sync();
    if (st != PAMC_OK) return st;
    st = materialise(i);
    if (st != PAMC_OK) return st;
    int32_t ctl[3];
    uint32_t status[2];
    st = read_ctl(i, ctl, status);
    if (st != PAMC_OK) return st;
    uint32_t Rk = 0;
    HIPCHK(hipMemcpy(&Rk, h.dev.Rk + std::min(ctl[0], h.nT - 1), 4, hipMemcpyDeviceToHost), "read Rk");
    if (status[0]) {
        // the failing step's population after its sweeps
        HIPCHK(hipMemcpy(&Rk, h.dev.Rk + status[1], 4, hipMemcpyDeviceToHost), "read Rk");
    }
    stt->step = ctl[0];
    stt->R = Rk;
    // ln Z at the current step
    {
        std::vector<pamc_step_obs> obs((size_t)h.nT);
        st = observables(i, obs.data(), h.nT);
        if (st != PAMC_OK) return st;
        double lnZ = h.lnZ_base;
        for (int k = h.k_base; k < ctl[0] && k < h.nT; ++k)
            if (!std::isnan(obs[k].lnQ)) lnZ = lnZ + obs[k].lnQ;
        stt->lnZ = lnZ;
    }
    const int cur = ctl[1];
    if (stt->spins) {
        // through the idle buffer, as many rows at a time as it holds
        const StateStage stage = state_stage(h, cur ^ 1);
        if (!stage.p) return PAMC_ERR_NOMEM;
        for (int64_t r = 0; st == PAMC_OK && r < (int64_t)Rk; r += stage.rows) {
            const int n = (int)std::min<int64_t>(stage.rows, (int64_t)Rk - r);
            launch_export(d_insts_ + i, h.N, stage.p, (int)r, n, stream_);
            hipError_t e = hipGetLastError();
            if (e == hipSuccess)
                e = hipMemcpyAsync(stt->spins + (size_t)r * h.N, stage.p, (size_t)n * h.N, hipMemcpyDeviceToHost, stream_);
            if (e == hipSuccess) e = hipStreamSynchronize(stream_);
            if (e != hipSuccess) st = dev_fail(e, "read spins");
        }
        alloc_.put(stage.own);
        if (st != PAMC_OK) return st;
    }
    if (h.real) {
        if (stt->E_fixed)
            HIPCHK(hipMemcpy(stt->E_fixed, h.dev.Eq[cur], (size_t)Rk * 8, hipMemcpyDeviceToHost), "read E");
    } else if (stt->E) {
        HIPCHK(hipMemcpy(stt->E, h.dev.E[cur], (size_t)Rk * 4, hipMemcpyDeviceToHost), "read E");
    }
    if (stt->family)
        HIPCHK(hipMemcpy(stt->family, h.dev.fam[cur], (size_t)Rk * 4, hipMemcpyDeviceToHost), "read family");
    return PAMC_OK;
}

int Runner::set_state(int i, const pamc_state *st)
{
    HostInst &h = inst_[i];
    if (!st || !st->spins || !st->family || st->step < 0 || st->step >= h.nT || st->R < 1 || st->R > h.Rcap) {
        set_error("set_state: invalid state");
        return PAMC_ERR_INVALID;
    }
    const int64_t R = st->R;
    for (int64_t r = 0; r < R; ++r) {
        const int8_t *in = st->spins + (size_t)r * h.N;
        uint32_t bad = 0;
        for (int s = 0; s < h.N; ++s) bad |= (uint32_t)(uint8_t)(in[s] + 1) & 0xFDu;
        if (bad) {
            set_error("set_state: spins must be +-1");
            return PAMC_ERR_INVALID;
        }
        if ((int64_t)st->family[r] >= h.R) {
            set_error("set_state: family id out of range");
            return PAMC_ERR_INVALID;
        }
    }
    int stt = sync();
    if (stt != PAMC_OK) return stt;
    const int32_t ctl[3] = {st->step, 0, 0};
    const uint32_t status[2] = {0, 0};
    const uint32_t Rk = (uint32_t)R;
    const StateStage stage = state_stage(h, 1);
    if (!stage.p) return PAMC_ERR_NOMEM;
    for (int64_t r = 0; stt == PAMC_OK && r < R; r += stage.rows) {
        const int n = (int)std::min<int64_t>(stage.rows, R - r);
        hipError_t e = hipMemcpyAsync(stage.p, st->spins + (size_t)r * h.N, (size_t)n * h.N, hipMemcpyHostToDevice, stream_);
        if (e == hipSuccess) {
            launch_import(d_insts_ + i, h.srow_bytes, stage.p, (int)r, n, stream_);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(stream_);
        if (e != hipSuccess) stt = dev_fail(e, "write spins");
    }
    alloc_.put(stage.own);
    if (stt != PAMC_OK) return stt;
    HIPCHK(hipMemcpy(h.dev.fam[0], st->family, (size_t)R * 4, hipMemcpyHostToDevice), "write family");
    HIPCHK(hipMemcpy(h.ctl, ctl, 12, hipMemcpyHostToDevice), "write ctl");
    HIPCHK(hipMemcpy(h.dev.status, status, 8, hipMemcpyHostToDevice), "write status");
    HIPCHK(hipMemcpy(h.dev.Rk + st->step, &Rk, 4, hipMemcpyHostToDevice), "write Rk");
    // parts of the energy histogram or minimum, which a step that failed in
    // its resampling or the last step left behind
    if (h.real) {
        const std::vector<long long> emin(kMinParts, kNoEnergy);
        HIPCHK(hipMemcpy(h.dev.emin, emin.data(), emin.size() * 8, hipMemcpyHostToDevice), "clear the lowest energies");
    } else {
        HIPCHK(hipMemset(h.dev.hist, 0, (size_t)h.dev.nlev * 4), "clear the histogram");
        HIPCHK(hipMemset(h.dev.loff, 0, (size_t)h.Rcap * 4), "clear the histogram");
    }
    // overlaps of the steps that run again are counted anew (slots follow the
    // order in which the steps were asked for)
    const size_t bins = 2 * (size_t)h.N + 1;
    for (int k = st->step; k < h.nT; ++k)
        if (h.ovl_slot[k] >= 0)
            HIPCHK(hipMemset(h.dev.qhist + (size_t)h.ovl_slot[k] * bins, 0, bins * 4), "clear the overlaps");
    // energies from the spins (Eq. (1)) for the imported rows
    std::vector<Work> rows;
    for (int64_t r = 0; r < R; r += kRowsPerBlock) rows.push_back(Work{(uint32_t)i, (uint32_t)r, 0u, 0u});
    Work *d = (Work *)alloc_.get(rows.size() * sizeof(Work));
    if (!d) return PAMC_ERR_NOMEM;
    HIPCHK(hipMemcpy(d, rows.data(), rows.size() * sizeof(Work), hipMemcpyHostToDevice), "upload rows");
    launch_energy(d_insts_, d, (int)rows.size(), d_Jptr_, stream_);
    HIPCHK(hipGetLastError(), "energy launch");
    HIPCHK(hipStreamSynchronize(stream_), "energy sync");
    alloc_.put(d);
    h.k_enq = st->step;
    h.k_base = st->step;
    h.lnZ_base = st->lnZ;
    return PAMC_OK;
}

int Runner::thresholds(int i, uint32_t *out, uint8_t *acc)
{
    const HostInst &h = inst_[i];
    if (h.real) {
        set_error("thresholds: runs with real couplings take their acceptance per move (no table)");
        return PAMC_ERR_STATE;
    }
    std::vector<uint32_t> thr((size_t)h.nT * 4);
    HIPCHK(hipMemcpy(thr.data(), h.dev.thr, thr.size() * 4, hipMemcpyDeviceToHost), "read thr");
    for (int k = 0; k < h.nT; ++k) {
        if (out)
            for (int j = 0; j < 3; ++j) out[3 * k + j] = thr[4 * k + j];
        if (acc) acc[k] = (uint8_t)thr[4 * k + 3];
    }
    return PAMC_OK;
}

}  // namespace pamc
