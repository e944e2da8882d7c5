// tune.cpp -- sweep workgroup shapes chosen by measurement.
//
// How fast the sweep runs depends on how many replicas share a word and how
// many sets of them a workgroup holds: a small population needs few to spread
// over the 256 compute units, a large one shares each block's fields and
// tables among many.  The
// tuner runs each candidate shape on a throw-away run of the instance (its
// couplings, L, R, capacity and sweeps per step) at a constant beta = 2
// after the beta = 0 start, where every replica gets one copy on average
// and the population stays near R, and keeps the shape whose fastest timed
// step (HIP events, after a warm-up step) is shortest; a burn-in first
// brings the energies to that temperature.
// Every shape gives bit-identical results, so the choice only affects
// speed.  Choices are cached for the life of the process, keyed by device
// (architecture and compute units), kernel, lattice (dimension and L),
// sweeps per step, the capacity rounded up to a power of two and the spin
// storage format; the cache starts from the file tune_cache.jsonl beside
// the library and from the file PAMC_TUNE_CACHE names, and new choices are
// appended to the latter, so a later process finds them.
#include <dlfcn.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <tuple>
#include <vector>

#include "runner.h"

namespace pamc {

int make_inst(int L, const int8_t *J, const int32_t *Jq, int64_t R, const double *beta, int nT, int NS,
              uint64_t seed, const pamc_options &opt, HostInst &h);

namespace {

constexpr int64_t kMaxLds = kMaxSweepLds;  // dynamic LDS of one sweep workgroup
constexpr int kTimedSteps = 3;      // timed steps per candidate shape (after one warm-up)
constexpr int kBurnIn = 8;          // steps before the first candidate
constexpr double kTuneBeta = 2.0;   // inside the low-temperature part where an anneal spends most steps

constexpr int kMaxWord = kSiteWord;  // replicas per word (more: words of sites, see sw_form)

bool is_rb(const HostInst &h) { return h.variant == kSweepRB; }

// The word kernels' launch: threads and LDS of a workgroup of `sets` sets, the
// waves a compute unit holds (80 to 188 registers a lane).
int words_threads(const HostInst &h, int m, int sets)
{
    return m > kMaxWord ? sw_threads(h.gmax, sets) : is_rb(h) ? rb_threads(h.gmax, sets) : rq_threads(h.gmax, sets);
}
int64_t words_lds(const HostInst &h, int m, int sets)
{
    const int plane = rb_plane(h.row_bytes);
    if (!is_rb(h)) return rq_lds(h.variant, plane, m, sets);
    if (m > kMaxWord) return (int64_t)sw_lds(h.row_bytes, m, sets);
    return (int64_t)(rs_small(h.gmax, m, sets) ? rs_lds(plane, h.gmax, sets) : rb_lds(plane, sets));
}
int64_t words_max_lds(const HostInst &h) { return is_rb(h) ? kMaxLds : kMaxWordLds; }
int words_cu_waves(const HostInst &h, int m, bool small)
{
    return !is_rb(h) ? 16 : m > kMaxWord ? 28 : !small ? 24 : h.ncol == 2 ? 12 : 8;
}

// Rows of a pass.
int words_rows(int m, int sets) { return (m > kMaxWord ? m - kMaxWord : m) * sets; }
// A shape of words: m replicas per word, `sets` sets per pass, tile_rows rows
// per workgroup.  rp, reported as group_replicas = 4 rp, is 0 where the caller
// cannot choose it.
bool fixed_group(const HostInst &h) { return is_rb(h) && (h.L == 8 || h.L == 16 || h.L > 21 || (h.L > 20 && h.L % 2 == 0)); }
void set_rb(HostInst &h, int m, int sets, int tile_rows)
{
    h.mrep = m;
    h.sets = sets;
    h.tile_rows = tile_rows;
    h.rp = fixed_group(h) ? 0 : (words_rows(m, sets) + 3) / 4;
}

struct Choice {
    int tile_rows, rp, mrep, sets;
    double ns_per_attempt;
};

using Key = std::tuple<int, int, int, int, int, int>;  // variant, dim, L, sweeps, log2 capacity, packed

// The variant a choice of words is stored under tells the replicas per word
// (kSweepRB + m; the variants are 64 apart); its workgroups sweep tile_rows =
// words_rows(m, sets) rows in one pass.

std::mutex g_mu;
std::map<std::pair<std::string, Key>, Choice> g_cache;  // by device and key
bool g_loaded = false;
std::string g_save_path;  // where new choices are appended ("" = nowhere)

// The device a choice was measured on: architecture and compute units.
std::string device_tag()
{
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess) return "unknown";
    std::string arch = p.gcnArchName;
    const size_t c = arch.find(':');
    if (c != std::string::npos) arch.resize(c);
    return arch + "-" + std::to_string(p.multiProcessorCount) + "cu";
}

// One choice per line, as a JSON object with these fields in this order
// (read with kLineFmt, written with kLineOut).
#define PAMC_TUNE_LINE(DEV, NS)                                                                     \
    "{\"device\": \"" DEV "\", \"variant\": %d, \"dim\": %d, \"L\": %d, \"sweeps\": %d, "  \
    "\"cap_log2\": %d, \"packed\": %d, \"tile_rows\": %d, \"group_quads\": %d, "               \
    "\"ns_per_attempt\": " NS "}"
const char *kLineFmt = PAMC_TUNE_LINE("%63[^\"]", "%lf");
const char *kLineOut = PAMC_TUNE_LINE("%s", "%.6e");
#undef PAMC_TUNE_LINE

void load_file(const std::string &path)
{
    FILE *f = std::fopen(path.c_str(), "r");
    if (!f) return;
    char line[512];
    while (std::fgets(line, sizeof line, f)) {
        char dev[64];
        int v, d, L, ns, cl, pk, tr, rp;
        double npa;
        if (std::sscanf(line, kLineFmt, dev, &v, &d, &L, &ns, &cl, &pk, &tr, &rp, &npa) != 10) continue;
        Choice c{tr, rp, 0, 0, npa};
        if (v >= kSweepRB) {
            c.mrep = v % 64;
            if (c.mrep < 1) continue;
            c.sets = tr / words_rows(c.mrep, 1);
            v -= c.mrep;
        }
        g_cache[{dev, Key(v, d, L, ns, cl, pk)}] = c;
    }
    std::fclose(f);
}

// The tuning cache file shipped beside the library (choices measured on
// MI355X for common sizes), then PAMC_TUNE_CACHE when it names a file;
// new choices are appended to PAMC_TUNE_CACHE.  Call with g_mu held.
void load_persistent()
{
    if (g_loaded) return;
    g_loaded = true;
    Dl_info info;
    if (dladdr((void *)&load_persistent, &info) && info.dli_fname) {
        std::string dir = info.dli_fname;
        const size_t sl = dir.rfind('/');
        dir = sl == std::string::npos ? std::string(".") : dir.substr(0, sl);
        load_file(dir + "/tune_cache.jsonl");
    }
    const char *env = std::getenv("PAMC_TUNE_CACHE");
    if (env && *env) {
        g_save_path = env;
        load_file(g_save_path);
    }
}

void save_choice(const std::string &dev, const Key &k, const Choice &c)
{
    if (g_save_path.empty()) return;
    FILE *f = std::fopen(g_save_path.c_str(), "a");
    if (!f) return;
    std::fprintf(f, kLineOut, dev.c_str(), std::get<0>(k) + c.mrep, std::get<1>(k), std::get<2>(k), std::get<3>(k),
                 std::get<4>(k), std::get<5>(k), c.tile_rows, c.rp, c.ns_per_attempt);
    std::fputc('\n', f);
    std::fclose(f);
}

int ceil_log2(int64_t v)
{
    int b = 0;
    while (((int64_t)1 << b) < v) ++b;
    return b;
}

}  // namespace

// Whether the sweep kernel of the instance can run its shape; on failure
// *why says what is wrong.
bool shape_valid(const HostInst &h, const char **why)
{
    const char *w = nullptr;
    if (h.tile_rows < 1 || h.tile_rows > 4096) {
        w = "tile_rows must be in [1, 4096]";
    } else {
        if (h.mrep < 1 || (h.mrep > kMaxWord && !(is_rb(h) && sw_form(h.L, h.mrep))) || h.sets < 1 ||
            words_threads(h, h.mrep, h.sets) > 1024 || (is_rb(h) && h.sets > 1 && h.gmax * h.sets > 1024))
            w = "no such grouping of replicas";
        else if (words_lds(h, h.mrep, h.sets) > words_max_lds(h))
            w = "the workgroup's tile does not fit in LDS";
    }
    if (why) *why = w;
    return w == nullptr;
}

// Quads of a workgroup whose caller asks for none: 256 / tpr of at most 64
// threads; above, the number of quads (of at most 512 threads together) that
// leaves the fewest idle lanes in the last wave, the one nearest 256 threads
// among equals.
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

// Sets of a workgroup of about `threads` threads: with +-1 couplings one where
// a set fills whole waves; else the count up to that size (at least one) with
// the fewest idle lanes.
static int words_sets(const HostInst &h, int threads)
{
    int best = 1;
    double best_use = 0.0;
    if (is_rb(h) && rb_uniform(h.gmax)) return 1;
    for (int s = 1; words_threads(h, 1, s) <= std::min(1024, std::max(threads, words_threads(h, 1, 1))); ++s) {
        if (words_lds(h, kMaxWord, s) > words_max_lds(h)) break;
        const double use = (double)h.gmax * s / words_threads(h, 1, s);
        if (use >= best_use - 0.005) {
            best = s;
            best_use = std::max(use, best_use);
        }
    }
    return best;
}

// Workgroups of nt threads and lds bytes a compute unit holds at once.  (At two
// or three waves a SIMD, a workgroup whose waves do not divide among the four
// SIMDs leaves room that the next one cannot take.)
constexpr int kCU = 256;
static int words_per_cu(const HostInst &h, int m, int nt, int64_t lds, bool small)
{
    const int waves = nt / 64, most = words_cu_waves(h, m, small);
    const int n = small && waves > 4 ? most / 4 / ((waves + 3) / 4) : most / waves;
    return std::max<int>(1, (int)std::min<int64_t>(n, 160 * 1024 / (lds + 512)));
}

// Replicas per word worth considering (+-1 couplings: the table mode draws for
// four at a time).
static bool words_worth(const HostInst &h, int m)
{
    return m > kMaxWord ? is_rb(h) && sw_form(h.L, m) : !is_rb(h) || m <= 2 || m % 4 == 0;
}

// Predicted time (cycles of a SIMD a colour step) of a launch over populations
// of these rows in workgroups of tile_rows rows, m replicas per word and `sets`
// words side by side: what a colour step of a lane issues, about a instructions
// for its fields and b per draw of four sites, at 4.45 cycles an instruction
// for each of the waves that share a SIMD (6 or 8 for one, 9.3 for two; the
// small words of sweep_rs.hip 6.3, 8.2 and 3.6 each).  Large words save fields,
// small ones fill the chip and its last round of workgroups.  The figures are
// measured; over 36 sizes with +-1 couplings from L = 4, R = 10^3 to L = 16,
// R = 5 10^4 and L = 32, R = 50 the shape chosen is within 10% of the best of
// all that can be tried.
// Launches beside others (a batch of several lattices) also count the issue
// time they take of the chip, at 0.3 of it: nine instances of L = 4 ... 11 with
// 3528 rows each ran 59 ms with every launch the shortest by itself, 51 so, 59
// with all of it; real couplings gain nothing from it.
static double shape_time(const HostInst &h, int m, int sets, int tile_rows, const std::vector<int64_t> &rows, int beside)
{
    const int nt = words_threads(h, m, sets), blocks = std::max(1, (h.gmax + nt - 1) / nt), pass = words_rows(m, sets);
    const bool site = m > kMaxWord, small = is_rb(h) && !site && rs_small(h.gmax, m, sets);
    const int per_cu = words_per_cu(h, m, nt, words_lds(h, m, sets), small);
    // instructions of a lane's colour step: fields, and draws and decisions of
    // four sites; tables, once a launch
    double a = site ? 36.0 : small ? 155.0 : 190.0, b = site ? 45.0 : small ? 90.0 : 42.0, once = 0.0;
    if (!is_rb(h)) {
        const int kind = rq_kind(h.variant, m * sets);
        if (kind == kRQBonds) {
            a = 180.0;
            b = 130.0;
        } else {
            a = m <= 4 ? 120.0 : 320.0;
            b = (kind == kRQThr ? 62.0 : 105.0) + (m <= 4 ? 48.0 : 0.0);
        }
        once = (double)h.N / nt * (kind == kRQThr ? h.dim == 3 ? 1400.0 : 400.0 : 150.0) / (h.NS * h.ncol);
    }
    const int64_t round = (int64_t)kCU * per_cu;
    int64_t wgs = 0, most = 0;
    for (int64_t r : rows) {
        wgs += (r + tile_rows - 1) / tile_rows;
        most = std::max(most, r);
    }
    // cycles per instruction of a lane's colour step with n workgroups on the
    // chip, from the waves that share a SIMD
    auto cycles = [&](int64_t n) {
        const int64_t w = ((n + kCU - 1) / kCU * (nt / 64) + 3) / 4;
        if (site) return w == 0 ? 0.0 : w == 1 ? 6.3 : 4.3 * (double)w + 1.0;
        if (small) return w == 0 ? 0.0 : w == 1 ? 6.3 : w == 2 ? 8.2 : 3.6 * (double)w;
        return w == 0 ? 0.0 : w == 1 ? (is_rb(h) ? 8.0 : 6.0) : w == 2 ? 9.3 : 4.45 * (double)w;
    };
    // (a further pass loads and stores rows of its own, about 6 us; tables of
    // thresholds are made anew)
    const int passes = std::max<int>(1, (int)((std::min<int64_t>(tile_rows, most) + pass - 1) / pass));
    const double step = (a + b * words_rows(m, 1)) * blocks + once;
    double t = step * ((double)(wgs / round) * cycles(round) + cycles(wgs % round));
    // many waves in step with each other, words of few replicas: L = 5, 128 rows
    // as two a word in 11 waves take 80 us (46 by the above), as four bytes a
    // word in 6 waves 60 (53); L = 3, R = 10^5, two a word in 12 waves 110
    if (is_rb(h) && !small && !site && sets > 1 && nt > 256) t *= 1.0 + std::max(0.0, 1.5 / m - 0.1);
    if (is_rb(h) && beside > 1)
        t = t / beside + 0.3 * step * 4.45 * (double)(wgs * (nt / 64)) / (4.0 * kCU);
    return t * passes + (passes - 1) * 14400.0 / (h.NS * h.ncol);
}

// Sets of words of sites side by side: one, or where a set is a wave four (a
// workgroup's rows and tables in fewer, larger transfers; L = 8, R = 20000:
// 63 us with one replica a lane in four sets, 60 with two).
static int site_sets(const HostInst &h, bool many) { return many && h.gmax == 64 ? 4 : 1; }

// The shape used without tuning: that of the shortest launch, one pass a
// workgroup.
// Words of sites take populations up to 2 10^7 spins, 10^7 where three launches
// run side by side (they issue more for an attempt; batches of L = 4 ... 8 in
// words of replicas and of sites: 12 x 9023 rows 42.5 and 40.7 ms, 15 x 12911
// rows 13.1 and 13.5), with two replicas a lane where one would give each SIMD
// more than four waves.  Launches of 10 sweeps, words of sites against the best
// of replicas: L = 8, R = 1000: 13 and 24 us; 10^4: 35 and 56; 2 10^4: 60 and
// 78; 5 10^4: 134 and 133; 10^5: 243 and 214; L = 16, R = 300: 21 and 33; 1000:
// 32 and 54; 3000: 74 and 89; 6000: 133 and 129.
void default_shape(HostInst &h, const std::vector<int64_t> &rows, int beside)
{
    const int64_t most = *std::max_element(rows.begin(), rows.end());
    const int64_t total = std::accumulate(rows.begin(), rows.end(), (int64_t)0);
    if (words_worth(h, kSiteWord + 1) && total * h.N * (beside + 1) <= 40'000'000) {
        const bool many = total * (h.gmax / 64) > 16 * kCU;
        const int m = kSiteWord + (many ? 2 : 1), sets = site_sets(h, many);
        set_rb(h, m, sets, words_rows(m, sets));
        return;
    }
    double best = INFINITY;
    int last = 0;
    for (int threads : {64, 256, 512, 1024}) {
        if (is_rb(h) && threads == 512) continue;
        const int sets = words_sets(h, threads);
        if (sets == last) continue;
        last = sets;
        for (int m = 1; m <= kMaxWord; ++m) {
            if (m > 4 && m * sets > most) break;
            if (!words_worth(h, m)) continue;
            const double t = shape_time(h, m, sets, m * sets, rows, beside);
            if (t < 0.98 * best) {
                best = t;
                set_rb(h, m, sets, m * sets);
            }
        }
    }
}

// What the sweep kernels need to know of the instance to weigh a shape.
static HostInst shape_of(const HostInst &h)
{
    HostInst t;
    t.dim = h.dim;
    t.L = h.L;
    t.N = h.N;
    t.ncol = h.ncol;
    t.NS = h.NS;
    t.variant = h.variant;
    t.gmax = h.gmax;
    t.row_bytes = h.row_bytes;
    t.real = h.real;
    t.tpr = h.tpr;
    return t;
}

static Key cache_key(const HostInst &h) { return Key(h.variant, h.dim, h.L, h.NS, ceil_log2(h.Rcap), h.packed); }

// The choice measured before for this key, as far as the kernel can run it.
static bool cached_shape(const std::pair<std::string, Key> &key, HostInst &t, double *ns_per_attempt)
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_persistent();
    const auto it = g_cache.find(key);
    if (it == g_cache.end()) return false;
    const Choice &c = it->second;
    t.tile_rows = c.tile_rows;
    t.rp = c.rp;
    t.mrep = c.mrep;
    t.sets = c.sets;
    if (!shape_valid(t, nullptr)) return false;
    if (ns_per_attempt) *ns_per_attempt = c.ns_per_attempt;
    return true;
}

// Whether the library reports this tile and group for a shape of its own
// choice (the rule's or the tuner's: one pass a workgroup).
bool reported_shape(const HostInst &h, int tile_rows, int group_replicas)
{
    if (group_replicas != (fixed_group(h) ? 0 : (tile_rows + 3) / 4 * 4)) return false;
    for (int threads : {64, 128, 256, 512, 1024}) {
        const int sets = words_sets(h, threads);
        const int m = tile_rows / sets;
        if (m >= 1 && m * sets == tile_rows && m <= kMaxWord && words_worth(h, m)) return true;
    }
    for (int m = kSiteWord + 1; words_worth(h, m); ++m)
        if (tile_rows == words_rows(m, 1) || tile_rows == words_rows(m, site_sets(h, true))) return true;
    return false;
}

// The shape a caller asked for (tile_rows > 0, group_replicas > 0 or both).
// The options keep the ranges documented for them: quads of replicas in byte
// planes, tiles that fit the workgroup's LDS at one byte per spin (and with +-1
// couplings, L = 8 and 16, whole passes of 8 and 2 rows; group_replicas is
// ignored there and where a lattice has no quads).  The tile's rows are then
// swept in the words and sets of the shortest launch.  (Words of 32 replicas in
// the lanes that few sets have blocks for, eight at L = 4: tile 128, group 64,
// R = 1000, 41 temperatures in 7.5 ms; now 1.9, quads of byte planes 2.8.  L = 8,
// tile 64: 7.8, 3.3 and 3.5; real couplings, L = 8, tile 64, R = 20000: 27.6,
// 8.2 and 12.9.)  What the library itself reports for a shape of its choice is
// taken back whatever those ranges are, and as that shape where it is the
// default or the one measured for this instance.
// h holds the default shape on entry.
bool explicit_shape(HostInst &h, int tile_rows, int group_replicas, const char **why)
{
    const char *w = nullptr;
    const int rb = h.row_bytes;
    const int asked = tile_rows;
    if (is_rb(h) && (h.L == 8 || h.L == 16)) {
        const int p = h.L == 8 ? 8 : 2;
        tile_rows = (tile_rows + p - 1) / p * p;
        if (tile_rows > 4096)
            w = "tile_rows must be in [1, 4096]";
        else if ((int64_t)tile_rows * h.N + 32 + 4 * (int64_t)tile_rows > kMaxLds)
            w = "the workgroup's tile does not fit in LDS";
    } else if (fixed_group(h)) {
        if ((int64_t)tile_rows * ((h.N + 15) & ~15) + 32 + 4 * (int64_t)tile_rows > kMaxLds)
            w = "the workgroup's tile does not fit in LDS";
    } else {
        const int rp0 = cm_replicas_per_block(h.tpr), rp = group_replicas > 0 ? group_replicas / 4 : rp0;
        const int64_t m = std::max<int64_t>(1, std::min<int64_t>(4, h.Rcap / (512 * 4 * rp0)));
        if (tile_rows <= 0) tile_rows = (int)m * 4 * rp;
        const int64_t slot = cm_slot_bytes(rb, h.tpr, is_rb(h) ? 8 : 4);
        int64_t table = 0;
        if (is_rb(h)) {
            table = h.ncol == 3 ? 16 + 144 * h.tpr : h.tpr <= 128 ? 16 + 96 * h.tpr : 0;
            if (slot * rp0 + 32 + 4 * 64 + table > kMaxLds || 8 * (int64_t)cm_plane_bytes(rb) > 65536) table = 0;
        }
        if (tile_rows > 4096)
            w = "tile_rows must be in [1, 4096]";
        else if (rp < 1 || (h.tpr <= 64 && (h.tpr * rp) % 64 != 0) || cm_launch_threads(h.tpr, rp) > 1024)
            w = "group_replicas must be a multiple of four giving at most 1024 threads (whole waves when a quad "
                "takes at most 64)";
        else if (slot * rp + 32 + (is_rb(h) ? 4 : 8) * (int64_t)tile_rows + table > kMaxLds)
            w = "the workgroup's tile does not fit in LDS";
    }
    if (reported_shape(h, asked, group_replicas)) {
        w = nullptr;
        if (h.tile_rows == asked && 4 * h.rp == group_replicas) return true;
        HostInst known = shape_of(h);
        if (cached_shape({device_tag(), cache_key(h)}, known, nullptr) && known.tile_rows == asked &&
            4 * known.rp == group_replicas) {
            take_shape(h, known);
            return true;
        }
    }
    if (why) *why = w;
    if (w) return false;
    // m replicas per word, as many sets as n passes over the tile take
    const int rows = (int)std::min<int64_t>(tile_rows, h.R);
    HostInst t = shape_of(h);
    double best = INFINITY;
    for (int m = 1; m <= kSiteWord + 2; ++m) {
        if (!words_worth(h, m)) continue;
        for (int n = 1, sets = 0; sets != 1; n += std::max(1, n / 4)) {
            sets = (rows + words_rows(m, n) - 1) / words_rows(m, n);
            set_rb(t, m, sets, tile_rows);
            if (!shape_valid(t, nullptr)) continue;
            const double time = shape_time(h, m, sets, tile_rows, {h.R}, 1);
            if (time < 0.98 * best) {
                best = time;
                take_shape(h, t);
            }
        }
    }
    return shape_valid(h, why);
}

// Replicas per word worth trying.
constexpr int kWords[] = {1, 2, 4, 8, 12, 16, 20, 24, 28, 32};

static std::vector<HostInst> shape_candidates(const HostInst &h)
{
    std::vector<HostInst> c;
    HostInst t = shape_of(h);
    int last = 0;
    for (int threads : {64, 128, 256, 512, 1024}) {
        const int sets = words_sets(h, threads);
        if (sets == last) continue;
        last = sets;
        for (int m : kWords) {
            set_rb(t, m, sets, m * sets);
            if ((m == 1 || m * sets <= 2 * h.Rcap) && shape_valid(t, nullptr)) c.push_back(t);
        }
    }
    for (int m = kSiteWord + 1; words_worth(h, m); ++m)
        for (int sets : {1, 4}) {
            set_rb(t, m, sets, words_rows(m, sets));
            if (shape_valid(t, nullptr)) c.push_back(t);
        }
    return c;
}

int tune_shape(HostInst &h, const pamc_options &opt, double *ns_per_attempt)
{
    const Key k0 = cache_key(h);
    const auto key = std::make_pair(device_tag(), k0);
    HostInst known = shape_of(h);
    if (cached_shape(key, known, ns_per_attempt)) {
        take_shape(h, known);
        return PAMC_OK;
    }
    const auto cand = shape_candidates(h);
    if (cand.empty()) {
        set_error("no valid sweep shape for this lattice");
        return PAMC_ERR_INVALID;
    }
    // throw-away run at a constant beta: a burn-in that brings the energies
    // to that temperature (the epilogue's cost depends on how many distinct
    // energies a wave holds), then 1 + kTimedSteps steps per candidate
    pamc_options o = opt;
    o.timing = 1;
    o.graphs = 0;
    o.overlap_steps = nullptr;
    o.n_overlap_steps = 0;
    o.capacity = h.Rcap;
    o.tile_rows = 0;
    o.group_replicas = 0;
    o.autotune = 0;
    o.pop_schedule = nullptr;
    o.fuse_gather = 1;
    o.icm_rounds = 0;  // the shape concerns the sweep alone
    // (beta_0 = 0, where every run starts; then the constant tuning beta)
    const int nT = 1 + kBurnIn + (1 + kTimedSteps) * (int)cand.size();
    std::vector<double> beta((size_t)nT, kTuneBeta);
    beta[0] = 0.0;
    HostInst t;
    int st = make_inst(h.L, h.real ? nullptr : h.J.data(), h.real ? h.Jq.data() : nullptr, h.R, beta.data(), nT,
                       h.NS, h.seed, o, t);
    if (st != PAMC_OK) return st;
    Runner run;
    st = run.setup(o, 1);
    if (st != PAMC_OK) return st;
    const int slot = run.add_instance(std::move(t));
    if (slot < 0) return slot;
    st = run.init_instances({slot});
    if (st == PAMC_OK) st = run.build_work({slot});
    if (st != PAMC_OK) return st;
    const double attempts = (double)h.R * h.N * h.NS;
    st = run.enqueue_steps(kBurnIn);
    if (st == PAMC_OK) st = run.sync();
    if (st == PAMC_OK) st = run.phase_times(nullptr, nullptr, nullptr, nullptr);
    if (st != PAMC_OK) return st;
    Choice best{h.tile_rows, h.rp, h.mrep, h.sets, INFINITY};
    for (const auto &c : cand) {
        // one warm-up step, then the fastest of three timed steps
        st = run.set_shape(slot, c);
        double best_ms = INFINITY;
        for (int rep = 0; rep < 1 + kTimedSteps && st == PAMC_OK; ++rep) {
            double sw = 0.0;
            st = run.enqueue_steps(1);
            if (st == PAMC_OK) st = run.sync();
            if (st == PAMC_OK) st = run.phase_times(&sw, nullptr, nullptr, nullptr);
            if (rep > 0) best_ms = std::min(best_ms, sw);
        }
        if (st == PAMC_OK) st = run.inst_status(slot, nullptr, nullptr);
        if (st != PAMC_OK) return st;
        const double ns = best_ms * 1e6 / attempts;
        if (ns < best.ns_per_attempt) best = Choice{c.tile_rows, c.rp, c.mrep, c.sets, ns};
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_cache[key] = best;
        save_choice(key.first, k0, best);
    }
    h.tile_rows = best.tile_rows;
    h.rp = best.rp;
    h.mrep = best.mrep;
    h.sets = best.sets;
    h.own_shape = true;
    if (ns_per_attempt) *ns_per_attempt = best.ns_per_attempt;
    return PAMC_OK;
}

// Loads the persistent choices now (the serving loop does this before its
// first request arrives).
void tune_cache_load()
{
    std::lock_guard<std::mutex> lk(g_mu);
    load_persistent();
}

}  // namespace pamc
