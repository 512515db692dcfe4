// Host side of libislf: the C ABI declared in include/islf.h.
//
// Owns contexts (replica slots, device buffers, work lists), builds the
// Metropolis threshold tables in IEEE double (Sec. II.A Eq. 1 energy change,
// acceptance min(1, exp(-beta dE)) on a uint32 draw), and issues the kernels
// of islf_kernels.hip in the plain, batched or persistent form, optionally as
// a captured HIP graph.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <chrono>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "islf_internal.h"

namespace islf {
hipError_t launch_sweep(int fmt, int kind, const RepDesc *descs, RepState *st, const Entry *items,
                        const int *first, int grid, const int *reps, int n_reps, uint32_t s, uint32_t flags,
                        hipStream_t strm);
hipError_t sweep_blocks_per_cu(int fmt, int *per_cu);
hipError_t launch_fold(const RepDesc *descs, RepState *st, const int *reps, int n_reps, uint32_t s,
                       uint32_t advance, hipStream_t strm);
const void *persistent_kernel(int fmt);
const void *persistent_teams_kernel(int fmt);
hipError_t launch_persistent(int fmt, const RepDesc *descs, RepState *st, const Entry *items, const int *first,
                             const int *reps, int nreps, uint32_t nsweeps, GridSync *sync, int grid, hipStream_t s);
hipError_t launch_persistent_teams(int fmt, const RepDesc *descs, RepState *st, const Entry *items, const int *first,
                                   const TeamInfo *teams, uint32_t nsweeps, GridSync *sync, SyncLine *rsync,
                                   int n_rsync, int grid, hipStream_t s);
hipError_t launch_init(int fmt, const RepDesc *descs, RepState *st, int rep, int mode, long n, hipStream_t s);
hipError_t launch_import(int fmt, const RepDesc *descs, RepState *st, int rep, int Lz, uint32_t c0, uint32_t c1,
                         size_t h0, const int8_t *host, hipStream_t s);
hipError_t launch_export(int fmt, const RepDesc *descs, int rep, int Lz, uint32_t c0, uint32_t c1, size_t h0,
                         int8_t *out, hipStream_t s);
hipError_t launch_fetch(const unsigned long long *error, const void *ring, long first, long n, long size,
                        unsigned long long *host, hipStream_t s);
hipError_t launch_recompute(int fmt, const RepDesc *descs, RepState *st, int rep, long n, unsigned long long *out,
                            hipStream_t s);
hipError_t launch_layer_profile(const RepDesc *descs, int rep, long rows, long words_per_row, int32_t *out,
                                long long *acc, hipStream_t s);
hipError_t launch_zero(unsigned long long *p, long n, hipStream_t s);
hipError_t launch_energy(const islf_obs *rec, uint32_t cap, uint64_t first, uint32_t count, double J,
                         double H, double h1, double hn, double *out, hipStream_t s);
hipError_t launch_means(const RepDesc *descs, const int *reps, int n, uint64_t first, uint32_t count,
                        double *out, hipStream_t s);
hipError_t launch_integrate(const double *h, const double *m1, const double *mn, int n, double c1, double cn,
                            double norm, double *out, hipStream_t s);
hipError_t noalloc_scratch(double **out);
hipError_t resident_lds_limit(int fmt, size_t bytes);
hipError_t launch_resident(int fmt, int form, const ResLaunch &L, size_t lds, hipStream_t s);
hipError_t launch_mark(ResSync *rs, unsigned long long *host, hipStream_t s);
}  // namespace islf

using namespace islf;

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string g_err;

static islf_status fail(islf_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

#define HIP_TRY(expr)                                                                     \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return fail(ISLF_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));     \
    } while (0)

extern "C" const char *islf_last_error(void) { return g_err.c_str(); }

// ---------------------------------------------------------------------------
// tile variants (main tiles, rows 2 .. Ly-2, both formats): a workgroup owns
// tj columns x ty rows (tj*ty <= 256 threads) and each thread marches through
// mx x planes; a column is an 8-byte column of a sublattice half-row (int8)
// or a 32-bit word of a sublattice row (bit-packed), and tj is the most even split of a row's
// columns into pieces of at most tj_max.  Seam-slab tiles (rows Ly-1, 0, 1):
// np mirror pairs of x planes x nj columns with np*nj <= 128, so that a row
// stage has at most one task per thread.
// ---------------------------------------------------------------------------
struct I8Tile {
    int tj_max, mx;
};
// tj_max = 0: linear tiles (a workgroup takes kBlock consecutive columns of
// a plane's main rows in row-major order, whatever the row length)
static const I8Tile kI8Tiles[] = {
    {16, 16}, {32, 16}, {64, 16}, {128, 16}, {256, 16}, {16, 8},  {32, 8},   {64, 8},
    {16, 32}, {32, 32}, {64, 32}, {128, 32}, {16, 64}, {32, 64}, {64, 64}, {256, 64},
    {0, 16},  {0, 8},   {0, 32},  {0, kMaxMarch},
};
static const I8Tile kBpTilesM[] = {
    {16, 4}, {32, 4}, {64, 4}, {8, 4}, {4, 4}, {16, 2}, {16, 8}, {32, 8}, {8, 8}, {64, 8}, {4, 8}, {16, 16},
    {0, 4},  {0, 2},  {0, 8},  {0, kMaxMarch},
};
static const int kNumBpTilesM = (int)(sizeof(kBpTilesM) / sizeof(kBpTilesM[0]));
static const int kNumI8Tiles = (int)(sizeof(kI8Tiles) / sizeof(kI8Tiles[0]));

static int num_tiles_of(int fmt) { return fmt == ISLF_SPIN_INT8 ? kNumI8Tiles : kNumBpTilesM; }

static long ceil_div(long a, long b) { return (a + b - 1) / b; }

// Columns of one sublattice row a thread takes: 8-byte columns (8 sites,
// int8) or 32-bit words (32 sites, bit-packed).
static long columns_of(const islf_replica_desc &d, int fmt)
{
    return fmt == ISLF_SPIN_INT8 ? (d.Lz + 15) / 16 : (d.Lz + 63) / 64;
}

struct I8Shape {
    int tj, ty, mx;
};
static I8Shape i8_shape(const islf_replica_desc &d, int tile, int fmt = ISLF_SPIN_INT8)
{
    const long C = columns_of(d, fmt);
    const I8Tile &t = fmt == ISLF_SPIN_INT8 ? kI8Tiles[tile] : kBpTilesM[tile];
    I8Shape s;
    s.mx = std::min(t.mx, d.Lx);
    if (t.tj_max == 0) {
        s.tj = s.ty = 0;
        return s;
    }
    const long pieces = ceil_div(C, t.tj_max);
    s.tj = (int)ceil_div(C, pieces);
    s.ty = (int)std::min<long>(kBlock / s.tj, std::max(1, d.Ly - 3));
    return s;
}

// fraction of a plane's thread slots that own a real column / word (the x
// extent costs nothing: plans cut tiles by x steps)
static double tile_efficiency(const islf_replica_desc &d, int fmt, int tile)
{
    const double ny = d.Ly - 3;
    if (ny <= 0) return 1.0;
    const long C = columns_of(d, fmt);
    const I8Shape s = i8_shape(d, tile, fmt);
    const double per_plane = s.tj == 0 ? (double)ceil_div((long)ny * C, kBlock)
                                       : (double)ceil_div((long)ny, s.ty) * ceil_div(C, s.tj);
    return ny * C / (per_plane * kBlock);
}

// The variant with the fewest idle thread slots among the default x extents
// (16 planes int8, 4 bit-packed) and the linear tile over the whole x range;
// that one wins ties: a workgroup's share of a plan is then mostly one
// contiguous piece, with one set-up (view, tables, first loads, flush)
// instead of one per tile.
static int default_tile(const islf_replica_desc *d, int fmt)
{
    double best = -1.0;
    int best_i = 0;
    for (int i = 0; i < num_tiles_of(fmt); ++i) {
        const I8Tile &t = fmt == ISLF_SPIN_INT8 ? kI8Tiles[i] : kBpTilesM[i];
        const bool whole = t.tj_max == 0 && t.mx == kMaxMarch;
        if (!whole && t.mx != (fmt == ISLF_SPIN_INT8 ? 16 : 4)) continue;
        const double eff = tile_efficiency(*d, fmt, i);
        if (eff > best + 1e-9 || (whole && eff > best - 1e-9)) {
            best = std::max(best, eff);
            best_i = i;
        }
    }
    return best_i;
}

struct SlabShape {
    int np, nj;
};
// the (pairs, columns) split with the fewest idle thread slots, then the
// fewest entries
static SlabShape slab_shape(const islf_replica_desc &d, int fmt)
{
    const long J = columns_of(d, fmt);
    const long P = (d.Lx + 1) / 2;
    const long cap = kBlock / 2;
    SlabShape best{1, 1};
    long best_cost = -1;
    for (long pieces = ceil_div(J, cap); pieces <= J; ++pieces) {
        const long nj = ceil_div(J, pieces);
        if (ceil_div(J, nj) != pieces) continue;
        const long np0 = std::min(P, std::max(1l, cap / nj));
        const long np = ceil_div(P, ceil_div(P, np0));
        const long entries = ceil_div(P, np) * pieces;
        const long cost = entries * cap;   // thread slots of one row stage
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = SlabShape{(int)np, (int)nj};
        }
    }
    return best;
}

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------
struct Replica {
    islf_replica_desc desc{};
    bool live = false;
    void *mem = nullptr;     // spins | records | accumulators
    size_t mem_bytes = 0;
    uint64_t t_host = 0;     // sweeps issued so far
    bool failed = false;     // its chain was cut short by a failed launch
    int tile = 0;
    bool tile_set = false;   // chosen by islf_set_tile
    RepDesc d{};
    std::vector<Entry> main, slab;
};

// A launch plan: `grid` workgroups, workgroup b running items
// [first[b], first[b+1]) (device arrays); slab items come first and sit in
// workgroups [0, slab_grid).
struct Plan {
    Entry *items = nullptr;
    int *first = nullptr;
    long items_cap = 0, first_cap = 0;
    int grid = 0, slab_grid = 0;
    bool valid = false;
};

// A launch of the resident form over some replicas: shares (jobs) by
// workgroup, cluster workgroups first, with their mailboxes and per-sweep sums.
struct ResPlan {
    bool valid = false;    // planned for the current replicas
    bool usable = false;   // they fit and the tables are on the device
    bool put_off = false;  // they fit, but the launch chain was the faster form when it was planned: no tables yet
    ResLaunch L{};         // the plan's tables (device memory) and counts; the rest is the context's, filled in per launch
    size_t jobs_b = 0, first_b = 0, planes_b = 0, rows_b = 0, reps_b = 0, part_b = 0, mbox_b = 0;   // bytes allocated
    int form = RES_WORDS;  // RES_GROUPS: no clusters and few words per film; RES_FINE: few words per stage
    size_t lds = 0;
    uint32_t max_sweeps = 0;
    double sweep_us = 0.0, fixed_us = 0.0;   // expected: per sweep, per launch
    long long sites = 0;
    int nreps = 0;
};

// A number of shares worth taking for a film: fewer are slower.
struct ShareChoice {
    int P, px, py;
    double us;
};

constexpr size_t kMaxShapes = 256;
constexpr long kResultWords = 8192;            // 64 KiB of results
constexpr size_t kWindow = 2u << 20;           // bytes of spins per window
constexpr size_t kPlanBytes = 32u << 20;       // of resident plans (3 x 160x480x600: 8 MB; thin films of 9,000-site rows: 20 MB)

struct islf_ctx {
    int fmt = 0;
    uint32_t cap = 0;
    hipStream_t stream = nullptr;
    islf_alloc_fn alloc = nullptr;
    islf_free_fn free_fn = nullptr;
    void *user = nullptr;
    int exec = ISLF_EXEC_BATCHED;
    int num_cu = 0;
    int resident_slots = 0;    // workgroups of the sweep kernels resident at once on the device
    int sweep_slots = 0;       // default workgroups per sweep launch (2 per resident slot)
    int grid_override = 0;     // workgroups per batched / plain launch (0: sweep_slots)
    double taper_override = -1.0;   // share taper of the batched and persistent plans (< 0: the built-in one)
    // islf_autotune's launch configuration of the chain is in use, not a caller's;
    // tuned_us: a sweep of this batch with it, measured (0: of another batch), in form tuned_exec
    bool tuned = false;
    double tuned_us = 0.0;
    int tuned_exec = -1;
    bool chain_only = false;   // while it is being tuned
    int persistent_grid = 0;   // workgroups of the persistent kernel's cooperative launch
    int persistent_bound = 0;  // co-residency bound computed for it on this device
    double *noalloc_scratch = nullptr;   // this device's copy of the means scratch array

    std::vector<Replica> reps;
    int slot_capacity = 0;
    RepDesc *d_desc = nullptr;
    RepState *d_state = nullptr;
    GridSync *d_sync = nullptr;
    // team form of the persistent plan: per-workgroup team records and one
    // arrival counter per replica slot
    bool persistent_teams = false;
    TeamInfo *d_teams = nullptr;
    long teams_cap = 0;
    SyncLine *d_rsync = nullptr;
    int rsync_cap = 0;
    int team_mode = -1;        // 1: team barriers when every live replica can have a workgroup; 0: grid; -1: automatic
    unsigned long long *d_scratch = nullptr;   // 64 x u64
    // what calls bring back, in pinned memory: word 0 the error word, HOST_*,
    // results from word 8 on; and two windows for spins too many for it (made by the
    // first call with such spins)
    unsigned long long *h_res = nullptr;
    int8_t *h_win = nullptr;
    hipEvent_t win_event[2] = {};
    int *d_live = nullptr;                      // live replica ids
    int live_capacity = 0;
    Plan batched, persistent;
    std::vector<Plan> plain;                    // per slot
    ResPlan resident;                           // all live replicas (batched and persistent forms)
    std::vector<ResPlan> resident_plain;        // per slot (plain form)
    ResSync *d_rsy = nullptr;
    // turns among the contexts of a device (see Turns; under its lock)
    int device = 0;
    hipEvent_t turn = nullptr;     // recorded on its stream by a context that is to come behind it
    uint32_t issued = 0;           // cluster launches and marks that will count HOST_ENDED up;
    uint32_t cluster_until = 0;    // the last one of clusters,
    uint32_t chain_until = 0;      // of the chain or the persistent kernel by its own choice,
    uint32_t joined_until = 0;     // and because another context's chain was in flight
    bool unmarked = false;         // a chain that is not counted is in flight
    int members = 0;               // cluster workgroups of the launches in flight, at most
    uint32_t aborts_seen = 0;
    bool chain_if_met = false;     // its last run with clusters would rather be a chain beside another context's
    int apart = 0;                 // runs that keep to the chain
    uint64_t cluster_runs = 0, chain_runs = 0;
    // batched form with concurrent replica groups: group g sweeps its
    // replicas on side_stream[g], a stream the context creates; the
    // context's stream only forks them and joins them
    int groups_req = 0;                         // 0: automatic
    bool groups_valid = false;
    std::vector<Plan> group_plan;
    std::vector<int> group_off, group_len;      // into d_group_live
    int *d_group_live = nullptr;
    int group_live_cap = 0;
    std::vector<hipStream_t> side_stream;       // group g issues on side_stream[g]
    std::vector<hipEvent_t> side_event;         // [0] fork, [g+1] join of group g
    std::vector<int> live;
    bool dirty = true;

    // captured sweeps: one single-stream graph per concurrent group (one
    // graph otherwise), replayed on the group's stream
    std::vector<hipGraph_t> graphs;
    std::vector<hipGraphExec_t> graph_execs;
    uint32_t graph_sweeps = 0;
    bool graph_valid = false;
    int graph_exec = 0;             // the form it was captured in,
    bool graph_resident = false;    // resident or not,
    int graph_members = 0;          // with so many cluster workgroups at most
    uint32_t graph_launches = 0;    // and so many launches of them;
    bool graph_prefers_chain = false;

    // the cuts of the shapes planned so far (kMaxShapes at most)
    std::map<std::array<int, 4>, std::vector<ShareChoice>> choices;

    // device bytes the context holds, by allocation
    std::unordered_map<void *, size_t> alloc_bytes;
    size_t dev_bytes = 0;
};

static islf_status check_none_failed(const islf_ctx *c);

static void *dev_alloc(islf_ctx *c, size_t bytes)
{
    if (bytes == 0) bytes = 256;
    void *p = nullptr;
    if (c->alloc) p = c->alloc(bytes, c->user);
    else if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
    if (p) {
        c->alloc_bytes[p] = bytes;
        c->dev_bytes += bytes;
    }
    return p;
}

static void dev_free(islf_ctx *c, void *p)
{
    if (!p) return;
    auto it = c->alloc_bytes.find(p);
    if (it != c->alloc_bytes.end()) {
        c->dev_bytes -= it->second;
        c->alloc_bytes.erase(it);
    }
    if (c->free_fn) c->free_fn(p, c->user);
    else (void)hipFree(p);
}

// ---------------------------------------------------------------------------
// validation, sizes, thresholds
// ---------------------------------------------------------------------------
static islf_status validate(const islf_replica_desc *d)
{
    if (!d) return fail(ISLF_EINVAL, "NULL replica descriptor");
    if (d->Lx < 1 || d->Ly < 2 || d->Lz < 2 || (d->Lz & 1))
        return fail(ISLF_EINVAL, "invalid shape %dx%dx%d (need Lx>=1, Ly>=2, Lz>=2 even)", d->Lx, d->Ly, d->Lz);
    if (d->ybc < 0 || d->ybc > 2) return fail(ISLF_EINVAL, "invalid y boundary %d", d->ybc);
    if (d->init < 0 || d->init > 3) return fail(ISLF_EINVAL, "invalid init mode %d", d->init);
    if (!(d->beta >= 0.0)) return fail(ISLF_EINVAL, "beta must be >= 0 (got %g)", d->beta);
    if (!isfinite(d->J) || !isfinite(d->H) || !isfinite(d->h1) || !isfinite(d->hn))
        return fail(ISLF_EINVAL, "J, H, h1, hn must be finite");
    const unsigned long long rows = (unsigned long long)d->Lx * (unsigned long long)d->Ly;
    const unsigned long long groups = rows * (unsigned long long)((d->Lz + 7) / 8);   // Philox groups of 8 z
    if (groups * 2ull > (1ull << 32))
        return fail(ISLF_ERANGE, "lattice %dx%dx%d exceeds the 32-bit Philox group counter", d->Lx, d->Ly, d->Lz);
    if (rows * 16ull * (unsigned long long)((d->Lz + 15) / 16) >= (1ull << 32))
        return fail(ISLF_ERANGE, "lattice %dx%dx%d exceeds 4 GiB of int8 spins", d->Lx, d->Ly, d->Lz);
    return ISLF_OK;
}

static size_t spin_bytes(const islf_replica_desc *d, int fmt)
{
    const size_t rows = (size_t)d->Lx * d->Ly;
    if (fmt == ISLF_SPIN_INT8) return rows * 16 * (size_t)((d->Lz + 15) / 16);
    return rows * 2 * 4 * (size_t)((d->Lz + 63) / 64);
}

static size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static size_t replica_bytes(const islf_replica_desc *d, int fmt, uint32_t cap)
{
    return round_up(spin_bytes(d, fmt), 256) + round_up((size_t)cap * sizeof(islf_obs), 256) +
           2 * kAccSlots * 4 * sizeof(long long);
}

// thr = 2^32 if dE <= 0 else floor(2^32 exp(-beta dE)), with
// dE = 2 s (J n + h), n = 2*cnt - k, h the field of the site's layer.
// Alongside: thr - 1 as 32 bits, the packed change (dB, dM) = (-2 s n, -2 s)
// of a flip as dB + 65536 dM, and the set of moves that can never be taken.
static void build_tables(const islf_replica_desc *d, RepDesc &D)
{
    uint64_t *thr = D.thr;
    D.never_mask = 0;
    for (int c = 0; c < kClasses; ++c) {
        double h = d->H;
        if (c & 1) h = h + d->h1;
        if (c & 2) h = h + d->hn;
        const int k = 6 - ((c & 1) ? 1 : 0) - ((c & 2) ? 1 : 0);
        for (int u = 0; u < 2; ++u) {
            const int s = 2 * u - 1;
            for (int cnt = 0; cnt < 8; ++cnt) {
                uint64_t v = 0;
                int32_t dp = 0;
                const int i = c * kThrPerClass + u * 8 + cnt;
                if (cnt <= k) {
                    const int n = 2 * cnt - k;
                    const double dE = 2.0 * (double)s * (d->J * (double)n + h);
                    if (dE <= 0.0) v = 1ull << 32;
                    else v = (uint64_t)floor(ldexp(exp(-(d->beta * dE)), 32));
                    dp = (-2 * s * n) + 65536 * (-2 * s);
                    if (v == 0) D.never_mask |= 1ull << i;
                }
                thr[i] = v;
                D.thr_m1[i] = v ? (uint32_t)(v - 1) : 0u;
                D.dpack[i] = dp;
            }
        }
    }
}

// Without a bulk field (H = 0) and with J >= 0 a bulk move costs energy only
// from four aligned neighbours on, and the same for both spins: four
// thresholds, the first of them "always".
static void build_sym(RepDesc &D)
{
    const uint64_t *t = D.thr;
    bool sym = true;
    for (int a = 0; a <= 6; ++a) {
        const uint64_t up = t[8 + a], down = t[6 - a];   // a aligned neighbours of an up / a down spin
        sym = sym && up == down && (a > 3 || up == 1ull << 32);
    }
    D.sym = sym ? 1 : 0;
    for (int c = 0; c < 4; ++c) D.thr_q[c] = D.thr_m1[8 + 3 + c];
}

static void build_work(Replica &R, int rep_id, int fmt)
{
    const islf_replica_desc &d = R.desc;
    R.main.clear();
    R.slab.clear();
    const int J = (int)columns_of(d, fmt);
    const I8Shape s = i8_shape(d, R.tile, fmt);
    const int cols = std::max(0, d.Ly - 3) * J;   // main columns of a plane (rows 2 .. Ly-2)
    for (int x0 = 0; x0 < d.Lx; x0 += s.mx) {
        if (s.tj == 0) {
            // linear tile: y0 = first column, j0 = end of the range
            for (int c0 = 0; c0 < cols; c0 += kBlock)
                R.main.push_back(Entry{rep_id, x0, c0, std::min(c0 + kBlock, cols), std::min(s.mx, d.Lx - x0),
                                       ITEM_MAIN});
            continue;
        }
        for (int y0 = 2; y0 < d.Ly - 1; y0 += s.ty)
            for (int j0 = 0; j0 < J; j0 += s.tj)
                R.main.push_back(Entry{rep_id, x0, y0, j0, std::min(s.mx, d.Lx - x0), ITEM_MAIN});
    }
    R.d.i8_tj = s.tj;
    R.d.i8_ty = s.ty;
    R.d.i8_mx = s.mx;
    const SlabShape sl = slab_shape(d, fmt);
    const int P = (d.Lx + 1) / 2;
    for (int p0 = 0; p0 < P; p0 += sl.np)
        for (int j0 = 0; j0 < J; j0 += sl.nj)
            R.slab.push_back(Entry{rep_id, p0, std::min(sl.np, P - p0), j0, std::min(sl.nj, J - j0), ITEM_SLAB});
}

// The number of entries that build_work makes.
static size_t work_entries(const islf_replica_desc &d, const I8Shape &s, int fmt)
{
    const int J = (int)columns_of(d, fmt), rows = std::max(0, d.Ly - 3);
    const SlabShape sl = slab_shape(d, fmt);
    const size_t main = (size_t)ceil_div(d.Lx, s.mx) *
                        (s.tj == 0 ? (size_t)ceil_div((long)rows * J, kBlock)
                                   : (size_t)ceil_div(rows, s.ty) * (size_t)ceil_div(J, s.tj));
    return main + (size_t)ceil_div((d.Lx + 1) / 2, sl.np) * (size_t)ceil_div(J, sl.nj);
}

static void fill_desc(Replica &R, int fmt, uint32_t cap)
{
    const islf_replica_desc &d = R.desc;
    RepDesc &D = R.d;
    uint8_t *m = (uint8_t *)R.mem;
    D.spins = m;
    const size_t sb = round_up(spin_bytes(&d, fmt), 256);
    D.rec = (islf_obs *)(m + sb);
    D.acc = (long long *)(m + sb + round_up((size_t)cap * sizeof(islf_obs), 256));
    build_tables(&d, D);
    build_sym(D);
    D.Lx = d.Lx; D.Ly = d.Ly; D.Lz = d.Lz;
    D.C = (d.Lz + 7) / 8;
    D.K = (d.Lz + 15) / 16;
    D.Hp = 8 * D.K;
    D.RB = 2 * D.Hp;
    D.Wq = (d.Lz + 63) / 64;
    D.seam_reflect = d.ybc == ISLF_YBC_GAPBC;
    D.seam_invert = d.ybc != ISLF_YBC_PBC;
    D.key0 = (uint32_t)(d.seed & 0xFFFFFFFFull);
    D.key1 = (uint32_t)(d.seed >> 32);
    D.replica = d.replica;
    D.cap = cap;
    D.fmt = fmt;
    D.J = d.J; D.H = d.H; D.h1 = d.h1; D.hn = d.hn;
}

// ---------------------------------------------------------------------------
// device-side tables
// ---------------------------------------------------------------------------
static islf_status ensure_slots(islf_ctx *c, int n)
{
    if (n <= c->slot_capacity) return ISLF_OK;
    int cap = std::max(n, std::max(16, 2 * c->slot_capacity));
    RepDesc *nd = (RepDesc *)dev_alloc(c, sizeof(RepDesc) * cap);
    RepState *ns = (RepState *)dev_alloc(c, sizeof(RepState) * cap);
    if (!nd || !ns) {
        dev_free(c, nd);
        dev_free(c, ns);
        return fail(ISLF_ENOMEM, "cannot allocate replica tables for %d slots", cap);
    }
    HIP_TRY(launch_zero((unsigned long long *)ns, (long)(sizeof(RepState) * cap / 8), c->stream));
    if (c->d_state) {
        HIP_TRY(hipMemcpyAsync(ns, c->d_state, sizeof(RepState) * c->slot_capacity, hipMemcpyDeviceToDevice,
                               c->stream));
        HIP_TRY(hipMemcpyAsync(nd, c->d_desc, sizeof(RepDesc) * c->slot_capacity, hipMemcpyDeviceToDevice,
                               c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
    }
    dev_free(c, c->d_desc);
    dev_free(c, c->d_state);
    c->d_desc = nd;
    c->d_state = ns;
    c->slot_capacity = cap;
    c->graph_valid = false;
    return ISLF_OK;
}

static void free_plan(islf_ctx *c, Plan &p)
{
    dev_free(c, p.items);
    dev_free(c, p.first);
    p = Plan();
}

// Shares of a launch are tapered by dispatch rank (later workgroups get
// less) against the uneven progress of the workgroups resident on one CU
// (issue goes oldest first).  Measured on the 3 x 160x480x600 workload, by
// graph replay of the grouped batched form: bit-packed is fastest untapered
// (+1.2% over +-20%), int8 at +-10..30% (+0.5%).
static double tail_taper(int fmt)
{
    return fmt == ISLF_SPIN_BITPACK ? 0.0 : 0.1;
}
// a plain launch holds one replica: shorter launches, whose tails weigh more
constexpr double kPlainTaper = 0.2;
// the persistent launch has no second round of workgroups to fill a CU
// whose resident workgroups finish at different times: issue goes oldest
// first, and per-workgroup timestamps of a launch over three 46M lattices
// showed the workgroups of the first, second and third dispatch round (one
// per CU each) finishing equal shares after 19.6, 27 and 36 us.  Its shares
// therefore step down by dispatch round (grid and team barriers alike);
// 0.4 measured best or within noise of it (grid barriers: bit-packed 1,869
// against 1,812 untapered, int8 1,133 against 1,122; teams: int8 1,297
// against 1,152, bit-packed 1,653 against 1,614; 0 .. 0.7 tried)
constexpr double kPersistentTaper = 0.4;
// three concurrent groups: measured as fast as two and faster than four on
// every batch tried (3 x 160x480x600, 64 x 40x120x120, 96 uneven replicas);
// four group streams can share one of the process's four hardware queues
constexpr int kAutoGroups = 3;
constexpr int kMaxStreamGroups = 16;   // concurrent replica groups of the batched form (hardware queues per process)

// Splits the work into about `grid` runs of equal cost, one per workgroup:
// workgroup b gets items [first[b], first[b+1]).  The slab items are spread
// over the first min(grid, #slab) workgroups (so that a final launch of
// those workgroups covers them all); main tiles follow in order and fill
// every workgroup up to its share.  A main tile costs 4 units per x step and
// may be cut between steps; a slab tile costs 6 units (1.5 steps) per task
// per thread over its three row stages and is never cut.  The runs may be a
// part of a larger launch: run r is then the launch's run p0 + r of
// launch_grid, which sets its dispatch rank for the taper.  Returns the
// number of workgroups holding slab items.
static int partition_items(const std::vector<Entry> &slab, const std::vector<Entry> &main, int grid,
                           std::vector<Entry> &items, std::vector<int> &first, double taper, int p0 = 0,
                           int launch_grid = 0, int round = 0)
{
    auto slab_cost = [](const Entry &e) -> long long {
        const long long tasks = 6ll * e.y0 * e.nsteps;
        return 6 * ((tasks + kBlock - 1) / kBlock);
    };
    const long long ns = (long long)slab.size();
    long long W = 0, steps = 0;
    for (const Entry &e : slab) W += slab_cost(e);
    for (const Entry &e : main) steps += e.nsteps;
    W += 4 * steps;
    grid = (int)std::max(1ll, std::min((long long)grid, ns + steps));
    const long long gs = std::min<long long>(grid, ns);   // workgroups holding slab items
    items.clear();
    first.assign(1, 0);
    size_t mi = 0;   // next main tile and x offset inside it
    int off = 0;
    long long acc = 0;
    // cumulative cost targets: run r goes to the workgroup dispatched at rank
    // d(r) (the inverse of the kernel's XCD-contiguous mapping); later ranks
    // get smaller shares, weight 1 + a (1 - 2 u) at u = (d + 0.5) / grid
    const double a = taper;
    const long LG = launch_grid > 0 ? launch_grid : grid;
    std::vector<double> cum(grid + 1, 0.0);
    const long q = LG / 8, r8 = LG % 8;
    for (int r = 0; r < grid; ++r) {
        // the kernel gives XCD x (blocks x, x+8, ...) the runs from x*q + min(x, r8)
        const long rg = std::min<long>(p0 + r, LG - 1);
        long x, k;
        if (rg < r8 * (q + 1)) {
            x = rg / (q + 1);
            k = rg % (q + 1);
        } else {
            x = r8 + (rg - r8 * (q + 1)) / q;
            k = (rg - r8 * (q + 1)) % q;
        }
        const long d = x + 8 * k;
        // round > 0: a cooperative grid of `round` workgroups per dispatch
        // round (one per CU); the taper is a step per round
        const double u = round > 0 ? ((double)(d / round) + 0.5) / (double)((LG + round - 1) / round) : (d + 0.5) / LG;
        cum[r + 1] = cum[r] + 1.0 + a * (1.0 - 2.0 * u);
    }
    for (int b = 0; b < grid; ++b) {
        const long long target = (long long)((double)W * cum[b + 1] / cum[grid]);
        if (b < gs)
            for (long long k = b * ns / gs; k < (b + 1) * ns / gs; ++k) {
                items.push_back(slab[k]);
                acc += slab_cost(slab[k]);
            }
        while (mi < main.size() && (b == grid - 1 || target - acc >= 2)) {
            const Entry &e = main[mi];
            const int rem = e.nsteps - off;
            const int take = b == grid - 1 ? rem : (int)std::min<long long>(rem, std::max(1ll, (target - acc + 2) / 4));
            Entry piece = e;
            piece.x0 = e.x0 + off;
            piece.nsteps = take;
            items.push_back(piece);
            acc += 4ll * take;
            off += take;
            if (off == e.nsteps) {
                ++mi;
                off = 0;
            }
        }
        first.push_back((int)items.size());
        if (b + 1 >= gs && mi == main.size()) break;   // nothing left for later workgroups
    }
    return (int)gs;
}

static islf_status upload_plan(islf_ctx *c, Plan &p, const std::vector<Entry> &items, const std::vector<int> &first);

static islf_status build_plan(islf_ctx *c, Plan &p, const std::vector<Entry> &slab, const std::vector<Entry> &main,
                              int grid, double taper = -1.0, int round = 0)
{
    std::vector<Entry> items;
    std::vector<int> first;
    p.slab_grid = partition_items(slab, main, grid, items, first, taper < 0.0 ? tail_taper(c->fmt) : taper, 0, 0,
                                  round);
    return upload_plan(c, p, items, first);
}

static islf_status upload_plan(islf_ctx *c, Plan &p, const std::vector<Entry> &items, const std::vector<int> &first)
{
    p.grid = (int)first.size() - 1;
    if ((long)items.size() > p.items_cap) {
        dev_free(c, p.items);
        p.items_cap = std::max<long>((long)items.size(), 2 * p.items_cap);
        p.items = (Entry *)dev_alloc(c, sizeof(Entry) * p.items_cap);
        if (!p.items) return fail(ISLF_ENOMEM, "cannot allocate a launch plan");
    }
    if ((long)first.size() > p.first_cap) {
        dev_free(c, p.first);
        p.first_cap = std::max<long>((long)first.size(), 2 * p.first_cap);
        p.first = (int *)dev_alloc(c, sizeof(int) * p.first_cap);
        if (!p.first) return fail(ISLF_ENOMEM, "cannot allocate a launch plan");
    }
    if (!items.empty())
        HIP_TRY(hipMemcpyAsync(p.items, items.data(), sizeof(Entry) * items.size(), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipMemcpyAsync(p.first, first.data(), sizeof(int) * first.size(), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    p.valid = true;
    return ISLF_OK;
}

// Rebuilds the live list and the device descriptors after a change of
// membership or tiles; launch plans are rebuilt on their next use.
static islf_status sync_tables(islf_ctx *c)
{
    if (!c->dirty) return ISLF_OK;
    // (the lists in use stay whole if the new one cannot be had)
    std::vector<int> live;
    const int n = (int)c->reps.size();
    for (int i = 0; i < n; ++i)
        if (c->reps[i].live) live.push_back(i);
    if ((int)live.size() > c->live_capacity) {
        const int cap = std::max<int>((int)live.size(), 2 * c->live_capacity);
        int *d = (int *)dev_alloc(c, sizeof(int) * cap);
        if (!d) return fail(ISLF_ENOMEM, "cannot allocate live list");
        dev_free(c, c->d_live);
        c->d_live = d;
        c->live_capacity = cap;
    }
    c->live = std::move(live);
    if (!c->live.empty())
        HIP_TRY(hipMemcpyAsync(c->d_live, c->live.data(), sizeof(int) * c->live.size(), hipMemcpyHostToDevice, c->stream));
    std::vector<RepDesc> all(n);
    for (int i = 0; i < n; ++i) all[i] = c->reps[i].d;
    if (n) HIP_TRY(hipMemcpyAsync(c->d_desc, all.data(), sizeof(RepDesc) * n, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->batched.valid = false;
    c->persistent.valid = false;
    for (Plan &p : c->plain) p.valid = false;
    c->groups_valid = false;
    c->resident.valid = false;
    for (ResPlan &p : c->resident_plain) p.valid = false;
    c->tuned_us = 0.0;
    c->dirty = false;
    c->graph_valid = false;
    return ISLF_OK;
}

// The plans the context's execution form launches, built if needed.
static int num_groups(const islf_ctx *c)
{
    const int nl = (int)c->live.size();
    const int want = c->groups_req ? c->groups_req : kAutoGroups;
    return std::max(1, std::min(want, nl));
}

// Workgroups per A / B launch of a form: the override, else two per resident
// slot for one launch chain.  Concurrent groups share the resident slots:
// together they keep 3/2 workgroups per slot in flight, split evenly among
// the groups (the tail of one group's launch is filled by the others').
static int launch_grid(const islf_ctx *c, int exec)
{
    if (c->grid_override) return c->grid_override;
    const int G = exec == ISLF_EXEC_BATCHED ? num_groups(c) : 1;
    if (G == 1) return c->sweep_slots;
    return (int)std::max(64l, (3l * c->resident_slots + G) / (2l * G));
}

// Concurrent groups of the batched form: live replicas dealt to the group
// with the fewest sites so far (largest first), one launch plan per group
// (launch_grid: 3/2 x resident slots / groups workgroups, so that all groups
// together keep about 3/2 per slot in flight and each group's tail is filled
// by the others' launches), the groups' live lists on the device, and the
// groups' streams and fork / join events.
static islf_status prepare_groups(islf_ctx *c)
{
    islf_status st = sync_tables(c);
    if (st != ISLF_OK) return st;
    if (c->groups_valid) return ISLF_OK;
    const int G = num_groups(c);
    std::vector<int> order(c->live);
    auto sites = [&](int r) {
        const islf_replica_desc &d = c->reps[r].desc;
        return (long long)d.Lx * d.Ly * d.Lz;
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return sites(a) > sites(b); });
    std::vector<std::vector<int>> grp(G);
    std::vector<long long> load(G, 0);
    for (int r : order) {
        const int g = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        grp[g].push_back(r);
        load[g] += sites(r);
    }
    std::vector<int> flat;
    c->group_off.assign(G, 0);
    c->group_len.assign(G, 0);
    for (int g = 0; g < G; ++g) {
        std::sort(grp[g].begin(), grp[g].end());
        c->group_off[g] = (int)flat.size();
        c->group_len[g] = (int)grp[g].size();
        flat.insert(flat.end(), grp[g].begin(), grp[g].end());
    }
    if ((int)flat.size() > c->group_live_cap) {
        dev_free(c, c->d_group_live);
        c->group_live_cap = std::max<int>((int)flat.size(), 2 * c->group_live_cap);
        c->d_group_live = (int *)dev_alloc(c, sizeof(int) * c->group_live_cap);
        if (!c->d_group_live) return fail(ISLF_ENOMEM, "cannot allocate group lists");
    }
    if (!flat.empty())
        HIP_TRY(hipMemcpyAsync(c->d_group_live, flat.data(), sizeof(int) * flat.size(), hipMemcpyHostToDevice,
                               c->stream));
    if ((int)c->group_plan.size() < G) c->group_plan.resize(G);
    for (int g = 0; g < G; ++g) {
        std::vector<Entry> S, M;
        for (int r : grp[g]) {
            S.insert(S.end(), c->reps[r].slab.begin(), c->reps[r].slab.end());
            M.insert(M.end(), c->reps[r].main.begin(), c->reps[r].main.end());
        }
        st = build_plan(c, c->group_plan[g], S, M, launch_grid(c, ISLF_EXEC_BATCHED), c->taper_override);
        if (st != ISLF_OK) return st;
    }
    while ((int)c->side_stream.size() < G) {
        hipStream_t sst = nullptr;
        HIP_TRY(hipStreamCreateWithFlags(&sst, hipStreamNonBlocking));
        c->side_stream.push_back(sst);
    }
    while ((int)c->side_event.size() < G + 1) {
        hipEvent_t ev = nullptr;
        HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        c->side_event.push_back(ev);
    }
    c->groups_valid = true;
    return ISLF_OK;
}

// The team form of the persistent plan: the grid's workgroups are dealt to
// the live replicas so that the largest number of sites per workgroup is as
// small as it can be (one each, then greedily), each replica's items are cut
// into equal-cost runs over its team, and the teams take contiguous plan
// slots (so a team's workgroups share an XCD where the team is small enough).
static islf_status build_team_plan(islf_ctx *c, int grid, double taper)
{
    const int nl = (int)c->live.size();
    std::vector<long long> sites(nl);
    for (int i = 0; i < nl; ++i) {
        const islf_replica_desc &d = c->reps[c->live[i]].desc;
        sites[i] = (long long)d.Lx * d.Ly * d.Lz;
    }
    // one workgroup each, then each further workgroup to the team with the
    // most sites per workgroup: the slowest team sets the launch's time
    std::vector<int> W(nl, 1);
    std::vector<std::pair<double, int>> heap;
    for (int i = 0; i < nl; ++i) heap.push_back({(double)sites[i], i});
    std::make_heap(heap.begin(), heap.end());
    for (int used = nl; used < grid; ++used) {
        std::pop_heap(heap.begin(), heap.end());
        const int i = heap.back().second;
        W[i] += 1;
        heap.back().first = (double)sites[i] / (double)W[i];
        std::push_heap(heap.begin(), heap.end());
    }
    std::vector<Entry> items;
    std::vector<int> first(1, 0);
    std::vector<TeamInfo> teams;
    for (int i = 0; i < nl; ++i) {
        const int r = c->live[i];
        std::vector<Entry> it;
        std::vector<int> fi;
        // the team's runs are the launch's runs first.size()-1 onwards: their
        // dispatch ranks in the launch set the taper
        partition_items(c->reps[r].slab, c->reps[r].main, W[i], it, fi, taper, (int)first.size() - 1, grid,
                        c->num_cu);
        const int n = (int)fi.size() - 1;
        const int off = (int)items.size();
        items.insert(items.end(), it.begin(), it.end());
        for (int b = 0; b < n; ++b) {
            first.push_back(off + fi[b + 1]);
            teams.push_back(TeamInfo{r, b, n, 0});
        }
    }
    if ((long)teams.size() > c->teams_cap) {
        dev_free(c, c->d_teams);
        c->teams_cap = std::max<long>((long)teams.size(), 2 * c->teams_cap);
        c->d_teams = (TeamInfo *)dev_alloc(c, sizeof(TeamInfo) * c->teams_cap);
        if (!c->d_teams) return fail(ISLF_ENOMEM, "cannot allocate team records");
    }
    if (c->slot_capacity > c->rsync_cap) {
        dev_free(c, c->d_rsync);
        c->rsync_cap = c->slot_capacity;
        c->d_rsync = (SyncLine *)dev_alloc(c, 2 * sizeof(SyncLine) * c->rsync_cap);
        if (!c->d_rsync) return fail(ISLF_ENOMEM, "cannot allocate team counters");
    }
    HIP_TRY(hipMemcpyAsync(c->d_teams, teams.data(), sizeof(TeamInfo) * teams.size(), hipMemcpyHostToDevice,
                           c->stream));
    c->persistent_teams = true;
    return upload_plan(c, c->persistent, items, first);
}

// Whether the persistent launch uses team barriers.  Automatic: teams for
// int8 spins or batches of 8 or more replicas, grid barriers for a few
// bit-packed replicas; measured (updates/ns, grid / team): 3 x 160x480x600
// bit-packed 1,780 / 1,562, int8 1,100 / 1,167; 64 x 40x120x120
// bit-packed 795 / 834, int8 646 / 779.  Teams need a workgroup for every
// live replica.
static bool use_teams(const islf_ctx *c, int grid)
{
    const int nl = (int)c->live.size();
    if (nl > grid) return false;
    if (c->team_mode >= 0) return c->team_mode == 1;
    return c->fmt == ISLF_SPIN_INT8 || nl >= 8;
}

static islf_status prepare_plans(islf_ctx *c, int exec)
{
    islf_status st = sync_tables(c);
    if (st != ISLF_OK) return st;
    auto lists = [&](const std::vector<int> &reps, std::vector<Entry> &S, std::vector<Entry> &M) {
        for (int r : reps) {
            S.insert(S.end(), c->reps[r].slab.begin(), c->reps[r].slab.end());
            M.insert(M.end(), c->reps[r].main.begin(), c->reps[r].main.end());
        }
    };
    if (c->live.empty()) return ISLF_OK;
    if (exec == ISLF_EXEC_BATCHED && num_groups(c) > 1) return prepare_groups(c);
    if (exec == ISLF_EXEC_BATCHED && !c->batched.valid) {
        std::vector<Entry> S, M;
        lists(c->live, S, M);
        return build_plan(c, c->batched, S, M, c->grid_override ? c->grid_override : c->sweep_slots,
                          c->taper_override);
    }
    if (exec == ISLF_EXEC_PERSISTENT && !c->persistent.valid) {
        std::vector<Entry> S, M;
        lists(c->live, S, M);
        const int grid = c->grid_override ? c->grid_override : c->persistent_grid;
        if (grid > c->persistent_bound)
            return fail(ISLF_ERANGE, "persistent grid %d exceeds the co-residency bound %d of this device", grid,
                        c->persistent_bound);
        // team plans taper by their launch-wide dispatch rounds too
        if (use_teams(c, grid))
            return build_team_plan(c, grid, c->taper_override >= 0.0 ? c->taper_override : kPersistentTaper);
        const double taper = c->taper_override >= 0.0 ? c->taper_override : kPersistentTaper;
        c->persistent_teams = false;
        return build_plan(c, c->persistent, S, M, grid, taper, c->num_cu);
    }
    if (exec == ISLF_EXEC_PLAIN) {
        if (c->plain.size() < c->reps.size()) c->plain.resize(c->reps.size());
        for (int r : c->live) {
            if (c->plain[r].valid) continue;
            std::vector<Entry> S, M;
            lists(std::vector<int>(1, r), S, M);
            st = build_plan(c, c->plain[r], S, M, c->grid_override ? c->grid_override : c->sweep_slots, kPlainTaper);
            if (st != ISLF_OK) return st;
        }
    }
    return ISLF_OK;
}


// ---------------------------------------------------------------------------
// Resident form: shares, plan and choice
// ---------------------------------------------------------------------------
static void free_resident(islf_ctx *c, ResPlan &p)
{
    dev_free(c, (void *)p.L.jobs);
    dev_free(c, (void *)p.L.first);
    dev_free(c, (void *)p.L.planes);
    dev_free(c, (void *)p.L.rows);
    dev_free(c, (void *)p.L.reps);
    dev_free(c, p.L.part);
    dev_free(c, p.L.mbox);
    p = ResPlan();
}

constexpr size_t kLatticeLds = 160 * 1024 - kResStaticLds;   // of a gfx950 CU's LDS

// Expected times (us) of the resident kernel: a chunk of 64 whole words on
// one SIMD; of partial words, and each of their four-site groups; the latency
// of a lone chunk; the exchange of a phase, and per 1,000 words received; a
// stage's barrier and the tail of its last chunks.  Without the four-site table
// (a bulk field, moves never accepted) a sweep takes 1 to 14% more; the chain
// takes 4% more with a field, 25% with moves never accepted.  Neither is
// charged, as the chain's estimate is low by as much: of 26 bit-packed batches
// with a field whose estimates lie within 15% of each other, one took the
// resident form where the chain is the faster (10 x 120x113x552: 41.7 against
// 37.7 us).
constexpr double kChunkUs = 0.80, kPartUs = 0.18, kGroupUs = 0.092, kLoneUs = 1.3, kExchangeUs = 0.8, kMailUs = 0.4,
                 kStageUs = 1.1;
// The fine form: a chunk of 16 words, the latency of a lone one, and what the
// form must promise against whole words where those are cut along y alone (at
// 0.97 of them, one film of 30x164x164 measured 11.2 us a sweep against 10.6;
// cut along x too, whole words fall short of their estimate: 16 x 40x120x120,
// both 11 by estimate, 15.8 us and 11.4 fine).
constexpr double kFineUs = 0.30, kFineLoneUs = 0.5, kFineGain = 0.95;
// Films of at most this many four-site groups per phase are updated by one
// lane per group when no film of the launch needs a cluster.
constexpr long kSmallGroups = (long)kSmallTasks * kResThreads;

// A film cut into px x py shares: px blocks of mirrored plane pairs (the last
// one the middle planes), py blocks of rows.
struct ShareCost {
    const islf_replica_desc &d;
    bool fine;
    int Wq, Wf, ng;
    explicit ShareCost(const islf_replica_desc &d_, bool fine_ = false) : d(d_), fine(fine_)
    {
        const int nbits = d.Lz / 2;
        Wq = (nbits + 31) / 32;
        Wf = nbits / 32;
        ng = (nbits % 32 + 3) / 4;
    }
    // block i of px: planes xa .. xa+n1-1 and n2 mirrored ones
    void planes(int px, int i, int &xa, int &n1, int &n2) const
    {
        const int H = (d.Lx + 1) / 2;
        xa = (int)((long)i * H / px);
        n1 = (int)((long)(i + 1) * H / px) - xa;
        n2 = n1;
        if (i == px - 1) {
            n1 = d.Lx - 2 * xa;
            n2 = 0;
        }
    }
    int max_planes(int px) const
    {
        int m = 0;
        for (int i = 0; i < px; ++i) {
            int xa, n1, n2;
            planes(px, i, xa, n1, n2);
            m = std::max(m, n1 + n2);
        }
        return m;
    }
    // LDS of a share of np planes (in two runs) and `rows` rows, one of px > 1 blocks
    size_t lds(int np, int px, int rows) const
    {
        const size_t lat = (size_t)(np + (px > 1 ? 4 : 2)) * (size_t)(rows + 2) * 8 * (size_t)Wq;
        // planes, columns, and the mail of all four faces
        return round_up(lat, 16) + 24 * (size_t)np + 28 * (size_t)rows * Wq + 4 * (size_t)(2 * np + (px > 1 ? 4 : 0) * rows) * Wq;
    }
    // SIMD time of a row set's chunks
    double work(long np, long rows) const
    {
        if (fine) return ceil_div(np * rows * Wf, kResFineChunk) * kFineUs + (ng ? ceil_div(np * rows, kResFineChunk) * kFineUs : 0.0);
        return ceil_div(np * rows * Wf, 64) * kChunkUs + (ng ? ceil_div(np * rows, 64) * (kPartUs + ng * kGroupUs) : 0.0);
    }
    double stage(double work_us) const
    {
        return std::max(work_us / 4.0, fine ? kFineLoneUs : Wf ? kLoneUs : 0.4 + 0.15 * ng) + kStageUs;
    }
    // a sweep of a share of np planes and `rows` rows (see ResStage)
    double sweep(long np, long rows, bool row0, bool has_x, bool has_y) const
    {
        const double mail = (has_y ? 2.0 * np * Wq : 0.0) + (has_x ? 4.0 * rows * Wq : 0.0);
        const double xch = has_x || has_y ? 2.0 * (kExchangeUs + kMailUs * mail * 1e-3) : 0.0;
        const double edge = has_y ? work(np, std::min(2l, rows)) : 0.0;
        const long r = rows - (has_y ? 2 : 0);   // beside the edge rows
        if (!row0) return 2.0 * stage(edge + (r > 0 ? work(np, r) : 0.0)) + xch;
        const double seam = work(np, 2), inner = r > 3 ? work(np, r - 3) : 0.0;
        return stage(edge + seam + inner) + stage(edge + seam) + 2.0 * stage(work(np, 1) + inner / 2.0) + xch +
               (fine && has_x ? 4.0 * kExchangeUs : 0.0);   // row 0's own mail
    }
    // rows of the shares with row 0 (Ly-1, 0, 1 at least) and the most rows of
    // the others when py >= 2; false if there are too few rows
    bool split(int px, int py, int &rows0, int &r) const
    {
        rows0 = d.Ly;
        r = 0;
        if (py == 1) return true;
        if (d.Ly < py + 2) return false;
        // row 0's two more stages cost their share as much as `extra` rows
        const double row_us = std::max(1e-3, work(max_planes(px), 64) / (2.0 * 64.0));
        const int extra = (int)(2.0 * kStageUs / row_us + 0.5);
        rows0 = std::max(3, d.Ly - (py - 1) * (int)ceil_div((long)d.Ly + extra, py));
        r = (int)ceil_div((long)d.Ly - rows0, py - 1);
        return true;
    }
    // expected sweep time in px x py shares, < 0 if they do not fit
    double time(int px, int py) const
    {
        int rows0, r;
        if (!split(px, py, rows0, r)) return -1.0;
        const int np = max_planes(px);
        if (lds(np, px, std::max(rows0, r)) > kLatticeLds) return -1.0;
        if (px == 1 && py == 1) {
            const long groups = (long)d.Lx * (d.Ly - 1) * ((d.Lz + 7) / 8);
            if (groups <= kSmallGroups) return 3.0 + 0.0005 * groups;
        }
        return std::max(sweep(np, rows0, true, px > 1, py > 1), py > 1 ? sweep(np, r, false, px > 1, true) : 0.0);
    }
};

// The useful cuts of a film into at most NW shares, by number of shares.  A cut
// into more has to be 3% faster: below that the films of 100,000 to 350,000
// sites, whose stages cost much the same at 4 shares as at 24, were cut fine
// for nothing and paid in mail (eight of them, 24 and 4 to 10 shares each: 14.4
// and 13.7 us a sweep; planning them took 0.5 and 0.35 ms).
static std::vector<ShareChoice> share_choices(const islf_replica_desc &d, bool fine, int NW)
{
    const ShareCost k(d, fine);
    std::vector<ShareChoice> all, best;
    const int H = (d.Lx + 1) / 2;
    for (int px : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16}) {
        if (px > H) break;
        int last = 0;
        for (int py = 1; px * py <= NW && py <= std::max(1, d.Ly - 2); ++py) {
            const int rows = (int)ceil_div(d.Ly, py);
            if (rows == last && py > 2) continue;   // as many rows as with one share fewer
            last = rows;
            const double t = k.time(px, py);
            if (t >= 0) all.push_back({px * py, px, py, t});
        }
    }
    std::stable_sort(all.begin(), all.end(), [](const ShareChoice &a, const ShareChoice &b) {
        return a.P != b.P ? a.P < b.P : a.us < b.us;
    });
    for (const ShareChoice &c : all)
        if (best.empty() || c.us < 0.97 * best.back().us) best.push_back(c);
    return best;
}

static uint32_t magic_of(int d) { return d >= 2 ? (uint32_t)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d) : 0u; }

static double chain_work_us(const islf_ctx *c, long long sites)
{
    return (double)sites / (c->fmt == ISLF_SPIN_BITPACK ? 2.65e6 : 1.53e6);
}

static double grouped_sweep_us(const islf_ctx *c, long long sites, int nreps)
{
    return 5.0 + 0.15 * nreps + chain_work_us(c, sites);
}

constexpr double kChainRunUs = 8.0;   // of a run of the launch chain, beside its sweeps

// A sweep of the launch chain in the context's form, measured: one chain takes 20 us a sweep in
// launches whose work does not overlap (19.5 us per launch of a 46 M-site
// bit-packed film), concurrent groups hide all but a few us of that on large
// replicas (3 x 160x480x600: 57 us bit-packed, 95 us int8) and less on many
// small ones (64 x 40x120x120: 31 us bit-packed).
static double chain_sweep_us(const islf_ctx *c, long long sites, int nreps)
{
    if (c->tuned && c->tuned_us > 0.0 && c->exec == c->tuned_exec) return c->tuned_us;
    if (c->exec != ISLF_EXEC_BATCHED || nreps == 1) return std::max(14.0, 20.0 + chain_work_us(c, sites));
    return std::max(20.0, grouped_sweep_us(c, sites, nreps));
}

// The tables of a resident plan on the host.
struct ResTablesHost {
    std::vector<ResJob> jobs;
    std::vector<int> first;
    std::vector<ResPlane> planes;
    std::vector<ResRow> rows;
    std::vector<ResRep> reps;
    size_t mbox_words = 0;
};

// The px x py shares of a film, appended to the tables; jobs go to `put`.
template <class PUT>
static void cut_film(const islf_replica_desc &d, int rep, int px, int py, int form, int &id, ResTablesHost &h, PUT put)
{
    const ShareCost k(d, form == RES_FINE);   // the split that was checked against the LDS
    const int P = px * py;
    const uint32_t Wq = (uint32_t)k.Wq;
    int rows0, rmax;
    k.split(px, py, rows0, rmax);
    std::vector<uint32_t> box(P), xface(P);   // a share's mailbox; its first x face in a slot
    size_t slot = 0;                          // words of a slot, the same for all shares of the film
    std::vector<int> R(py), y0(py);
    const int before = py > 1 ? rows0 / 2 : 0;   // rows below row 0 in its shares
    R[0] = rows0;
    y0[0] = py > 1 ? d.Ly - before : 0;
    long left = d.Ly - rows0;
    for (int j = 1, y = rows0 - before; j < py; ++j) {
        R[j] = (int)ceil_div(left, py - j);
        y0[j] = y;
        y += R[j];
        left -= R[j];
    }
    std::vector<int> plane_off(px);
    std::vector<int> np(px), ne(px), nh(px), nt(px);
    for (int i = 0; i < px; ++i) {
        int xa, n1, n2;
        k.planes(px, i, xa, n1, n2);
        np[i] = n1 + n2;
        plane_off[i] = (int)h.planes.size();
        std::vector<ResPlane> edge, mid, surf;
        for (int q = 0; q < np[i]; ++q) {
            ResPlane e{};
            auto slot = [&](int v) { return (int16_t)(v < n1 ? v + 1 : v + 3); };
            e.slot = slot(q);
            e.mirror = slot(np[i] - 1 - q);
            e.x = (int16_t)(q < n1 ? xa + q : d.Lx - xa - n2 + (q - n1));
            e.flags = (int16_t)((e.x & 1) * PL_ODD + (e.x == 0 ? PL_X0 : 0) + (e.x == d.Lx - 1 ? PL_XL : 0));
            // the outer share's inner face takes the first and the last plane, the inner share's outer face the two in the middle
            if (i > 0) e.flags = (int16_t)(e.flags | (q == 0 ? 1 * PL_SEND : 0) | (q == np[i] - 1 ? 2 * PL_SEND : 0));
            if (n2) e.flags = (int16_t)(e.flags | (q == n1 - 1 ? 4 * PL_SEND : 0) | (q == n1 ? 8 * PL_SEND : 0));
            (e.flags >= PL_SEND ? edge : (e.flags & (PL_X0 | PL_XL)) ? surf : mid).push_back(e);
        }
        ne[i] = (int)edge.size();
        nh[i] = 0;
        for (int q = 0; q < ne[i]; ++q)
            if (edge[q].flags & (PL_X0 | PL_XL)) nh[i] = q + 1;
        nt[i] = (int)surf.size();
        h.planes.insert(h.planes.end(), edge.begin(), edge.end());
        h.planes.insert(h.planes.end(), mid.begin(), mid.end());
        h.planes.insert(h.planes.end(), surf.begin(), surf.end());
    }
    for (int j = 0; j < py; ++j)
        for (int i = 0; i < px; ++i) {
            const size_t y = py > 1 ? 2 * (size_t)np[i] * Wq : 0;
            const size_t x = (size_t)((i > 0 ? 2 : 0) + (i < px - 1 ? 2 : 0)) * R[j] * Wq;
            xface[j * px + i] = (uint32_t)y;
            slot = std::max(slot, y + x);
        }
    for (uint32_t &v : box) {
        v = (uint32_t)h.mbox_words;
        if (P > 1) h.mbox_words += 2 * slot;
    }
    for (int j = 0; j < py; ++j) {
        // the block's rows by set
        const int lr0 = j == 0 ? before + 1 : 0, ls = j == 0 ? (py > 1 ? before : d.Ly) : 0;
        const int row_off = (int)h.rows.size();
        ResRows set[4] = {};
        // (chunk counts depend on the block's planes: filled in below)
        auto add = [&](int k_, const std::vector<int> &lrs) {
            set[k_].r0 = (int)h.rows.size() - row_off;
            set[k_].n = (int)lrs.size();
            set[k_].m = magic_of((int)lrs.size());
            set[k_].m_w = magic_of((int)lrs.size() * k.Wf);
            for (int lr : lrs) {
                ResRow e{};
                e.y = lr0 && lr >= lr0 ? lr - lr0 : y0[j] + lr - 1;
                e.lr = (int16_t)lr;
                e.flags = (int16_t)((e.y & 1) * RW_ODD + (lr == ls ? RW_LAST : 0) + (lr == lr0 ? RW_ROW0 : 0) +
                                    (py > 1 && lr == 1 ? RW_DOWN : 0) + (py > 1 && lr == R[j] ? RW_UP : 0));
                set[k_].seam |= (lr == ls || lr == lr0) ? 1 : 0;
                h.rows.push_back(e);
            }
        };
        std::vector<int> edge, last, inner;
        for (int lr = 1; lr <= R[j]; ++lr) {
            if (lr == lr0) continue;
            if (py > 1 && (lr == 1 || lr == R[j])) edge.push_back(lr);
            else if (lr0 && (lr == ls || lr == lr0 + 1) && form != RES_GROUPS) last.push_back(lr);
            else inner.push_back(lr);
        }
        add(RES_EDGE, edge);
        add(RES_SEAM, last);
        add(RES_INNER, inner);
        add(RES_ROW0, lr0 ? std::vector<int>(1, lr0) : std::vector<int>());
        for (int i = 0; i < px; ++i) {
            ResJob b{};
            b.rep = rep;
            b.P = P;
            b.id = id++;
            b.y0 = y0[j];
            b.R = R[j];
            b.ls = ls;
            b.lr0 = lr0;
            k.planes(px, i, b.xa, b.n1, b.n2);
            b.has = (py > 1 ? HAS_Y : 0) | (i > 0 ? HAS_OUTER : 0) | (i < px - 1 ? HAS_INNER : 0);
            b.planes = plane_off[i];
            b.rows = row_off;
            b.n_edge = ne[i];
            b.n_head = nh[i];
            b.n_tail = nt[i];
            const long per = form == RES_FINE ? kResFineChunk : 64;   // words of a chunk
            for (int q = 0; q < 4; ++q) {
                b.set[q] = set[q];
                b.set[q].whole = (int)ceil_div((long)np[i] * set[q].n * k.Wf, per);
                b.set[q].part = k.ng ? (int)ceil_div((long)np[i] * set[q].n, per) : 0;
            }
            // Stages.  Row 0's phases 2 and 3 follow phase 1 of the rows beside it and precede their next
            // phase 0; a share with row 0 does those rows first and splits the interior rows' phase 1 over
            // the two stages of row 0, which hides their latency and that of row 0's own mail.
            const bool two = px > 1;
            auto part = [&](int set_, int phase, int c0 = 0, int c1 = -1) {
                return ResPart{(int16_t)set_, (int16_t)phase, c0, c1 < 0 ? b.set[set_].whole + b.set[set_].part : c1};
            };
            auto stage = [&](std::vector<ResPart> v, int mail, int mail_row0) {
                ResStage &t = b.stage[b.stages++];
                for (int q = 0; q < 3; ++q) t.part[q] = q < (int)v.size() ? v[q] : ResPart{RES_INNER, 0, 0, 0};
                t.mail = P > 1 ? mail : -1;
                t.mail_row0 = two ? mail_row0 : -1;
            };
            const int inner_n = b.set[RES_INNER].whole + b.set[RES_INNER].part;
            stage({part(RES_EDGE, 0), part(RES_SEAM, 0), part(RES_INNER, 0)}, 0, lr0 ? 3 : -1);
            if (!lr0) {
                stage({part(RES_EDGE, 1), part(RES_INNER, 1)}, 1, -1);
            } else {
                stage({part(RES_EDGE, 1), part(RES_SEAM, 1)}, -1, -1);
                stage({part(RES_ROW0, 2), part(RES_INNER, 1, 0, inner_n / 2)}, -1, 2);
                stage({part(RES_ROW0, 3), part(RES_INNER, 1, inner_n / 2, inner_n)}, 1, -1);
            }
            b.Wf = k.Wf;
            b.ng = k.ng;
            b.m_c = magic_of((d.Lz + 7) / 8);
            b.m_q = magic_of(k.Wq);
            b.m_f = magic_of(R[j] * k.Wq);
            b.in = box[j * px + i];
            b.slot = (uint32_t)slot;
            if (py > 1) {
                b.out_y[0] = box[(j + py - 1) % py * px + i] + (uint32_t)np[i] * Wq;   // the lower share's upper face
                b.out_y[1] = box[(j + 1) % py * px + i];                               // the upper share's lower face
            }
            // the outer share's inner face (after its outer one, if any); the inner share's outer face
            if (i > 0) b.out_x[0] = box[j * px + i - 1] + xface[j * px + i - 1] + (i > 1 ? 2u : 0u) * (uint32_t)R[j] * Wq;
            if (i < px - 1) b.out_x[1] = box[j * px + i + 1] + xface[j * px + i + 1];
            put(b, k.lds(np[i], px, R[j]));
        }
    }
}

// Shares of the listed replicas for one launch of at most num_cu workgroups
// (one per CU: the kernel's registers allow no second one).  Replicas that
// need several workgroups get a share each on workgroups of their own, the
// single-workgroup ones then go, largest first, to the workgroup with the
// least work (they wait for nobody, so a workgroup may hold several).  The
// target time per sweep that sets the shares is scanned for the shortest
// launch.  Returns false if the replicas do not fit.
static bool plan_resident(islf_ctx *c, const std::vector<int> &reps, ResPlan &p, ResTablesHost &h)
{
    const int n = (int)reps.size(), NW = c->num_cu;
    // replicas of one shape share their choices
    if (c->choices.size() > kMaxShapes) c->choices.clear();
    std::vector<const std::vector<ShareChoice> *> shape(n);
    std::vector<const ShareChoice *> pick(n), best_pick;
    double best = 1e300;
    p.form = RES_WORDS;
    auto pack = [&](std::vector<int> *where) -> double {
        // cluster workgroups first, then singles by LPT; returns the longest workgroup
        std::vector<std::pair<double, int>> heap;   // (-load, workgroup)
        double longest = 0.0;
        int w = 0;
        std::vector<int> single;
        for (int i = 0; i < n; ++i) {
            if (pick[i]->P == 1) {
                single.push_back(i);
                continue;
            }
            for (int k = 0; k < pick[i]->P; ++k) heap.push_back({-pick[i]->us, w++});
            longest = std::max(longest, pick[i]->us);
        }
        for (; w < NW; ++w) heap.push_back({0.0, w});
        std::make_heap(heap.begin(), heap.end());
        std::stable_sort(single.begin(), single.end(), [&](int a, int b) { return pick[a]->us > pick[b]->us; });
        for (int i : single) {
            std::pop_heap(heap.begin(), heap.end());
            heap.back().first -= pick[i]->us;
            longest = std::max(longest, -heap.back().first);
            if (where) (*where)[i] = heap.back().second;
            std::push_heap(heap.begin(), heap.end());
        }
        return longest;
    };
    for (int form : {RES_WORDS, RES_FINE}) {
        double total = 0.0;
        for (int i = 0; i < n; ++i) {
            const islf_replica_desc &d = c->reps[reps[i]].desc;
            if (d.Lx > 32000 || d.Ly > 32000) return false;   // 16-bit table entries
            const std::array<int, 4> key = {d.Lx, d.Ly, d.Lz, form};
            auto it = c->choices.find(key);
            if (it == c->choices.end()) it = c->choices.emplace(key, share_choices(d, form == RES_FINE, NW)).first;
            if (it->second.empty()) return false;
            shape[i] = &it->second;
            const ShareChoice &f = shape[i]->front();
            total += f.P * f.us;
        }
        const double t0 = std::max(2.0, 0.7 * total / NW);
        for (int step = 0; step < 64; ++step) {
            const double T = t0 * pow(1.04, step);
            long used = 0;
            for (int i = 0; i < n; ++i) {
                // the fewest shares within T, else the fastest cut
                const std::vector<ShareChoice> &v = *shape[i];
                size_t q = 0;
                while (q + 1 < v.size() && v[q].us > T) ++q;
                pick[i] = &v[q];
                if (v[q].P > 1) used += v[q].P;
            }
            if (used > NW) continue;
            const double m = pack(nullptr);
            const bool cut_x = form != p.form && std::any_of(best_pick.begin(), best_pick.end(),
                                                             [](const ShareChoice *q) { return q->px > 1; });
            if (m < (form == p.form || cut_x ? 1.0 : kFineGain) * best) {
                best = m;
                best_pick = pick;
                p.form = form;
            }
            if (m < T) break;
        }
    }
    if (best_pick.empty()) return false;
    pick = best_pick;
    std::vector<int> where(n, -1);
    p.sweep_us = pack(&where);
    bool groups = true;
    for (int i = 0; i < n; ++i) {
        const islf_replica_desc &d = c->reps[reps[i]].desc;
        const long row = (long)d.Lx * ((d.Lz + 7) / 8);   // groups of a row
        groups = groups && pick[i]->P == 1 && row <= kResThreads && row * (d.Ly - 1) <= kSmallGroups;
    }
    if (groups) p.form = RES_GROUPS;
    std::vector<std::vector<ResJob>> wg(NW);
    p.L.members = 0;
    p.lds = 0;
    int id = 0;
    for (int i = 0; i < n; ++i) {
        h.reps.push_back(ResRep{reps[i], id, pick[i]->P, 0});
        cut_film(c->reps[reps[i]].desc, reps[i], pick[i]->px, pick[i]->py, p.form, id, h,
                 [&](const ResJob &j, size_t lds) {
                     wg[j.P > 1 ? p.L.members++ : where[i]].push_back(j);
                     p.lds = std::max(p.lds, lds);
                 });
        if (h.mbox_words >= (1ull << 29)) return false;   // 32-bit byte offsets
    }
    if (p.lds > kLatticeLds) return false;   // (a launch that asks for more is refused)
    // a workgroup's cluster share comes before its single films
    h.first.assign(1, 0);
    for (int w = 0; w < NW; ++w) {
        if (wg[w].empty()) continue;
        std::stable_sort(wg[w].begin(), wg[w].end(), [](const ResJob &a, const ResJob &b) { return (a.P > 1) > (b.P > 1); });
        h.jobs.insert(h.jobs.end(), wg[w].begin(), wg[w].end());
        h.first.push_back((int)h.jobs.size());
    }
    p.L.grid = (int)h.first.size() - 1;
    p.L.njobs = (int)h.jobs.size();
    p.L.nreps = n;
    return true;
}

static size_t resident_bytes(const ResPlan &p)
{
    return p.jobs_b + p.first_b + p.planes_b + p.rows_b + p.reps_b + p.part_b + p.mbox_b;
}

// Puts a host table into a device buffer of the plan, grown if needed.
template <class T>
static bool put_table(islf_ctx *c, const T *&ptr, size_t &have, const std::vector<T> &v, hipError_t &e)
{
    const size_t bytes = sizeof(T) * std::max<size_t>(1, v.size());
    if (bytes > have) {
        dev_free(c, (void *)ptr);
        have = 0;
        ptr = (const T *)dev_alloc(c, bytes);
        if (!ptr) return false;
        have = bytes;
    }
    if (!v.empty() && e == hipSuccess)
        e = hipMemcpyAsync((void *)ptr, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice, c->stream);
    return true;
}

// Builds the resident plan of some replicas (synchronises).  A plan that
// cannot be had (too large, no memory) is valid but not usable.
static islf_status build_resident(islf_ctx *c, ResPlan &p, const std::vector<int> &reps)
{
    p.valid = true;
    p.usable = p.put_off = false;
    ResTablesHost h;
    if (reps.empty() || !plan_resident(c, reps, p, h)) return ISLF_OK;
    p.sites = 0;
    p.nreps = (int)reps.size();
    size_t bytes = 0;
    for (int r : reps) {
        const islf_replica_desc &d = c->reps[r].desc;
        p.sites += (long long)d.Lx * d.Ly * d.Lz;
        bytes += spin_bytes(&d, c->fmt);
    }
    p.fixed_us = 16.0 + 2.0 * (double)bytes / 2.0e6;
    p.put_off = p.sweep_us >= chain_sweep_us(c, p.sites, p.nreps);
    if (p.put_off) return ISLF_OK;
    // per-sweep sums: 8 MiB at most, had here for the longest launch, so that runs allocate nothing
    p.max_sweeps = (uint32_t)std::max<size_t>(1, std::min<size_t>(kResMaxSweeps, (8u << 20) / (16 * (size_t)p.L.njobs)));
    // a context's plans of one kind hold at most kPlanBytes (no part of the replicas' footprint)
    size_t held = sizeof(ResJob) * h.jobs.size() + sizeof(int) * h.first.size() + sizeof(ResPlane) * h.planes.size() +
                  sizeof(ResRow) * h.rows.size() + sizeof(ResRep) * h.reps.size() + 8 * h.mbox_words +
                  sizeof(int4) * p.max_sweeps * (size_t)p.L.njobs;
    if (&p != &c->resident)
        for (const ResPlan &o : c->resident_plain)
            if (&o != &p) held += resident_bytes(o);
    if (held > kPlanBytes) return ISLF_OK;
    hipError_t e = hipSuccess;
    if (!put_table(c, p.L.jobs, p.jobs_b, h.jobs, e) || !put_table(c, p.L.first, p.first_b, h.first, e) ||
        !put_table(c, p.L.planes, p.planes_b, h.planes, e) || !put_table(c, p.L.rows, p.rows_b, h.rows, e) ||
        !put_table(c, p.L.reps, p.reps_b, h.reps, e)) {
        (void)hipStreamSynchronize(c->stream);   // no copy may outlive its source
        return ISLF_OK;
    }
    auto grow = [&](auto *&ptr, size_t &have, size_t bytes) {
        if (bytes <= have) return;
        dev_free(c, ptr);
        ptr = (std::remove_reference_t<decltype(ptr)>)dev_alloc(c, bytes);
        have = ptr ? bytes : 0;
    };
    grow(p.L.mbox, p.mbox_b, 8 * std::max<size_t>(1, h.mbox_words));
    grow(p.L.part, p.part_b, sizeof(int4) * p.max_sweeps * (size_t)p.L.njobs);
    // no mailbox word may carry an epoch still to come
    if (e == hipSuccess && p.L.mbox) e = launch_zero(p.L.mbox, (long)h.mbox_words, c->stream);
    if (e == hipSuccess) e = resident_lds_limit(c->fmt, kLatticeLds);
    const hipError_t es = hipStreamSynchronize(c->stream);
    HIP_TRY(e);
    HIP_TRY(es);
    if (!p.L.mbox || !p.L.part) return ISLF_OK;
    p.usable = true;
    return ISLF_OK;
}

// Whether the caller has chosen a launch configuration of the chain or of the persistent kernel.
static bool config_chosen(const islf_ctx *c)
{
    return !c->tuned && (c->grid_override || c->groups_req || c->taper_override >= 0.0 || c->team_mode >= 0);
}

// Whether a run of n sweeps takes the resident form (its plans are then
// built).  A launch configuration chosen by the caller (grid, groups, taper,
// barriers, a tile) asks for the launch chain or the persistent kernel; one
// that islf_autotune found is only the chain's own.
static islf_status resident_applies(islf_ctx *c, uint32_t n, bool *use)
{
    *use = false;
    islf_status st = sync_tables(c);
    if (st != ISLF_OK) return st;
    if (n == 0 || c->live.empty()) return ISLF_OK;
    if (c->chain_only || config_chosen(c)) return ISLF_OK;
    for (int r : c->live)
        if (c->reps[r].tile_set) return ISLF_OK;
    double res = 0.0, chain = 0.0;
    auto add = [&](ResPlan &p, const std::vector<int> &reps) -> islf_status {
        // (the chain's time depends on the execution form, which may have changed since the plan was built)
        if (!p.valid || (p.put_off && p.sweep_us < chain_sweep_us(c, p.sites, p.nreps))) {
            islf_status s = build_resident(c, p, reps);
            if (s != ISLF_OK) return s;
        }
        res += p.usable ? p.fixed_us * (double)((n + p.max_sweeps - 1) / p.max_sweeps) + n * p.sweep_us : 1e300;
        chain += kChainRunUs + n * chain_sweep_us(c, p.sites, p.nreps);
        return ISLF_OK;
    };
    if (c->exec == ISLF_EXEC_PLAIN) {
        if (c->resident_plain.size() < c->reps.size()) c->resident_plain.resize(c->reps.size());
        for (int r : c->live) {
            st = add(c->resident_plain[r], std::vector<int>(1, r));
            if (st != ISLF_OK) return st;
        }
    } else {
        st = add(c->resident, c->live);
        if (st != ISLF_OK) return st;
    }
    *use = res < chain;
    return ISLF_OK;
}

// Enqueues n sweeps in the resident form (plans built, no checks, no sync).
static hipError_t enqueue_resident(islf_ctx *c, uint32_t n)
{
    auto run = [&](const ResPlan &p) -> hipError_t {
        ResLaunch L = p.L;
        L.descs = c->d_desc;
        L.st = c->d_state;
        L.rs = c->d_rsy;
        L.sync = c->d_sync;
        L.host = c->h_res;
        L.check_error = c->exec == ISLF_EXEC_PERSISTENT;
        hipError_t e = hipSuccess;
        for (uint32_t done = 0; done < n && e == hipSuccess; done += L.n) {
            L.n = std::min(n - done, p.max_sweeps);
            e = launch_resident(c->fmt, p.form, L, p.lds, c->stream);
        }
        return e;
    };
    if (c->exec != ISLF_EXEC_PLAIN) return run(c->resident);
    hipError_t e = hipSuccess;
    for (size_t i = 0; i < c->live.size() && e == hipSuccess; ++i) e = run(c->resident_plain[c->live[i]]);
    return e;
}

// Contexts that sweep at the same time.  The workgroups of a cluster launch
// wait for each other, and each needs a whole CU: two such launches dispatched
// into each other would both give up, and a launch chain on other streams can
// keep every CU partly busy for as long as it has launches queued.  So, for the
// contexts of a process on one device (of different streams):
//  - Cluster launches that do not all find a CU each beside those that others
//    have in flight are ordered behind them.
//  - A run of the chain is ordered behind the clusters that others have in flight.
//  - While another context has a chain in flight, a run joins it: takes the
//    chain too.  Runs that joined are no reason to join (contexts would keep
//    each other on the chain): clusters are ordered behind them.
//  - Where chains side by side are the faster form (see prefers_chain),
//    contexts that met keep to the chain for kApartRuns runs; so does a context
//    with a launch that the census called off (work of another process or of
//    the caller on the CUs).
// Measured, two contexts on threads of their own, 250 sweeps each, ms for both,
// on the chain and so: 64 x 40x120x120 bit-packed 15.8 and 10.6 (in turn), 8 x
// 28x94x94 12.3 and 2.5 (side by side), 3 x 160x480x600 int8 46 and 31 (in
// turn), one 88x504x504 int8 12.0 and 8.1 (in turn), bit-packed 7.2 and 7.2 (on
// the chain; in turn 8.2, and 16 against 14.0 for four contexts).
// What is in flight is read from the counts that closing kernels write to
// pinned memory (an event query from another thread would break a stream
// capture in global mode there).  Runs that a caller captures on the context's
// stream, and replays of them, are not seen: for them the census stands.
struct Turns {
    std::mutex m;
    std::vector<islf_ctx *> all;
};
constexpr int kMaxDevices = 64, kApartRuns = 256;

static Turns &turns(const islf_ctx *c)
{
    static Turns *t = new Turns[kMaxDevices];   // (outlives contexts closed at exit)
    return t[c->device % kMaxDevices];
}

static bool ahead(const islf_ctx *o, uint32_t until)
{
    return (int32_t)(until - (uint32_t)__atomic_load_n(o->h_res + HOST_ENDED, __ATOMIC_RELAXED)) > 0;
}

static bool chain_in_flight(const islf_ctx *o) { return o->unmarked || ahead(o, o->chain_until); }

static int members_in_flight(islf_ctx *o)
{
    if (!ahead(o, o->cluster_until)) o->members = 0;
    return o->members;
}

// After the host has waited for the context's stream.
static void landed(islf_ctx *c)
{
    std::lock_guard<std::mutex> lock(turns(c).m);
    c->issued = (uint32_t)__atomic_load_n(c->h_res + HOST_ENDED, __ATOMIC_RELAXED);
    c->cluster_until = c->chain_until = c->joined_until = c->issued;
    c->unmarked = false;
    c->members = 0;
}

static bool being_captured(const islf_ctx *c)
{
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    return c->stream && hipStreamIsCapturing(c->stream, &s) == hipSuccess && s != hipStreamCaptureStatusNone;
}

// Puts what c enqueues next behind what o has in flight (lock held).  The event
// is recorded here, on o's stream, and not by o behind each of its runs, which
// cost a run 3 us (five of 10 sweeps of a 184x504x504 film: 1,485 instead of
// 1,465 us).  While o's caller captures a graph of its own on that stream no event
// can be recorded there, and c waits here.  (islf_graph_capture holds the lock.)
static hipError_t order_behind(islf_ctx *c, islf_ctx *o)
{
    // (contexts share no data: the event orders launches and needs no fence)
    hipError_t e = hipSuccess;
    if (!o->turn) e = hipEventCreateWithFlags(&o->turn, hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return e;
    if (!being_captured(o) && hipEventRecord(o->turn, o->stream) == hipSuccess && !being_captured(o))
        return hipStreamWaitEvent(c->stream, o->turn, 0);
    (void)hipGetLastError();
    const auto give_up = std::chrono::steady_clock::now() + std::chrono::seconds(60);
    while ((members_in_flight(o) || ahead(o, o->joined_until)) && std::chrono::steady_clock::now() < give_up)
        std::this_thread::yield();
    return hipSuccess;
}

enum Turn { TURN_GO, TURN_CHAIN, TURN_JOIN };

// What a run with clusters of `members` workgroups does now (lock held): goes,
// put behind those of others where need be, or is a chain, or joins one.
static Turn take_turn(islf_ctx *c, int members, bool chain_if_met, hipError_t *e)
{
    const uint32_t aborts = (uint32_t)__atomic_load_n(c->h_res + HOST_ABORTS, __ATOMIC_RELAXED);
    if (aborts != c->aborts_seen) c->apart = kApartRuns;
    c->aborts_seen = aborts;
    bool chain = false;
    int sum = members;
    std::vector<islf_ctx *> clusters, joined;
    for (islf_ctx *o : turns(c).all) {
        if (o == c || o->stream == c->stream) continue;
        chain = chain || chain_in_flight(o);
        sum += members_in_flight(o);
        if (o->members) clusters.push_back(o);
        if (ahead(o, o->joined_until)) joined.push_back(o);
    }
    const bool full = sum > c->num_cu;
    if (chain_if_met && (full || chain || !joined.empty())) {
        c->apart = kApartRuns;
        for (islf_ctx *o : clusters)
            if (o->chain_if_met) o->apart = kApartRuns;
    }
    c->chain_if_met = chain_if_met;
    if (c->apart > 0) {
        --c->apart;
        return TURN_CHAIN;
    }
    if (chain) return TURN_JOIN;
    if (!full) clusters.clear();
    clusters.insert(clusters.end(), joined.begin(), joined.end());
    for (islf_ctx *o : clusters)
        if (*e == hipSuccess) *e = order_behind(c, o);
    return TURN_GO;
}

// Puts a run of the chain behind the clusters that others have in flight and
// counts it as in flight (lock held); end_chain marks its end where somebody
// may look.
static hipError_t start_chain(islf_ctx *c, bool joins, bool *mark)
{
    hipError_t e = hipSuccess;
    for (islf_ctx *o : turns(c).all)
        if (e == hipSuccess && o != c && o->stream != c->stream && members_in_flight(o)) e = order_behind(c, o);
    *mark = turns(c).all.size() > 1;
    if (*mark) (joins ? c->joined_until : c->chain_until) = ++c->issued;
    c->unmarked = !*mark;   // (a mark ends what came before it, too)
    c->chain_runs += 1;
    return e;
}

static hipError_t end_chain(islf_ctx *c, bool mark)
{
    return mark ? launch_mark(c->d_rsy, c->h_res, c->stream) : hipSuccess;
}

// Acts on the error word, fetched to h_res.  A raised word means a launch gave
// up at a grid barrier (persistent kernel) or waiting for its neighbours' edges
// (resident kernel, in any form) and left its sweeps half done, so
// every live replica is marked failed (its calls return ESTATE until
// islf_set_spins restarts it or it is retired); the word is then cleared so
// that later launches can run.  With rep >= 0, that replica's chain has to be
// intact too.
static islf_status take_error(islf_ctx *c, int rep)
{
    if (c->h_res[0]) {
        for (int r : c->live) c->reps[r].failed = true;
        c->graph_valid = false;
        HIP_TRY(launch_zero((unsigned long long *)&c->d_sync->error, 16, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        return fail(ISLF_EDEVICE, "a launch whose workgroups wait for each other gave up (a grid barrier of the "
                                  "persistent kernel or an exchange of the resident one: not all were resident at "
                                  "once, or the wait was cut short); every live replica is marked failed");
    }
    if (rep >= 0 && c->reps[rep].failed)
        return fail(ISLF_ESTATE, "replica %d was cut short by a failed launch (restart it with "
                                 "islf_set_spins or retire it)", rep);
    return ISLF_OK;
}

// The error word, and with it n 64-bit words of the ring of `size` at `ring`
// from word `first` on (n <= kResultWords; to h_res + 8), by one kernel and one
// wait: each copy from device memory to pageable memory took 15 us, and a
// second wait came with the error word (one record: 41 us, 12 us so).
static islf_status fetch(islf_ctx *c, int rep, const void *ring = nullptr, long first = 0, long n = 0, long size = 1)
{
    HIP_TRY(launch_fetch(&c->d_sync->error.v, ring, first, n, size, c->h_res, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    landed(c);
    return take_error(c, rep);
}

static islf_status check_device_error(islf_ctx *c) { return fetch(c, -1); }

// A live replica whose chain is intact: checks the device error word, then
// the replica's failed mark.
static islf_status check_intact(islf_ctx *c, int rep) { return fetch(c, rep); }

// Rows times 16-site columns: what the kernels over all spins of a replica are sized by.
static long host_columns(const islf_replica_desc &d)
{
    return (long)d.Lx * d.Ly * ((d.Lz + 15) / 16);
}

// Spins of slot i by its init mode, and their observables (its descriptor is on the device).
static hipError_t start_replica(islf_ctx *c, int i)
{
    Replica &R = c->reps[i];
    const long n = host_columns(R.desc);
    const int mode = R.desc.init == ISLF_INIT_HOST ? ISLF_INIT_UP : R.desc.init;
    R.t_host = 0;
    const hipError_t e = launch_init(c->fmt, c->d_desc, c->d_state, i, mode, n, c->stream);
    return e != hipSuccess ? e : launch_recompute(c->fmt, c->d_desc, c->d_state, i, n, nullptr, c->stream);
}

// A slot with memory and tables for a replica; start_replica sets its spins.
static islf_status add_replica(islf_ctx *c, const islf_replica_desc *desc, int *slot_out)
{
    islf_status st = validate(desc);
    if (st != ISLF_OK) return st;
    int slot = -1;
    for (int i = 0; i < (int)c->reps.size(); ++i)
        if (!c->reps[i].live) {
            slot = i;
            break;
        }
    // no slot without a place in the device tables: they are uploaded whole
    st = ensure_slots(c, slot < 0 ? (int)c->reps.size() + 1 : (int)c->reps.size());
    if (st != ISLF_OK) return st;
    if (slot < 0) {
        slot = (int)c->reps.size();
        c->reps.emplace_back();
    }
    Replica &R = c->reps[slot];
    R.desc = *desc;
    const size_t bytes = replica_bytes(desc, c->fmt, c->cap);
    if (R.mem && R.mem_bytes < bytes) {
        dev_free(c, R.mem);
        R.mem = nullptr;
    }
    if (!R.mem) {
        R.mem = dev_alloc(c, bytes);
        if (!R.mem) return fail(ISLF_ENOMEM, "cannot allocate %zu device bytes for a replica", bytes);
        R.mem_bytes = bytes;
    }
    R.tile = default_tile(desc, c->fmt);
    R.tile_set = false;
    fill_desc(R, c->fmt, c->cap);
    build_work(R, slot, c->fmt);
    R.live = true;
    c->dirty = true;
    *slot_out = slot;
    return ISLF_OK;
}

static void destroy_graphs(islf_ctx *c)
{
    for (hipGraphExec_t ex : c->graph_execs) (void)hipGraphExecDestroy(ex);
    for (hipGraph_t g : c->graphs) (void)hipGraphDestroy(g);
    c->graph_execs.clear();
    c->graphs.clear();
    c->graph_valid = false;
}

static void destroy_ctx(islf_ctx *c)
{
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    {
        std::lock_guard<std::mutex> lock(turns(c).m);
        std::vector<islf_ctx *> &all = turns(c).all;
        all.erase(std::remove(all.begin(), all.end(), c), all.end());
    }
    if (c->turn) (void)hipEventDestroy(c->turn);
    destroy_graphs(c);
    for (auto &R : c->reps) dev_free(c, R.mem);
    dev_free(c, c->d_desc);
    dev_free(c, c->d_state);
    dev_free(c, c->d_sync);
    dev_free(c, c->d_rsy);
    free_resident(c, c->resident);
    for (ResPlan &p : c->resident_plain) free_resident(c, p);
    dev_free(c, c->d_teams);
    dev_free(c, c->d_rsync);
    dev_free(c, c->d_scratch);
    if (c->h_res) (void)hipHostFree(c->h_res);
    if (c->h_win) (void)hipHostFree(c->h_win);
    for (hipEvent_t ev : c->win_event)
        if (ev) (void)hipEventDestroy(ev);
    dev_free(c, c->d_live);
    free_plan(c, c->batched);
    free_plan(c, c->persistent);
    for (Plan &p : c->plain) free_plan(c, p);
    for (Plan &p : c->group_plan) free_plan(c, p);
    dev_free(c, c->d_group_live);
    for (hipStream_t sst : c->side_stream) (void)hipStreamDestroy(sst);
    for (hipEvent_t ev : c->side_event) (void)hipEventDestroy(ev);
    delete c;
}

// Workgroups of a 256-thread kernel that can be resident on one CU at once,
// the smaller of the runtime's occupancy answer and a count from the
// kernel's own resources: a workgroup is four wave64s, one per SIMD, so a
// SIMD's 512 VGPRs per lane (allocated in granules of 8) bound the
// workgroups per CU, and so do the CU's thread slots and LDS.
static int coresident_per_cu(const void *kernel, const hipDeviceProp_t &prop)
{
    int rt = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&rt, kernel, kBlock, 0) != hipSuccess || rt < 1) rt = 1;
    hipFuncAttributes a;
    if (hipFuncGetAttributes(&a, kernel) != hipSuccess) return rt;
    int per_cu = rt;
    const int vgprs = std::max(1, (a.numRegs + 7) / 8 * 8);
    per_cu = std::min(per_cu, 512 / vgprs);
    if (prop.maxThreadsPerMultiProcessor > 0) per_cu = std::min(per_cu, prop.maxThreadsPerMultiProcessor / kBlock);
    if (a.sharedSizeBytes > 0 && prop.maxSharedMemoryPerMultiProcessor > 0)
        per_cu = std::min(per_cu, (int)(prop.maxSharedMemoryPerMultiProcessor / a.sharedSizeBytes));
    return std::max(1, per_cu);
}

// ---------------------------------------------------------------------------
// public API
// ---------------------------------------------------------------------------
extern "C" islf_status islf_create_with_allocator(const islf_replica_desc *reps, int32_t n_reps,
                                                  int32_t spin_format, uint32_t obs_capacity,
                                                  void *hip_stream, islf_alloc_fn alloc,
                                                  islf_free_fn free_fn, void *user, islf_ctx **out)
{
    if (!out) return fail(ISLF_EINVAL, "NULL output pointer");
    *out = nullptr;
    if (!reps || n_reps < 1) return fail(ISLF_EINVAL, "need at least one replica");
    if (spin_format != ISLF_SPIN_INT8 && spin_format != ISLF_SPIN_BITPACK)
        return fail(ISLF_EINVAL, "invalid spin format %d", spin_format);
    if (obs_capacity < 1) return fail(ISLF_EINVAL, "obs_capacity must be >= 1");
    if ((alloc == nullptr) != (free_fn == nullptr)) return fail(ISLF_EINVAL, "give both alloc and free or neither");
    for (int i = 0; i < n_reps; ++i) {
        islf_status st = validate(&reps[i]);
        if (st != ISLF_OK) return st;
    }
    islf_ctx *c = new islf_ctx();
    c->fmt = spin_format;
    c->cap = obs_capacity;
    c->stream = (hipStream_t)hip_stream;
    c->alloc = alloc;
    c->free_fn = free_fn;
    c->user = user;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        delete c;
        return fail(ISLF_EDEVICE, "no HIP device");
    }
    c->device = dev;
    c->num_cu = prop.multiProcessorCount;
    int per_cu_sweep = 0;
    if (sweep_blocks_per_cu(spin_format, &per_cu_sweep) != hipSuccess || per_cu_sweep < 1) per_cu_sweep = 1;
    // two workgroups per resident slot: measured faster than one (a single
    // round leaves slots idle while the last workgroups finish)
    c->resident_slots = c->num_cu * per_cu_sweep;
    c->sweep_slots = 2 * c->resident_slots;
    // both forms of the persistent kernel (grid and team barriers) launch on
    // the same grid: the bound is the smaller of the two
    const int per_cu = std::min(coresident_per_cu(persistent_kernel(spin_format), prop),
                                coresident_per_cu(persistent_teams_kernel(spin_format), prop));
    c->persistent_bound = std::min(c->num_cu * per_cu, kBarrierGroup * kMaxGroups);
    // one slot per CU stays free by default: at the full occupancy the
    // runtime reported for an earlier build of the int8 kernel (7 workgroups
    // per CU at 72 VGPRs) a cooperative launch was accepted but its workgroups
    // were not all resident at once, and the grid barrier's bounded wait
    // expired
    const int per_cu_p = per_cu > 1 ? per_cu - 1 : 1;
    c->persistent_grid = std::min(c->num_cu * per_cu_p, c->persistent_bound);
    if (noalloc_scratch(&c->noalloc_scratch) != hipSuccess) {
        delete c;
        return fail(ISLF_EDEVICE, "cannot look up the means scratch array on device %d", dev);
    }
    c->d_sync = (GridSync *)dev_alloc(c, sizeof(GridSync));
    c->d_scratch = (unsigned long long *)dev_alloc(c, 64 * sizeof(unsigned long long));
    c->d_rsy = (ResSync *)dev_alloc(c, sizeof(ResSync));
    if (hipHostMalloc((void **)&c->h_res, 8 * (8 + kResultWords), hipHostMallocCoherent) != hipSuccess) c->h_res = nullptr;
    if (c->h_res) memset(c->h_res, 0, 8 * 8);
    if (!c->d_sync || !c->d_scratch || !c->d_rsy || !c->h_res) {
        destroy_ctx(c);
        return fail(ISLF_ENOMEM, "cannot allocate context buffers");
    }
    if (launch_zero((unsigned long long *)c->d_sync, sizeof(GridSync) / 8, c->stream) != hipSuccess ||
        launch_zero((unsigned long long *)c->d_rsy, sizeof(ResSync) / 8, c->stream) != hipSuccess) {
        destroy_ctx(c);
        return fail(ISLF_EDEVICE, "cannot clear sync words");
    }
    islf_status st = ensure_slots(c, n_reps);
    for (int i = 0; i < n_reps && st == ISLF_OK; ++i) {
        int slot;
        st = add_replica(c, &reps[i], &slot);
    }
    if (st == ISLF_OK) st = sync_tables(c);
    hipError_t e = hipSuccess;
    for (int i = 0; i < n_reps && st == ISLF_OK && e == hipSuccess; ++i) e = start_replica(c, i);
    if (st == ISLF_OK && e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) st = fail(ISLF_EDEVICE, "replica init failed: %s", hipGetErrorString(e));
    if (st != ISLF_OK) {
        std::string keep = g_err;
        destroy_ctx(c);
        g_err = keep;
        return st;
    }
    {
        std::lock_guard<std::mutex> lock(turns(c).m);
        turns(c).all.push_back(c);
    }
    *out = c;
    return ISLF_OK;
}

extern "C" islf_status islf_create(const islf_replica_desc *reps, int32_t n_reps, int32_t spin_format,
                                   uint32_t obs_capacity, void *hip_stream, islf_ctx **out)
{
    return islf_create_with_allocator(reps, n_reps, spin_format, obs_capacity, hip_stream, nullptr, nullptr,
                                      nullptr, out);
}

extern "C" islf_status islf_destroy(islf_ctx *ctx)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    destroy_ctx(ctx);
    return ISLF_OK;
}

extern "C" islf_status islf_num_replicas(const islf_ctx *ctx, int32_t *n)
{
    if (!ctx || !n) return fail(ISLF_EINVAL, "NULL argument");
    *n = (int32_t)ctx->reps.size();
    return ISLF_OK;
}

static islf_status check_rep(const islf_ctx *ctx, int32_t rep)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (rep < 0 || rep >= (int32_t)ctx->reps.size() || !ctx->reps[rep].live)
        return fail(ISLF_ERANGE, "replica %d is not live", rep);
    return ISLF_OK;
}

extern "C" islf_status islf_get_desc(const islf_ctx *ctx, int32_t rep, islf_replica_desc *out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!out) return fail(ISLF_EINVAL, "NULL output");
    *out = ctx->reps[rep].desc;
    return ISLF_OK;
}

// Threads that copy or check host spins with the calling one, for the length of
// a call.  One thread copies 16 to 27 GB/s here, the link carries 57: 22 M sites
// set in 1050 and read in 1270 us by pageable copies, 890 and 740 us so.
class Crew {
public:
    explicit Crew(size_t bytes)
    {
        const int most = (int)std::min(4u, std::thread::hardware_concurrency() / 2);
        if (bytes < 2 * kWindow) return;   // starting threads costs as much as they would save
        try {
            for (int i = 1; i < most; ++i) threads_.emplace_back([this, i] { work(i); });
        } catch (...) {
            // those that started do it
        }
    }
    ~Crew()
    {
        stop_ = true;
        turn_.fetch_add(1, std::memory_order_release);
        for (std::thread &t : threads_) t.join();
    }
    Crew(const Crew &) = delete;
    Crew &operator=(const Crew &) = delete;
    // copies n bytes (dst may be null), or with check_ looks for bytes that are
    // neither +1 nor -1; true if there are any
    bool run(int8_t *dst, const int8_t *src, size_t n, bool check)
    {
        dst_ = dst;
        src_ = src;
        n_ = n;
        check_ = check;
        parts_ = (int)threads_.size() + 1;
        bad_.store(0, std::memory_order_relaxed);
        left_.store((int)threads_.size(), std::memory_order_relaxed);
        turn_.fetch_add(1, std::memory_order_release);
        part(0);
        while (left_.load(std::memory_order_acquire)) std::this_thread::yield();
        return bad_.load(std::memory_order_relaxed) != 0;
    }

private:
    void part(int i)
    {
        const size_t step = round_up((n_ + parts_ - 1) / parts_, 4096), a = std::min(n_, i * step);
        const size_t m = std::min(n_ - a, step);
        if (!check_) {
            memcpy(dst_ + a, src_ + a, m);
            return;
        }
        // +1 and -1 are the bytes 0x01 and 0xFF: (byte + 1) & 0xFD is 0 exactly
        // for them (a branch-free pass the compiler vectorises)
        uint8_t bad = 0;
        const uint8_t *p = (const uint8_t *)src_ + a;
        for (size_t k = 0; k < m; ++k) bad |= (uint8_t)(p[k] + 1u) & 0xFDu;
        if (bad) bad_.store(1, std::memory_order_relaxed);
    }
    void work(int i)
    {
        for (unsigned seen = 0;;) {
            for (int spins = 0; turn_.load(std::memory_order_acquire) == seen;)
                if (++spins > 256) std::this_thread::yield();
            ++seen;
            if (stop_) return;
            part(i);
            left_.fetch_sub(1, std::memory_order_release);
        }
    }
    std::vector<std::thread> threads_;
    std::atomic<unsigned> turn_{0};
    std::atomic<int> left_{0}, bad_{0};
    int8_t *dst_ = nullptr;
    const int8_t *src_ = nullptr;
    size_t n_ = 0;
    int parts_ = 1;
    bool check_ = false, stop_ = false;
};

// Moves the host layout of a replica through pinned memory: by way of h_res
// where it fits, else window by window, the threads' copy of one beside the
// transfer and kernel of the other.  With `out`, the error word comes first and
// nothing is written to host when it is raised.
static islf_status move_spins(islf_ctx *c, int rep, int8_t *host, bool out, Crew &crew)
{
    const Replica &R = c->reps[rep];
    const int Lz = R.desc.Lz, K = (Lz + 15) / 16;
    const long n = host_columns(R.desc);
    const size_t N = (size_t)R.desc.Lx * R.desc.Ly * Lz;
    auto at = [&](long col) { return (size_t)(col / K) * Lz + (size_t)(16 * (col % K)); };   // host byte of a column
    if (out) HIP_TRY(launch_fetch(&c->d_sync->error.v, nullptr, 0, 0, 1, c->h_res, c->stream));
    if (N <= 8 * (size_t)kResultWords) {
        int8_t *p = (int8_t *)(c->h_res + 8);
        if (!out) {
            memcpy(p, host, N);
            HIP_TRY(launch_import(c->fmt, c->d_desc, c->d_state, rep, Lz, 0, (uint32_t)n, 0, p, c->stream));
            return ISLF_OK;
        }
        HIP_TRY(launch_export(c->fmt, c->d_desc, rep, Lz, 0, (uint32_t)n, 0, p, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        landed(c);
        const islf_status st = take_error(c, rep);
        if (st == ISLF_OK) memcpy(host, p, N);
        return st;
    }
    for (hipEvent_t &ev : c->win_event)
        if (!ev) HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    if (!c->h_win && hipHostMalloc((void **)&c->h_win, 2 * kWindow, hipHostMallocDefault) != hipSuccess) {
        c->h_win = nullptr;
        return fail(ISLF_ENOMEM, "cannot allocate staging");
    }
    int8_t *dev = (int8_t *)dev_alloc(c, 2 * kWindow);
    if (!dev) return fail(ISLF_ENOMEM, "cannot allocate staging");
    const long per = (long)(kWindow / 16), wins = (n + per - 1) / per;
    hipError_t e = hipSuccess;
    islf_status st = ISLF_OK;
    auto start = [&](long w) {   // device side of window w
        const long c0 = w * per, c1 = std::min(n, c0 + per);
        const size_t h0 = at(c0), bytes = (c1 == n ? N : at(c1)) - h0;
        int8_t *d = dev + (w & 1) * kWindow, *p = c->h_win + (w & 1) * kWindow;
        if (out) {
            e = launch_export(c->fmt, c->d_desc, rep, Lz, (uint32_t)c0, (uint32_t)c1, h0, d, c->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(p, d, bytes, hipMemcpyDeviceToHost, c->stream);
        } else {
            e = hipMemcpyAsync(d, p, bytes, hipMemcpyHostToDevice, c->stream);
            if (e == hipSuccess)
                e = launch_import(c->fmt, c->d_desc, c->d_state, rep, Lz, (uint32_t)c0, (uint32_t)c1, h0, d, c->stream);
        }
        if (e == hipSuccess) e = hipEventRecord(c->win_event[w & 1], c->stream);
    };
    auto copy = [&](long w) {    // host side of window w
        const size_t h0 = at(w * per), bytes = (w + 1 == wins ? N : at((w + 1) * per)) - h0;
        int8_t *p = c->h_win + (w & 1) * kWindow;
        if (out) crew.run(host + h0, p, bytes, false);
        else crew.run(p, host + h0, bytes, false);
    };
    if (out) start(0);
    for (long w = 0; w < wins && e == hipSuccess && st == ISLF_OK; ++w) {
        if (out) {
            if (w + 1 < wins) start(w + 1);
            if (e == hipSuccess) e = hipEventSynchronize(c->win_event[w & 1]);
            if (e == hipSuccess && w == 0) st = take_error(c, rep);
            if (e == hipSuccess && st == ISLF_OK) copy(w);
        } else {
            if (w >= 2) e = hipEventSynchronize(c->win_event[w & 1]);
            if (e != hipSuccess) break;
            copy(w);
            start(w);
        }
    }
    const hipError_t es = hipStreamSynchronize(c->stream);
    if (es == hipSuccess) landed(c);
    dev_free(c, dev);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return fail(ISLF_EDEVICE, "copy of spins failed: %s", hipGetErrorString(e));
    return st;
}

extern "C" islf_status islf_set_spins(islf_ctx *ctx, int32_t rep, const int8_t *host, size_t n)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    Replica &R = ctx->reps[rep];
    const size_t N = (size_t)R.desc.Lx * R.desc.Ly * R.desc.Lz;
    if (!host || n != N) return fail(ISLF_EINVAL, "expected %zu spins, got %zu", N, n);
    if (R.t_host != 0 && !R.failed)
        return fail(ISLF_ESTATE, "set_spins is only valid before the first sweep (or after a failed launch)");
    Crew crew(N);
    if (crew.run(nullptr, host, N, true))
        for (size_t i = 0; i < n; ++i)
            if (host[i] != 1 && host[i] != -1) return fail(ISLF_EINVAL, "spin %zu is %d, not +-1", i, (int)host[i]);
    HIP_TRY(hipMemcpyAsync(ctx->d_desc + rep, &R.d, sizeof(RepDesc), hipMemcpyHostToDevice, ctx->stream));
    st = move_spins(ctx, rep, (int8_t *)host, false, crew);
    if (st != ISLF_OK) return st;
    hipError_t e = launch_recompute(ctx->fmt, ctx->d_desc, ctx->d_state, rep, host_columns(R.desc), nullptr, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail(ISLF_EDEVICE, "replica init failed: %s", hipGetErrorString(e));
    R.t_host = 0;
    if (R.failed) {
        R.failed = false;
        ctx->graph_valid = false;
    }
    return ISLF_OK;
}

extern "C" islf_status islf_get_spins(islf_ctx *ctx, int32_t rep, int8_t *host, size_t n)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    const Replica &R = ctx->reps[rep];
    const size_t N = (size_t)R.desc.Lx * R.desc.Ly * R.desc.Lz;
    if (!host || n != N) return fail(ISLF_EINVAL, "expected %zu spins, got %zu", N, n);
    Crew crew(N);
    return move_spins(ctx, rep, host, true, crew);
}

extern "C" islf_status islf_set_exec(islf_ctx *ctx, int32_t mode)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (mode < ISLF_EXEC_PLAIN || mode > ISLF_EXEC_PERSISTENT) return fail(ISLF_EINVAL, "invalid exec mode %d", mode);
    ctx->exec = mode;
    return ISLF_OK;
}

// Enqueues n >= 1 sweeps of the replicas in the device list dl (nl ids) over
// a plan: A(s) B(s) for each sweep, then F and the closing fold.  Optional
// events bracket each launch (A and B of sweep s at ev[4s..4s+3], F + fold
// at ev[4n], ev[4n+1]).
static hipError_t enqueue_plan(islf_ctx *c, const Plan &p, const int *dl, int nl, uint32_t n,
                               hipEvent_t *ev = nullptr, hipStream_t strm = nullptr)
{
    if (!strm) strm = c->stream;
    hipError_t e = hipSuccess;
    auto mark = [&](size_t i) {
        if (ev && e == hipSuccess) e = hipEventRecord(ev[i], strm);
    };
    for (uint32_t s = 0; s < n && e == hipSuccess; ++s) {
        mark(4 * (size_t)s);
        if (e == hipSuccess)
            e = launch_sweep(c->fmt, KIND_A, c->d_desc, c->d_state, p.items, p.first, p.grid, dl, nl, s,
                             s ? FLAG_PREV : 0u, strm);
        mark(4 * (size_t)s + 1);
        mark(4 * (size_t)s + 2);
        if (e == hipSuccess)
            e = launch_sweep(c->fmt, KIND_B, c->d_desc, c->d_state, p.items, p.first, p.grid, dl, nl, s,
                             s ? FLAG_FOLD : 0u, strm);
        mark(4 * (size_t)s + 3);
    }
    mark(4 * (size_t)n);
    if (e == hipSuccess)
        e = launch_sweep(c->fmt, KIND_F, c->d_desc, c->d_state, p.items, p.first, p.slab_grid, dl, nl, n - 1, 0u,
                         strm);
    if (e == hipSuccess) e = launch_fold(c->d_desc, c->d_state, dl, nl, n - 1, n, strm);
    mark(4 * (size_t)n + 1);
    return e;
}

// Enqueues n sweeps in the context's execution form (plans prepared, no
// checks, no sync).
// Concurrent groups: group g issues on side stream g, a stream the context
// creates, group 0 included.  Fork: every side stream waits for the work
// issued before on the context's stream; join: the context's stream waits for
// every side stream.  The context's own stream (the caller's) carries no group
// work: the runtime maps streams onto a few hardware queues, and with the
// caller's stream carrying group 0, some contexts of a process ran a batch at
// 1,700 instead of 2,400 updates/ns (bit-packed), as when two groups share a
// queue and serialise; with the context's own streams for every group they
// did not.  An ungrouped context issues on its own stream.
static hipStream_t group_stream(const islf_ctx *c, int g, int G)
{
    return G > 1 ? c->side_stream[g] : c->stream;
}

static hipError_t fork_groups(islf_ctx *c, int G)
{
    hipError_t e = hipEventRecord(c->side_event[0], c->stream);
    for (int g = 0; g < G && e == hipSuccess; ++g) e = hipStreamWaitEvent(c->side_stream[g], c->side_event[0], 0);
    return e;
}

static hipError_t join_groups(islf_ctx *c, int G)
{
    hipError_t e = hipSuccess;
    for (int g = 0; g < G && e == hipSuccess; ++g) {
        e = hipEventRecord(c->side_event[g + 1], c->side_stream[g]);
        if (e == hipSuccess) e = hipStreamWaitEvent(c->stream, c->side_event[g + 1], 0);
    }
    return e;
}

static hipError_t enqueue_group(islf_ctx *c, int g, uint32_t n)
{
    return enqueue_plan(c, c->group_plan[g], c->d_group_live + c->group_off[g], c->group_len[g], n, nullptr,
                        c->side_stream[g]);
}

static islf_status enqueue_sweeps(islf_ctx *c, uint32_t n)
{
    const int nl = (int)c->live.size();
    if (nl == 0 || n == 0) return ISLF_OK;
    if (c->exec == ISLF_EXEC_PERSISTENT) {
        const Plan &p = c->persistent;
        hipError_t e = c->persistent_teams
                           ? launch_persistent_teams(c->fmt, c->d_desc, c->d_state, p.items, p.first, c->d_teams, n,
                                                     c->d_sync, c->d_rsync, c->rsync_cap, p.grid, c->stream)
                           : launch_persistent(c->fmt, c->d_desc, c->d_state, p.items, p.first, c->d_live, nl, n,
                                               c->d_sync, p.grid, c->stream);
        if (e != hipSuccess) return fail(ISLF_EDEVICE, "persistent launch failed: %s", hipGetErrorString(e));
        return ISLF_OK;
    }
    if (c->exec == ISLF_EXEC_BATCHED && num_groups(c) > 1) {
        const int G = num_groups(c);
        HIP_TRY(fork_groups(c, G));
        for (int g = 0; g < G; ++g) HIP_TRY(enqueue_group(c, g, n));
        HIP_TRY(join_groups(c, G));
        return ISLF_OK;
    }
    if (c->exec == ISLF_EXEC_BATCHED) {
        HIP_TRY(enqueue_plan(c, c->batched, c->d_live, nl, n));
        return ISLF_OK;
    }
    // plain: one lattice per launch; replica r's fold list is its entry in d_live
    for (uint32_t s = 0; s < n; ++s)
        for (int k = 0; k < 2; ++k)
            for (int li = 0; li < nl; ++li) {
                const Plan &p = c->plain[c->live[li]];
                HIP_TRY(launch_sweep(c->fmt, k, c->d_desc, c->d_state, p.items, p.first, p.grid, c->d_live + li, 1,
                                     s, s ? (k == 0 ? FLAG_PREV : FLAG_FOLD) : 0u, c->stream));
            }
    for (int li = 0; li < nl; ++li) {
        const Plan &p = c->plain[c->live[li]];
        HIP_TRY(launch_sweep(c->fmt, KIND_F, c->d_desc, c->d_state, p.items, p.first, p.slab_grid, c->d_live + li,
                             1, n - 1, 0u, c->stream));
    }
    HIP_TRY(launch_fold(c->d_desc, c->d_state, c->d_live, nl, n - 1, n, c->stream));
    return ISLF_OK;
}

// The form a run of n sweeps takes, its plans built.
static islf_status prepare_form(islf_ctx *c, uint32_t n, bool *resident)
{
    islf_status st = resident_applies(c, n, resident);
    if (st != ISLF_OK || *resident) return st;
    return prepare_plans(c, c->exec);
}

static islf_status enqueue_form(islf_ctx *c, uint32_t n, bool resident)
{
    if (!resident) return enqueue_sweeps(c, n);
    HIP_TRY(enqueue_resident(c, n));
    return ISLF_OK;
}

static const ResPlan &resident_plan(const islf_ctx *c, int rep)
{
    return c->exec == ISLF_EXEC_PLAIN ? c->resident_plain[rep] : c->resident;
}

// Launches with clusters of a run of n sweeps, and the cluster workgroups of one at most.
static void resident_size(const islf_ctx *c, uint32_t n, uint32_t *launches, int *members)
{
    *launches = 0;
    *members = 0;
    for (int r : c->live) {
        const ResPlan &p = resident_plan(c, r);
        if (p.L.members) *launches += (n + p.max_sweeps - 1) / p.max_sweeps;
        *members = std::max(*members, p.L.members);
        if (c->exec != ISLF_EXEC_PLAIN) break;
    }
}

// Whether chains of several contexts side by side beat resident runs in turn.
// A chain of one stream leaves the device idle between its launches, which
// other contexts' chains fill: they then cost about what concurrent groups do.
// Chains that are such groups already gain nothing from each other.
static bool prefers_chain(const islf_ctx *c)
{
    if (c->exec == ISLF_EXEC_PERSISTENT || (c->exec == ISLF_EXEC_BATCHED && c->live.size() > 1)) return false;
    double res = 0.0, chain = 0.0;
    for (int r : c->live) {
        const ResPlan &p = resident_plan(c, r);
        res += p.sweep_us;
        chain += grouped_sweep_us(c, p.sites, 1);
    }
    return chain < res;
}

// A run of the chain, in its turn.
template <class ENQUEUE>
static islf_status run_chain(islf_ctx *c, bool joins, ENQUEUE enqueue)
{
    std::unique_lock<std::mutex> lock(turns(c).m);
    bool mark = false;
    HIP_TRY(start_chain(c, joins, &mark));
    // (clusters are ordered behind runs that joined, by an event behind all of them; nobody goes beside the others)
    if (!joins) lock.unlock();
    const islf_status st = enqueue();
    if (st != ISLF_OK) return st;
    HIP_TRY(end_chain(c, mark));
    return ISLF_OK;
}

// A resident run, in its turn; enqueued if that is TURN_GO.
template <class ENQUEUE>
static islf_status run_resident(islf_ctx *c, uint32_t launches, int members, bool chain_if_met, Turn *turn,
                                ENQUEUE enqueue)
{
    *turn = TURN_GO;
    if (!members) return enqueue();   // waits for nobody, and nobody has to wait for it
    std::lock_guard<std::mutex> lock(turns(c).m);
    hipError_t e = hipSuccess;
    *turn = take_turn(c, members, chain_if_met, &e);
    HIP_TRY(e);
    if (*turn != TURN_GO) return ISLF_OK;
    c->members = std::max(members_in_flight(c), members);
    c->issued += launches;
    c->cluster_until = c->issued;
    c->unmarked = false;   // (these end what came before them, too)
    const islf_status st = enqueue();
    if (st != ISLF_OK) return st;
    c->cluster_runs += 1;
    return ISLF_OK;
}

static islf_status run_form(islf_ctx *c, uint32_t n, bool resident)
{
    if (n == 0 || c->live.empty()) return ISLF_OK;
    if (being_captured(c)) return enqueue_form(c, n, resident);
    Turn turn = TURN_CHAIN;
    if (resident) {
        uint32_t launches;
        int members;
        resident_size(c, n, &launches, &members);
        islf_status st = run_resident(c, launches, members, prefers_chain(c), &turn,
                                      [&] { return enqueue_form(c, n, true); });
        if (st != ISLF_OK || turn == TURN_GO) return st;
        st = prepare_plans(c, c->exec);
        if (st != ISLF_OK) return st;
    }
    return run_chain(c, turn == TURN_JOIN, [&] { return enqueue_sweeps(c, n); });
}

static islf_status check_none_failed(const islf_ctx *c)
{
    for (int r : c->live)
        if (c->reps[r].failed)
            return fail(ISLF_ESTATE, "replica %d was cut short by a failed launch (restart it with "
                                     "islf_set_spins or retire it)", r);
    return ISLF_OK;
}

static islf_status check_sweep_range(islf_ctx *c, uint64_t n)
{
    for (int r : c->live)
        if (c->reps[r].t_host + n > 0xFFFFFFFFull)
            return fail(ISLF_ERANGE, "replica %d would pass 2^32-1 sweeps", r);
    return ISLF_OK;
}

extern "C" islf_status islf_sweep(islf_ctx *ctx, uint32_t n_sweeps)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    islf_status st = check_none_failed(ctx);
    if (st != ISLF_OK) return st;
    bool resident = false;
    st = prepare_form(ctx, n_sweeps, &resident);
    if (st != ISLF_OK) return st;
    st = check_sweep_range(ctx, n_sweeps);
    if (st != ISLF_OK) return st;
    st = run_form(ctx, n_sweeps, resident);
    if (st != ISLF_OK) return st;
    for (int r : ctx->live) ctx->reps[r].t_host += n_sweeps;
    return ISLF_OK;
}

extern "C" islf_status islf_sweep_count(islf_ctx *ctx, int32_t rep, uint64_t *t)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!t) return fail(ISLF_EINVAL, "NULL output");
    RepState s;
    st = fetch(ctx, rep, ctx->d_state + rep, 0, sizeof s / 8, sizeof s / 8);
    if (st != ISLF_OK) return st;
    memcpy(&s, ctx->h_res + 8, sizeof s);
    if (s.t != (uint32_t)ctx->reps[rep].t_host)
        return fail(ISLF_EDEVICE, "device sweep counter %u != issued %llu", s.t,
                    (unsigned long long)ctx->reps[rep].t_host);
    *t = s.t;
    return ISLF_OK;
}

static islf_status check_records(islf_ctx *c, int rep, uint64_t first, uint32_t count)
{
    const uint64_t t = c->reps[rep].t_host;
    if (count == 0) return fail(ISLF_EINVAL, "count must be >= 1");
    if (first + count > t) return fail(ISLF_ERANGE, "records up to sweep %llu requested, %llu run",
                                       (unsigned long long)(first + count), (unsigned long long)t);
    if (t > c->cap && first < t - c->cap)
        return fail(ISLF_ERANGE, "record %llu has left the ring (capacity %u)", (unsigned long long)first, c->cap);
    return ISLF_OK;
}

extern "C" islf_status islf_measure(islf_ctx *ctx, int32_t rep, uint64_t first, uint32_t count, islf_obs *out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!out) return fail(ISLF_EINVAL, "NULL output");
    st = check_records(ctx, rep, first, count);
    if (st != ISLF_OK) return st;
    const Replica &R = ctx->reps[rep];
    constexpr long W = sizeof(islf_obs) / 8;
    if (count <= kResultWords / W && count <= ctx->cap) {
        st = fetch(ctx, rep, R.d.rec, (long)(first % ctx->cap) * W, (long)count * W, (long)ctx->cap * W);
        if (st == ISLF_OK) memcpy(out, ctx->h_res + 8, count * sizeof(islf_obs));
        return st;
    }
    st = check_intact(ctx, rep);
    if (st != ISLF_OK) return st;
    uint32_t done = 0;
    while (done < count) {
        const uint32_t slot = (uint32_t)((first + done) % ctx->cap);
        const uint32_t n = std::min<uint32_t>(count - done, ctx->cap - slot);
        HIP_TRY(hipMemcpyAsync(out + done, R.d.rec + slot, n * sizeof(islf_obs), hipMemcpyDeviceToHost, ctx->stream));
        done += n;
    }
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return ISLF_OK;
}

extern "C" islf_status islf_recompute(islf_ctx *ctx, int32_t rep, islf_obs *out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!out) return fail(ISLF_EINVAL, "NULL output");
    const Replica &R = ctx->reps[rep];
    const hipError_t e = launch_recompute(ctx->fmt, ctx->d_desc, ctx->d_state, rep, host_columns(R.desc), ctx->d_scratch,
                                          ctx->stream);
    if (e != hipSuccess) return fail(ISLF_EDEVICE, "recompute failed: %s", hipGetErrorString(e));
    st = fetch(ctx, rep, ctx->d_scratch, 0, 4, 4);
    if (st != ISLF_OK) return st;
    const unsigned long long *h = ctx->h_res + 8;
    out->B = (int64_t)h[0];
    out->M = (int64_t)h[1];
    out->M1 = (int64_t)h[2];
    out->Mn = (int64_t)h[3];
    return ISLF_OK;
}

extern "C" islf_status islf_record_energy(islf_ctx *ctx, int32_t rep, uint64_t first, uint32_t count,
                                          double *out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!out) return fail(ISLF_EINVAL, "NULL output");
    st = check_records(ctx, rep, first, count);
    if (st != ISLF_OK) return st;
    const Replica &R = ctx->reps[rep];
    if ((long)count <= kResultWords) {
        HIP_TRY(launch_energy(R.d.rec, ctx->cap, first, count, R.desc.J, R.desc.H, R.desc.h1, R.desc.hn,
                              (double *)(ctx->h_res + 8), ctx->stream));
        st = fetch(ctx, rep);
        if (st == ISLF_OK) memcpy(out, ctx->h_res + 8, sizeof(double) * count);
        return st;
    }
    st = check_intact(ctx, rep);
    if (st != ISLF_OK) return st;
    double *tmp = (double *)dev_alloc(ctx, sizeof(double) * count);
    if (!tmp) return fail(ISLF_ENOMEM, "cannot allocate staging");
    hipError_t e = launch_energy(R.d.rec, ctx->cap, first, count, R.desc.J, R.desc.H, R.desc.h1, R.desc.hn, tmp,
                                 ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(out, tmp, sizeof(double) * count, hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    dev_free(ctx, tmp);
    if (e != hipSuccess) return fail(ISLF_EDEVICE, "energy failed: %s", hipGetErrorString(e));
    return ISLF_OK;
}

extern "C" islf_status islf_means(islf_ctx *ctx, uint64_t first, uint32_t count, double *out)
{
    if (!ctx || !out) return fail(ISLF_EINVAL, "NULL argument");
    islf_status st = sync_tables(ctx);
    if (st != ISLF_OK) return st;
    const int n = (int)ctx->reps.size();
    for (int r = 0; r < n; ++r) {
        if (!ctx->reps[r].live) continue;
        st = check_records(ctx, r, first, count);
        if (st != ISLF_OK) return st;
    }
    // live replicas only; dead slots report NaN
    const int nl = (int)ctx->live.size();
    const bool fits = 5l * nl <= kResultWords;
    std::vector<double> tmp_h(fits ? 0 : 5 * (size_t)nl);
    double *tmp = (double *)(ctx->h_res + 8);
    if (fits && nl > 0) HIP_TRY(launch_means(ctx->d_desc, ctx->d_live, nl, first, count, tmp, ctx->stream));
    st = check_device_error(ctx);
    if (st != ISLF_OK) return st;
    st = check_none_failed(ctx);
    if (st != ISLF_OK) return st;
    if (!fits) {
        double *dev = (double *)dev_alloc(ctx, sizeof(double) * 5 * nl);
        if (!dev) return fail(ISLF_ENOMEM, "cannot allocate staging");
        hipError_t e = launch_means(ctx->d_desc, ctx->d_live, nl, first, count, dev, ctx->stream);
        tmp = tmp_h.data();
        if (e == hipSuccess) e = hipMemcpyAsync(tmp, dev, sizeof(double) * 5 * nl, hipMemcpyDeviceToHost, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        dev_free(ctx, dev);
        if (e != hipSuccess) return fail(ISLF_EDEVICE, "means failed: %s", hipGetErrorString(e));
    }
    for (int r = 0; r < n; ++r)
        for (int k = 0; k < 5; ++k) out[5 * r + k] = NAN;
    for (int i = 0; i < nl; ++i)
        for (int k = 0; k < 5; ++k) out[5 * ctx->live[i] + k] = tmp[5 * i + k];
    return ISLF_OK;
}

// Host FP64 energies of records (Sec. II.A Eq. 1), in the order the header
// states; plain C arithmetic (the library is built without FMA contraction).
extern "C" islf_status islf_energy(const islf_replica_desc *desc, const islf_obs *obs, size_t n, double *E_out)
{
    if (!desc) return fail(ISLF_EINVAL, "NULL replica descriptor");
    if (n > 0 && (!obs || !E_out)) return fail(ISLF_EINVAL, "NULL records or output");
    const double J = desc->J, H = desc->H, h1 = desc->h1, hn = desc->hn;
    if (!isfinite(J) || !isfinite(H) || !isfinite(h1) || !isfinite(hn))
        return fail(ISLF_EINVAL, "J, H, h1, hn must be finite");
    for (size_t k = 0; k < n; ++k) {
        double e = -J * (double)obs[k].B;
        e = e - H * (double)obs[k].M;
        e = e - h1 * (double)obs[k].M1;
        e = e - hn * (double)obs[k].Mn;
        E_out[k] = e;
    }
    return ISLF_OK;
}

// The means of islf_means with the kernel's output in the device's scratch
// array instead of a staging allocation; the per-replica results are copied
// to the front of out and moved to their slots from the back (slot ids of
// live replicas are ascending and never below their rank, so no result is
// overwritten before it is moved).
extern "C" islf_status islf_means_noalloc(islf_ctx *ctx, uint64_t first, uint32_t count, double *out)
{
    if (!ctx || !out) return fail(ISLF_EINVAL, "NULL argument");
    if (ctx->dirty)
        return fail(ISLF_ESTATE, "replica tables are not current (after islf_set_tile, sweep or call islf_means once)");
    const int n = (int)ctx->reps.size();
    const int nl = (int)ctx->live.size();
    if (nl > kNoAllocMaxReps)
        return fail(ISLF_ERANGE, "%d live replicas exceed the %d the allocation-free means serve per call", nl,
                    kNoAllocMaxReps);
    islf_status st;
    for (int r : ctx->live) {
        st = check_records(ctx, r, first, count);
        if (st != ISLF_OK) return st;
    }
    st = check_device_error(ctx);
    if (st != ISLF_OK) return st;
    st = check_none_failed(ctx);
    if (st != ISLF_OK) return st;
    if (nl > 0) {
        HIP_TRY(launch_means(ctx->d_desc, ctx->d_live, nl, first, count, ctx->noalloc_scratch, ctx->stream));
        HIP_TRY(hipMemcpyAsync(out, ctx->noalloc_scratch, sizeof(double) * 5 * nl, hipMemcpyDeviceToHost,
                               ctx->stream));
        HIP_TRY(hipStreamSynchronize(ctx->stream));
    }
    for (int i = nl - 1; i >= 0; --i) {
        const int r = ctx->live[i];
        if (r != i)
            for (int k = 0; k < 5; ++k) out[5 * r + k] = out[5 * i + k];
    }
    int li = 0;
    for (int r = 0; r < n; ++r) {
        if (li < nl && ctx->live[li] == r) {
            ++li;
            continue;
        }
        for (int k = 0; k < 5; ++k) out[5 * r + k] = NAN;
    }
    return ISLF_OK;
}

// Host FP64 cumulative trapezoid (Eq. 9 / Eq. 22 over the field, Eq. 19 over
// beta), left to right.
extern "C" islf_status islf_integrate(const double *h, const double *mean_M1, const double *mean_Mn, int32_t n,
                                      double c1, double cn, double norm, double *cumulative_out)
{
    if (!h || !mean_M1 || !mean_Mn || !cumulative_out) return fail(ISLF_EINVAL, "NULL argument");
    if (n < 1) return fail(ISLF_EINVAL, "need n >= 1 points");
    double g_prev = norm * (c1 * mean_M1[0] + cn * mean_Mn[0]);
    double acc = 0.0;
    cumulative_out[0] = 0.0;
    for (int32_t r = 1; r < n; ++r) {
        const double g = norm * (c1 * mean_M1[r] + cn * mean_Mn[r]);
        const double step = 0.5 * (h[r] - h[r - 1]);
        acc = acc + step * (g_prev + g);
        cumulative_out[r] = acc;
        g_prev = g;
    }
    return ISLF_OK;
}

extern "C" islf_status islf_integrate_device(const double *h, const double *m1, const double *mn, int32_t n,
                                             double c1, double cn, double norm, double *out, void *hip_stream)
{
    if (!h || !m1 || !mn || !out) return fail(ISLF_EINVAL, "NULL argument");
    if (n < 1) return fail(ISLF_EINVAL, "need n >= 1 points");
    HIP_TRY(launch_integrate(h, m1, mn, n, c1, cn, norm, out, (hipStream_t)hip_stream));
    return ISLF_OK;
}

extern "C" islf_status islf_footprint_bytes(const islf_replica_desc *desc, int32_t spin_format,
                                            uint32_t obs_capacity, uint64_t *bytes)
{
    if (!bytes) return fail(ISLF_EINVAL, "NULL output");
    islf_status st = validate(desc);
    if (st != ISLF_OK) return st;
    if (spin_format != ISLF_SPIN_INT8 && spin_format != ISLF_SPIN_BITPACK)
        return fail(ISLF_EINVAL, "invalid spin format %d", spin_format);
    *bytes = replica_bytes(desc, spin_format, obs_capacity) +
             sizeof(Entry) * work_entries(*desc, i8_shape(*desc, default_tile(desc, spin_format), spin_format), spin_format) +
             sizeof(RepDesc) + sizeof(RepState);
    return ISLF_OK;
}

extern "C" islf_status islf_plan_preview(const islf_replica_desc *descs, int32_t n_reps, int32_t spin_format,
                                         int32_t tile, int32_t grid, int32_t *shapes, int32_t *items,
                                         int32_t items_cap, int32_t *n_items, int32_t *first, int32_t first_cap,
                                         int32_t *n_first)
{
    if (!descs || !n_items || !n_first) return fail(ISLF_EINVAL, "NULL argument");
    if (n_reps < 1) return fail(ISLF_EINVAL, "n_reps must be >= 1");
    if (spin_format != ISLF_SPIN_INT8 && spin_format != ISLF_SPIN_BITPACK)
        return fail(ISLF_EINVAL, "invalid spin format %d", spin_format);
    if (tile < -1 || tile >= num_tiles_of(spin_format)) return fail(ISLF_EINVAL, "invalid tile %d", tile);
    if (grid < 1 || grid > (1 << 20)) return fail(ISLF_EINVAL, "invalid workgroup count %d", grid);
    if (items_cap < 0 || first_cap < 0) return fail(ISLF_EINVAL, "negative capacity");
    std::vector<Entry> S, M;
    for (int r = 0; r < n_reps; ++r) {
        islf_status st = validate(descs + r);
        if (st != ISLF_OK) return st;
        Replica R;
        R.desc = descs[r];
        R.tile = tile >= 0 ? tile : default_tile(descs + r, spin_format);
        build_work(R, r, spin_format);
        if (shapes) {
            shapes[4 * r + 0] = R.tile;
            shapes[4 * r + 1] = R.d.i8_tj;
            shapes[4 * r + 2] = R.d.i8_ty;
            shapes[4 * r + 3] = R.d.i8_mx;
        }
        S.insert(S.end(), R.slab.begin(), R.slab.end());
        M.insert(M.end(), R.main.begin(), R.main.end());
    }
    std::vector<Entry> it;
    std::vector<int> fi;
    partition_items(S, M, grid, it, fi, tail_taper(spin_format));
    *n_items = (int32_t)it.size();
    *n_first = (int32_t)fi.size();
    if ((items && (int64_t)it.size() > items_cap) || (first && (int64_t)fi.size() > first_cap))
        return fail(ISLF_ERANGE, "plan needs %zu items and %zu offsets", it.size(), fi.size());
    if (items)
        for (size_t i = 0; i < it.size(); ++i) {
            const Entry &e = it[i];
            const int32_t v[6] = {e.rep, e.x0, e.y0, e.j0, e.nsteps, e.kind};
            for (int k = 0; k < 6; ++k) items[6 * i + k] = v[k];
        }
    if (first)
        for (size_t i = 0; i < fi.size(); ++i) first[i] = fi[i];
    return ISLF_OK;
}

extern "C" islf_status islf_batch_add(islf_ctx *ctx, const islf_replica_desc *desc, int32_t *slot)
{
    if (!ctx || !slot) return fail(ISLF_EINVAL, "NULL argument");
    int s = -1;
    islf_status st = add_replica(ctx, desc, &s);
    if (st != ISLF_OK) return st;
    st = sync_tables(ctx);
    hipError_t e = st == ISLF_OK ? start_replica(ctx, s) : hipSuccess;
    if (st == ISLF_OK && e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) st = fail(ISLF_EDEVICE, "replica init failed: %s", hipGetErrorString(e));
    if (st != ISLF_OK) {
        // the tables without it again (they were not replaced if there was no memory)
        const std::string keep = g_err;
        ctx->reps[s].live = false;
        ctx->dirty = true;
        (void)sync_tables(ctx);
        g_err = keep;
        return st;
    }
    *slot = s;
    return ISLF_OK;
}

extern "C" islf_status islf_batch_retire(islf_ctx *ctx, int32_t slot)
{
    islf_status st = check_rep(ctx, slot);
    if (st != ISLF_OK) return st;
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    Replica &R = ctx->reps[slot];
    R.live = false;
    R.t_host = 0;
    R.failed = false;
    // the slot's memory goes back to the allocator, so the device memory a
    // context holds follows its live replicas
    dev_free(ctx, R.mem);
    R.mem = nullptr;
    R.mem_bytes = 0;
    R.main.clear();
    R.slab.clear();
    free_resident(ctx, ctx->resident);
    for (ResPlan &p : ctx->resident_plain) free_resident(ctx, p);
    ctx->dirty = true;
    return sync_tables(ctx);
}

extern "C" islf_status islf_graph_capture(islf_ctx *ctx, uint32_t k_sweeps)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (k_sweeps < 1) return fail(ISLF_EINVAL, "k_sweeps must be >= 1");
    if (!ctx->stream) return fail(ISLF_ESTATE, "graph capture needs a non-default stream");
    islf_status st = check_none_failed(ctx);
    if (st != ISLF_OK) return st;
    bool resident = false;
    st = prepare_form(ctx, k_sweeps, &resident);
    if (st != ISLF_OK) return st;
    destroy_graphs(ctx);
    // concurrent groups: one graph per group, captured on the group's own
    // stream, so that replays run each group on a stream the context owns
    // (the streams a runtime picks for the branches of one multi-stream graph
    // may share a hardware queue and serialise the groups)
    const bool grouped = !resident && ctx->exec == ISLF_EXEC_BATCHED && num_groups(ctx) > 1;
    const int G = grouped ? num_groups(ctx) : 1;
    for (int gi = 0; gi < G; ++gi) {
        hipStream_t sg = group_stream(ctx, gi, G);
        // (another context may record an event on the stream: not while it is captured)
        std::unique_lock<std::mutex> lock(turns(ctx).m);
        HIP_TRY(hipStreamBeginCapture(sg, hipStreamCaptureModeThreadLocal));
        hipError_t ee = hipSuccess;
        if (grouped) ee = enqueue_group(ctx, gi, k_sweeps);
        else st = enqueue_form(ctx, k_sweeps, resident);
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(sg, &g);
        lock.unlock();
        if (st != ISLF_OK || ee != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            destroy_graphs(ctx);
            return st != ISLF_OK ? st : fail(ISLF_EDEVICE, "launch during capture failed: %s", hipGetErrorString(ee));
        }
        if (e != hipSuccess) {
            destroy_graphs(ctx);
            return fail(ISLF_EDEVICE, "graph capture failed: %s", hipGetErrorString(e));
        }
        ctx->graphs.push_back(g);
        hipGraphExec_t ex = nullptr;
        e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            destroy_graphs(ctx);
            return fail(ISLF_EDEVICE, "graph instantiation failed: %s", hipGetErrorString(e));
        }
        ctx->graph_execs.push_back(ex);
    }
    ctx->graph_sweeps = k_sweeps;
    ctx->graph_exec = ctx->exec;
    ctx->graph_resident = resident;
    if (resident) {
        resident_size(ctx, k_sweeps, &ctx->graph_launches, &ctx->graph_members);
        ctx->graph_prefers_chain = prefers_chain(ctx);
    }
    ctx->graph_valid = true;
    return ISLF_OK;
}

static islf_status launch_graphs(islf_ctx *c, uint32_t n)
{
    const int G = (int)c->graph_execs.size();
    if (G > 1) HIP_TRY(fork_groups(c, G));
    for (uint32_t i = 0; i < n; ++i)
        for (int g = 0; g < G; ++g) HIP_TRY(hipGraphLaunch(c->graph_execs[g], group_stream(c, g, G)));
    if (G > 1) HIP_TRY(join_groups(c, G));
    return ISLF_OK;
}

// n replays in their turn.  A graph of cluster launches that may not go now is
// left alone: the same sweeps are enqueued as a chain.
static islf_status run_graphs(islf_ctx *c, uint32_t n)
{
    if (being_captured(c)) return launch_graphs(c, n);
    if (!c->graph_resident) return run_chain(c, false, [&] { return launch_graphs(c, n); });
    Turn turn = TURN_GO;
    islf_status st = run_resident(c, c->graph_launches * n, c->graph_members, c->graph_prefers_chain, &turn,
                                  [&] { return launch_graphs(c, n); });
    if (st != ISLF_OK || turn == TURN_GO) return st;
    const int now = c->exec;
    c->exec = c->graph_exec;
    st = prepare_plans(c, c->exec);
    if (st == ISLF_OK)
        st = run_chain(c, turn == TURN_JOIN, [&] {
            islf_status s = ISLF_OK;
            for (uint32_t i = 0; i < n && s == ISLF_OK; ++i) s = enqueue_sweeps(c, c->graph_sweeps);
            return s;
        });
    c->exec = now;
    return st;
}

extern "C" islf_status islf_run_graph(islf_ctx *ctx, uint32_t n_replays)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (!ctx->graph_valid || ctx->dirty) return fail(ISLF_ESTATE, "no valid captured graph");
    islf_status st = check_none_failed(ctx);
    if (st != ISLF_OK) return st;
    st = check_sweep_range(ctx, (uint64_t)ctx->graph_sweeps * n_replays);
    if (st != ISLF_OK) return st;
    if (n_replays > 0 && !ctx->live.empty()) {
        st = run_graphs(ctx, n_replays);
        if (st != ISLF_OK) return st;
    }
    for (int r : ctx->live) ctx->reps[r].t_host += (uint64_t)ctx->graph_sweeps * n_replays;
    return ISLF_OK;
}

extern "C" islf_status islf_num_tiles(int32_t spin_format, int32_t *n)
{
    if (!n) return fail(ISLF_EINVAL, "NULL output");
    if (spin_format != ISLF_SPIN_INT8 && spin_format != ISLF_SPIN_BITPACK)
        return fail(ISLF_EINVAL, "invalid spin format %d", spin_format);
    *n = num_tiles_of(spin_format);
    return ISLF_OK;
}

extern "C" islf_status islf_get_tile(const islf_ctx *ctx, int32_t rep, int32_t *tile)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!tile) return fail(ISLF_EINVAL, "NULL output");
    *tile = ctx->reps[rep].tile;
    return ISLF_OK;
}

extern "C" islf_status islf_set_tile(islf_ctx *ctx, int32_t rep, int32_t tile)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (tile < 0 || tile >= num_tiles_of(ctx->fmt)) return fail(ISLF_EINVAL, "tile %d out of range", tile);
    Replica &R = ctx->reps[rep];
    R.tile = tile;
    R.tile_set = true;
    build_work(R, rep, ctx->fmt);
    ctx->dirty = true;
    return ISLF_OK;
}

// Timed runs per autotune trial (the shortest counts), and per finalist of
// the launch-configuration search.
constexpr int kTrialRuns = 3;
constexpr int kFinalRuns = 6;
constexpr int kFinalists = 4;

// Times one tile variant for one size class: the class's replicas sweep
// `sweeps` times in the batched form over a plan of their own (events on the
// context stream).  Spins, records and state are restored afterwards by the
// caller.
static islf_status time_variant(islf_ctx *c, const std::vector<int> &cls, int tile, uint32_t sweeps, double *ms)
{
    std::vector<Entry> M, S;
    for (int r : cls) {
        Replica &R = c->reps[r];
        R.tile = tile;
        build_work(R, r, c->fmt);
        M.insert(M.end(), R.main.begin(), R.main.end());
        S.insert(S.end(), R.slab.begin(), R.slab.end());
        HIP_TRY(hipMemcpyAsync(c->d_desc + r, &R.d, sizeof(RepDesc), hipMemcpyHostToDevice, c->stream));
    }
    Plan plan;
    islf_status st = build_plan(c, plan, S, M, c->grid_override ? c->grid_override : c->sweep_slots);
    if (st != ISLF_OK) {
        free_plan(c, plan);
        return st;
    }
    int *dl = (int *)dev_alloc(c, sizeof(int) * cls.size());
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t err = dl ? hipSuccess : hipErrorOutOfMemory;
    if (err == hipSuccess) err = hipEventCreate(&e0);
    if (err == hipSuccess) err = hipEventCreate(&e1);
    if (err == hipSuccess) err = hipMemcpyAsync(dl, cls.data(), sizeof(int) * cls.size(), hipMemcpyHostToDevice, c->stream);
    // one warm-up sweep, then the shortest of three timed runs (a single run
    // of a few sweeps is too noisy to rank variants)
    if (err == hipSuccess) err = enqueue_plan(c, plan, dl, (int)cls.size(), 1);
    float t = 0.f;
    for (int run = 0; run < kTrialRuns && err == hipSuccess; ++run) {
        err = hipEventRecord(e0, c->stream);
        if (err == hipSuccess) err = enqueue_plan(c, plan, dl, (int)cls.size(), sweeps);
        if (err == hipSuccess) err = hipEventRecord(e1, c->stream);
        if (err == hipSuccess) err = hipStreamSynchronize(c->stream);
        float tr = 0.f;
        if (err == hipSuccess) err = hipEventElapsedTime(&tr, e0, e1);
        if (err == hipSuccess && (run == 0 || tr < t)) t = tr;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    free_plan(c, plan);
    dev_free(c, dl);
    if (err != hipSuccess) return fail(ISLF_EDEVICE, "autotune trial failed: %s", hipGetErrorString(err));
    *ms = t;
    return ISLF_OK;
}

extern "C" islf_status islf_autotune(islf_ctx *ctx, uint32_t sweeps)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (sweeps < 1) return fail(ISLF_EINVAL, "sweeps must be >= 1");
    islf_status st = sync_tables(ctx);
    if (st != ISLF_OK) return st;
    bool mark = false;
    {
        std::lock_guard<std::mutex> lock(turns(ctx).m);
        HIP_TRY(start_chain(ctx, false, &mark));   // (its trials are in flight to the end)
    }
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    // size classes: replicas of one shape share a variant
    std::vector<std::vector<int>> classes;
    for (int r : ctx->live) {
        bool placed = false;
        for (auto &cl : classes) {
            const islf_replica_desc &a = ctx->reps[cl[0]].desc, &b = ctx->reps[r].desc;
            if (a.Lx == b.Lx && a.Ly == b.Ly && a.Lz == b.Lz) {
                cl.push_back(r);
                placed = true;
                break;
            }
        }
        if (!placed) classes.push_back({r});
    }
    // back up every live replica's memory block and state
    std::vector<void *> backup(ctx->reps.size(), nullptr);
    RepState *st_backup = (RepState *)dev_alloc(ctx, sizeof(RepState) * ctx->slot_capacity);
    islf_status result = st_backup ? ISLF_OK : fail(ISLF_ENOMEM, "cannot back up replica state");
    for (int r : ctx->live) {
        if (result != ISLF_OK) break;
        Replica &R = ctx->reps[r];
        backup[r] = dev_alloc(ctx, R.mem_bytes);
        if (!backup[r]) result = fail(ISLF_ENOMEM, "cannot back up replica %d", r);
        else if (hipMemcpyAsync(backup[r], R.mem, R.mem_bytes, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess)
            result = fail(ISLF_EDEVICE, "backup copy failed");
    }
    if (result == ISLF_OK &&
        hipMemcpyAsync(st_backup, ctx->d_state, sizeof(RepState) * ctx->slot_capacity, hipMemcpyDeviceToDevice,
                       ctx->stream) != hipSuccess)
        result = fail(ISLF_EDEVICE, "state backup failed");
    auto restore = [&]() -> islf_status {
        for (int r : ctx->live)
            HIP_TRY(hipMemcpyAsync(ctx->reps[r].mem, backup[r], ctx->reps[r].mem_bytes, hipMemcpyDeviceToDevice,
                                   ctx->stream));
        HIP_TRY(hipMemcpyAsync(ctx->d_state, st_backup, sizeof(RepState) * ctx->slot_capacity,
                               hipMemcpyDeviceToDevice, ctx->stream));
        return ISLF_OK;
    };
    for (auto &cl : classes) {
        if (result != ISLF_OK) break;
        const int orig = ctx->reps[cl[0]].tile;
        // the fastest variant, if it beats the replica's own by 1%
        double best = 1e300, orig_ms = 1e300;
        int best_tile = orig;
        for (int tile = 0; tile < num_tiles_of(ctx->fmt) && result == ISLF_OK; ++tile) {
            double ms = 0;
            result = time_variant(ctx, cl, tile, sweeps, &ms);
            if (result == ISLF_OK) result = restore();
            if (result == ISLF_OK && tile == orig) orig_ms = ms;
            if (result == ISLF_OK && ms < best) {
                best = ms;
                best_tile = tile;
            }
        }
        if (best_tile != orig && orig_ms < 1e300 && best >= 0.99 * orig_ms) best_tile = orig;
        for (int r : cl) {
            ctx->reps[r].tile = (result == ISLF_OK) ? best_tile : orig;
            build_work(ctx->reps[r], r, ctx->fmt);
        }
    }
    if (result == ISLF_OK) {
        islf_status rs = restore();
        if (rs != ISLF_OK) result = rs;
    }
    // the launch configuration of the context's form on the whole batch:
    // batched: concurrent groups x workgroups per launch x share taper;
    // persistent: barrier form x grid (up to the co-residency bound) x taper.
    // Each trial captures `sweeps` sweeps as graphs and times replays of
    // them; the chains advance during the trials and are restored once
    // afterwards.  The resident form has none of these settings: whether it
    // is the faster one depends on a run's length, so each run decides, by
    // the time measured here.
    double tuned_ms = 0.0;
    if (result == ISLF_OK && !ctx->live.empty() &&
        (ctx->exec == ISLF_EXEC_BATCHED || ctx->exec == ISLF_EXEC_PERSISTENT)) {
        ctx->dirty = true;
        result = sync_tables(ctx);
        const int keep_groups = ctx->groups_req, keep_grid = ctx->grid_override;
        const double keep_taper = ctx->taper_override;
        struct Trial { int groups, grid; double taper; int team; };
        const int keep_team = ctx->team_mode;
        const bool chosen = config_chosen(ctx);
        ctx->chain_only = true;
        std::vector<Trial> trials;
        const double tapers[] = {0.0, 0.1, 0.2};
        if (ctx->exec == ISLF_EXEC_BATCHED) {
            const int nl = (int)ctx->live.size();
            for (int G = 1; G <= std::min(4, nl); ++G) {
                const int base = G == 1 ? ctx->sweep_slots : std::max(64, (3 * ctx->resident_slots + G) / (2 * G));
                for (double f : {0.5, 1.0, 1.5})
                    for (double tp : tapers) trials.push_back(Trial{G, std::max(32, (int)(base * f + 0.5)), tp, keep_team});
            }
        } else {
            // up to one workgroup per CU below the bound, like the default grid
            const int per_cu = std::max(1, ctx->persistent_bound / std::max(1, ctx->num_cu));
            const int top = std::max(1, per_cu - 1);
            // the persistent shares step down by dispatch round: stronger tapers
            for (int team = 0; team <= 1; ++team)
                for (int k = std::max(1, top - 2); k <= top; ++k)
                    for (double tp : {0.0, 0.2, 0.4, 0.6})
                        trials.push_back(Trial{0, std::min(ctx->num_cu * k, ctx->persistent_bound), tp, team});
        }
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (result == ISLF_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess))
            result = fail(ISLF_EDEVICE, "cannot create events");
        // one trial: the shortest of `runs` timed replays of a captured graph
        // of `sweeps` sweeps after one untimed replay (eager launches without
        // a stream to capture on)
        auto time_trial = [&](const Trial &t, int runs, float *best_ms) -> islf_status {
            ctx->groups_req = t.groups ? t.groups : keep_groups;
            ctx->grid_override = t.grid;
            ctx->taper_override = t.taper;
            ctx->team_mode = t.team;
            ctx->groups_valid = false;
            ctx->batched.valid = false;
            ctx->persistent.valid = false;
            islf_status rs = prepare_plans(ctx, ctx->exec);
            if (rs != ISLF_OK) return rs;
            hipError_t e = hipSuccess;
            int G = 1;
            if (ctx->stream) {
                rs = islf_graph_capture(ctx, sweeps);
                if (rs != ISLF_OK) return rs;
                G = (int)ctx->graph_execs.size();
            }
            for (int run = 0; run <= runs && e == hipSuccess; ++run) {
                if (run == 1) e = hipEventRecord(e0, ctx->stream);
                if (e == hipSuccess && ctx->stream) {
                    if (G > 1) e = fork_groups(ctx, G);
                    for (int g = 0; g < G && e == hipSuccess; ++g)
                        e = hipGraphLaunch(ctx->graph_execs[g], group_stream(ctx, g, G));
                    if (e == hipSuccess && G > 1) e = join_groups(ctx, G);
                } else if (e == hipSuccess) {
                    rs = enqueue_sweeps(ctx, run == 0 ? 1 : sweeps);
                    if (rs != ISLF_OK) break;
                }
                if (run >= 1 && e == hipSuccess) {
                    e = hipEventRecord(e1, ctx->stream);
                    if (e == hipSuccess) e = hipEventSynchronize(e1);
                    float ms = 0.f;
                    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
                    if (e == hipSuccess && (run == 1 || ms < *best_ms)) *best_ms = ms;
                    if (e == hipSuccess && run < runs) e = hipEventRecord(e0, ctx->stream);
                }
            }
            if (ctx->stream) destroy_graphs(ctx);
            if (rs != ISLF_OK) return rs;
            if (e != hipSuccess) return fail(ISLF_EDEVICE, "autotune trial failed: %s", hipGetErrorString(e));
            return ISLF_OK;
        };
        // first pass over every trial, then the fastest few and the entry
        // configuration again with more runs; the entry configuration stays
        // unless a finalist beats it by 1%
        const Trial entry{keep_groups, keep_grid, keep_taper, keep_team};
        std::vector<std::pair<float, size_t>> first;
        for (size_t i = 0; i < trials.size() && result == ISLF_OK; ++i) {
            float ms = 0.f;
            result = time_trial(trials[i], kTrialRuns, &ms);
            if (result == ISLF_OK) first.push_back({ms, i});
        }
        Trial best_t = entry;
        if (result == ISLF_OK) {
            std::sort(first.begin(), first.end());
            float entry_ms = 0.f;
            result = time_trial(entry, kFinalRuns, &entry_ms);
            float best = entry_ms;
            for (size_t k = 0; k < first.size() && (int)k < kFinalists && result == ISLF_OK; ++k) {
                float ms = 0.f;
                result = time_trial(trials[first[k].second], kFinalRuns, &ms);
                if (result == ISLF_OK && ms < best && ms < 0.99f * entry_ms) {
                    best = ms;
                    best_t = trials[first[k].second];
                }
            }
            tuned_ms = best;
        }
        ctx->chain_only = false;
        if (result == ISLF_OK) ctx->tuned = !chosen;
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        ctx->groups_req = (result == ISLF_OK && best_t.groups) ? best_t.groups : keep_groups;
        ctx->grid_override = result == ISLF_OK ? best_t.grid : keep_grid;
        ctx->taper_override = result == ISLF_OK ? best_t.taper : keep_taper;
        ctx->team_mode = result == ISLF_OK ? best_t.team : keep_team;
        ctx->groups_valid = false;
        ctx->batched.valid = false;
        ctx->persistent.valid = false;
        ctx->graph_valid = false;
        if (result == ISLF_OK) {
            islf_status rs = restore();
            if (rs != ISLF_OK) result = rs;
        }
    }
    if (hipStreamSynchronize(ctx->stream) != hipSuccess && result == ISLF_OK)
        result = fail(ISLF_EDEVICE, "autotune synchronisation failed");
    landed(ctx);
    for (void *b : backup) dev_free(ctx, b);
    dev_free(ctx, st_backup);
    ctx->dirty = true;
    if (result != ISLF_OK) return result;
    result = sync_tables(ctx);
    ctx->tuned_us = std::max(0.0, 1e3 * tuned_ms - kChainRunUs) / sweeps;
    ctx->tuned_exec = ctx->exec;
    return result;
}

// 32-bit words per (x, y) row of the spin array
static long profile_row_words(const Replica &R)
{
    return R.d.fmt == ISLF_SPIN_INT8 ? R.d.RB / 4 : 2l * R.d.Wq;
}

extern "C" islf_status islf_layer_profile(islf_ctx *ctx, int32_t rep, int32_t *dev_out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!dev_out) return fail(ISLF_EINVAL, "NULL output");
    if (ctx->reps[rep].failed)
        return fail(ISLF_ESTATE, "replica %d was cut short by a failed launch", rep);
    st = sync_tables(ctx);
    if (st != ISLF_OK) return st;
    const Replica &R = ctx->reps[rep];
    HIP_TRY(launch_layer_profile(ctx->d_desc, rep, (long)R.desc.Lx * R.desc.Ly, profile_row_words(R), dev_out,
                                 nullptr, ctx->stream));
    return ISLF_OK;
}

extern "C" islf_status islf_layer_profile_add(islf_ctx *ctx, int32_t rep, int64_t *dev_acc)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!dev_acc) return fail(ISLF_EINVAL, "NULL accumulator");
    if (ctx->reps[rep].failed)
        return fail(ISLF_ESTATE, "replica %d was cut short by a failed launch", rep);
    st = sync_tables(ctx);
    if (st != ISLF_OK) return st;
    const Replica &R = ctx->reps[rep];
    HIP_TRY(launch_layer_profile(ctx->d_desc, rep, (long)R.desc.Lx * R.desc.Ly, profile_row_words(R), nullptr,
                                 (long long *)dev_acc, ctx->stream));
    return ISLF_OK;
}

extern "C" islf_status islf_set_grid(islf_ctx *ctx, int32_t workgroups)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (workgroups < 0 || workgroups > (1 << 20)) return fail(ISLF_EINVAL, "invalid workgroup count %d", workgroups);
    if (ctx->exec == ISLF_EXEC_PERSISTENT && workgroups > ctx->persistent_bound)
        return fail(ISLF_ERANGE, "persistent grid %d exceeds the co-residency bound %d of this device", workgroups,
                    ctx->persistent_bound);
    ctx->grid_override = workgroups;
    ctx->tuned = false;
    ctx->batched.valid = false;
    ctx->persistent.valid = false;
    ctx->groups_valid = false;
    for (Plan &p : ctx->plain) p.valid = false;
    ctx->graph_valid = false;
    return ISLF_OK;
}

extern "C" islf_status islf_set_groups(islf_ctx *ctx, int32_t groups)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (groups < 0 || groups > kMaxStreamGroups) return fail(ISLF_EINVAL, "invalid group count %d", groups);
    ctx->groups_req = groups;
    ctx->tuned = false;
    ctx->groups_valid = false;
    ctx->graph_valid = false;
    return ISLF_OK;
}

extern "C" islf_status islf_get_groups(const islf_ctx *ctx, int32_t *groups)
{
    if (!ctx || !groups) return fail(ISLF_EINVAL, "NULL argument");
    *groups = num_groups(ctx);
    return ISLF_OK;
}

extern "C" islf_status islf_get_grid(const islf_ctx *ctx, int32_t *workgroups)
{
    if (!ctx || !workgroups) return fail(ISLF_EINVAL, "NULL argument");
    if (ctx->exec == ISLF_EXEC_PERSISTENT)
        *workgroups = ctx->grid_override ? ctx->grid_override : ctx->persistent_grid;
    else
        *workgroups = launch_grid(ctx, ctx->exec);
    return ISLF_OK;
}

extern "C" islf_status islf_phase_timings(islf_ctx *ctx, uint32_t n_sweeps, double *mean_ms, uint32_t *launches)
{
    if (!ctx || !mean_ms || !launches) return fail(ISLF_EINVAL, "NULL argument");
    if (n_sweeps < 1) return fail(ISLF_EINVAL, "n_sweeps must be >= 1");
    islf_status st = sync_tables(ctx);
    if (st == ISLF_OK && !ctx->batched.valid && !ctx->live.empty()) {
        std::vector<Entry> S, M;
        for (int r : ctx->live) {
            S.insert(S.end(), ctx->reps[r].slab.begin(), ctx->reps[r].slab.end());
            M.insert(M.end(), ctx->reps[r].main.begin(), ctx->reps[r].main.end());
        }
        st = build_plan(ctx, ctx->batched, S, M, ctx->grid_override ? ctx->grid_override : ctx->sweep_slots);
    }
    if (st != ISLF_OK) return st;
    st = check_sweep_range(ctx, n_sweeps);
    if (st != ISLF_OK) return st;
    const int nl = (int)ctx->live.size();
    std::vector<hipEvent_t> ev(4 * (size_t)n_sweeps + 2, nullptr);
    for (auto &e : ev)
        if (hipEventCreate(&e) != hipSuccess) {
            for (auto &f : ev)
                if (f) (void)hipEventDestroy(f);
            return fail(ISLF_EDEVICE, "cannot create events");
        }
    bool mark = false;
    hipError_t err;
    {
        std::lock_guard<std::mutex> lock(turns(ctx).m);
        err = start_chain(ctx, false, &mark);
    }
    if (err == hipSuccess && nl) err = enqueue_plan(ctx, ctx->batched, ctx->d_live, nl, n_sweeps, ev.data());
    if (err == hipSuccess) err = end_chain(ctx, mark);
    if (err == hipSuccess) err = hipStreamSynchronize(ctx->stream);
    if (err == hipSuccess) landed(ctx);
    double sum[3] = {0, 0, 0};
    uint32_t cnt[3] = {0, 0, 0};
    if (err == hipSuccess && nl) {
        for (size_t k = 0; k <= 2 * (size_t)n_sweeps; ++k) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev[2 * k], ev[2 * k + 1]) != hipSuccess) continue;
            const int kind = k == 2 * (size_t)n_sweeps ? 2 : (int)(k & 1);
            sum[kind] += ms;
            cnt[kind] += 1;
        }
    }
    for (auto &e : ev) (void)hipEventDestroy(e);
    if (err != hipSuccess) return fail(ISLF_EDEVICE, "timed sweeps failed: %s", hipGetErrorString(err));
    for (int r : ctx->live) ctx->reps[r].t_host += n_sweeps;
    for (int k = 0; k < 3; ++k) {
        mean_ms[k] = cnt[k] ? sum[k] / cnt[k] : 0.0;
        launches[k] = cnt[k];
    }
    return ISLF_OK;
}

extern "C" islf_status islf_replica_means(islf_ctx *ctx, int32_t rep, uint64_t first, uint32_t count, double *out)
{
    islf_status st = check_rep(ctx, rep);
    if (st != ISLF_OK) return st;
    if (!out) return fail(ISLF_EINVAL, "NULL output");
    st = check_records(ctx, rep, first, count);
    if (st != ISLF_OK) return st;
    // its entry in the list of live replicas (which only an addition or a retirement changes)
    const long i = std::lower_bound(ctx->live.begin(), ctx->live.end(), (int)rep) - ctx->live.begin();
    HIP_TRY(launch_means(ctx->d_desc, ctx->d_live + i, 1, first, count, (double *)(ctx->h_res + 8), ctx->stream));
    st = fetch(ctx, rep);
    if (st == ISLF_OK) memcpy(out, ctx->h_res + 8, 5 * sizeof(double));
    return st;
}

extern "C" islf_status islf_device_bytes(const islf_ctx *ctx, uint64_t *total, uint64_t *replica_bytes)
{
    if (!ctx || !total) return fail(ISLF_EINVAL, "NULL argument");
    *total = (uint64_t)ctx->dev_bytes;
    if (replica_bytes) {
        uint64_t r = 0;
        for (const Replica &R : ctx->reps)
            if (R.mem) r += R.mem_bytes;
        *replica_bytes = r;
    }
    return ISLF_OK;
}

// Test support, not part of the public header: raises the persistent
// kernel's error word from the host, as a block that gave up at a grid
// barrier would, so that the failure path can be exercised without a launch
// that really fails.  Every block of the next persistent launch then stops
// at its first barrier.
extern "C" islf_status islf_testing_raise_barrier_error(islf_ctx *ctx)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    const unsigned long long one = 1;
    HIP_TRY(hipMemcpyAsync(&ctx->d_sync->error.v, &one, sizeof one, hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return ISLF_OK;
}

// Test support, not part of the public header: puts the resident form's state
// word to aborted, as a launch whose workgroups did not all become resident
// would, so that the next launch's closing kernel sweeps its cluster replicas.
extern "C" islf_status islf_testing_abort_resident(islf_ctx *ctx)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    const unsigned int v = RES_ABORT;
    HIP_TRY(hipMemcpyAsync(&ctx->d_rsy->state, &v, sizeof v, hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return ISLF_OK;
}

// Test support, not part of the public header: whether a run of n sweeps would
// take the resident form now.
extern "C" islf_status islf_testing_takes_resident(islf_ctx *ctx, uint32_t n, int32_t *takes)
{
    if (!ctx || !takes) return fail(ISLF_EINVAL, "NULL argument");
    bool use = false;
    const islf_status st = resident_applies(ctx, n, &use);
    *takes = use ? 1 : 0;
    return st;
}

// Test support, not part of the public header: runs with clusters, runs of the
// chain, launches called off by the census, runs still kept to the chain.
extern "C" islf_status islf_testing_runs(const islf_ctx *ctx, uint64_t out[4])
{
    if (!ctx || !out) return fail(ISLF_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lock(turns(ctx).m);
    out[0] = ctx->cluster_runs;
    out[1] = ctx->chain_runs;
    out[2] = ctx->h_res[HOST_ABORTS];
    out[3] = (uint64_t)ctx->apart;
    return ISLF_OK;
}

// Test support, not part of the public header: the plan of a resident launch
// over n films on a device of num_cu CUs, built on the host, as a list of
// int32: form, grid, jobs, mailbox words; then per job its replica, shares,
// id, workgroup, rows, words of a row, whole ones, groups of the last one,
// has, in, slot, out_y, out_x, planes (count, x of each), row sets (count, y of
// each, chunks of whole and of partial words) and stages (count, parts (set,
// phase, c0, c1) and the phases taken in).  *len: the words there are (0: no
// plan); at most `room` are written.
extern "C" islf_status islf_testing_resident_plan(const islf_replica_desc *descs, int32_t n, int32_t spin_format,
                                                  int32_t num_cu, int32_t *out, int64_t room, int64_t *len)
{
    if (!descs || n < 1 || !len || (room > 0 && !out)) return fail(ISLF_EINVAL, "NULL argument");
    *len = 0;
    islf_ctx c;
    c.fmt = spin_format;
    c.num_cu = num_cu;
    std::vector<int> reps(n);
    c.reps.resize(n);
    for (int i = 0; i < n; ++i) {
        const islf_status st = validate(&descs[i]);
        if (st != ISLF_OK) return st;
        c.reps[i].desc = descs[i];
        reps[i] = i;
    }
    ResPlan p;
    ResTablesHost h;
    if (!plan_resident(&c, reps, p, h)) return ISLF_OK;
    std::vector<int32_t> v = {p.form, p.L.grid, p.L.njobs, (int32_t)h.mbox_words};
    for (int w = 0; w < p.L.grid; ++w)
        for (int q = h.first[w]; q < h.first[w + 1]; ++q) {
            const ResJob &j = h.jobs[q];
            const islf_replica_desc &d = descs[j.rep];
            const int np = j.n1 + j.n2;
            v.insert(v.end(), {j.rep, j.P, j.id, w, j.R, (d.Lz + 63) / 64, j.Wf, j.ng, j.has, (int32_t)j.in,
                               (int32_t)j.slot, (int32_t)j.out_y[0], (int32_t)j.out_y[1], (int32_t)j.out_x[0],
                               (int32_t)j.out_x[1], np});
            for (int k = 0; k < np; ++k) v.push_back(h.planes[j.planes + k].x);
            for (const ResRows &r : j.set) {
                v.push_back(r.n);
                for (int k = 0; k < r.n; ++k) v.push_back(h.rows[j.rows + r.r0 + k].y);
                v.push_back(r.whole);
                v.push_back(r.part);
            }
            v.push_back(j.stages);
            for (int t = 0; t < j.stages; ++t) {
                for (const ResPart &r : j.stage[t].part) v.insert(v.end(), {r.set, r.phase, r.c0, r.c1});
                v.push_back(j.stage[t].mail);
                v.push_back(j.stage[t].mail_row0);
            }
        }
    *len = (int64_t)v.size();
    std::copy(v.begin(), v.begin() + std::min<int64_t>(*len, room), out);
    return ISLF_OK;
}

extern "C" islf_status islf_set_taper(islf_ctx *ctx, double taper)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (!(taper < 1.0)) return fail(ISLF_EINVAL, "taper must be below 1 (got %g)", taper);
    ctx->taper_override = taper < 0.0 ? -1.0 : taper;
    ctx->tuned = false;
    ctx->batched.valid = false;
    ctx->persistent.valid = false;
    ctx->groups_valid = false;
    ctx->graph_valid = false;
    return ISLF_OK;
}

extern "C" islf_status islf_get_taper(const islf_ctx *ctx, double *taper)
{
    if (!ctx || !taper) return fail(ISLF_EINVAL, "NULL argument");
    if (ctx->taper_override >= 0.0) *taper = ctx->taper_override;
    else if (ctx->exec == ISLF_EXEC_PERSISTENT)
        *taper = kPersistentTaper;
    else *taper = tail_taper(ctx->fmt);
    return ISLF_OK;
}

extern "C" islf_status islf_set_barriers(islf_ctx *ctx, int32_t mode)
{
    if (!ctx) return fail(ISLF_EINVAL, "NULL context");
    if (mode != ISLF_BARRIER_GRID && mode != ISLF_BARRIER_TEAM && mode != ISLF_BARRIER_AUTO)
        return fail(ISLF_EINVAL, "invalid barrier mode %d", mode);
    ctx->team_mode = mode == ISLF_BARRIER_TEAM ? 1 : mode == ISLF_BARRIER_GRID ? 0 : -1;
    ctx->tuned = false;
    ctx->persistent.valid = false;
    ctx->graph_valid = false;
    return ISLF_OK;
}

extern "C" islf_status islf_get_barriers(const islf_ctx *ctx, int32_t *mode)
{
    if (!ctx || !mode) return fail(ISLF_EINVAL, "NULL argument");
    // the form the next persistent launch uses
    const int grid = ctx->grid_override ? ctx->grid_override : ctx->persistent_grid;
    *mode = use_teams(ctx, grid) ? ISLF_BARRIER_TEAM : ISLF_BARRIER_GRID;
    return ISLF_OK;
}
