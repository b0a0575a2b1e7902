// Host engine of libfciqmc: the C ABI declared in include/fciqmc.h.
//
// A handle holds up to max_slots independent systems. Each system owns a main
// list in device memory, hash-partitioned into buckets of at most 256 packed
// entries (structure of arrays: determinant, population, stored diagonal
// element, plus a count per bucket), its integrals, and a row of the device
// descriptor table. One iteration of every system is one pass of the kernels
// over the descriptor table; up to 64 iterations are captured in one HIP graph.
// Between launches the host reads the per-iteration records, feeds the
// estimator averages, and re-buckets a list whose buckets would fill up, or
// gives its buckets more record slots. An iteration whose records overflowed a
// bucket's slots is abandoned and re-run with more (the counter-based random
// numbers make the re-run identical); new determinants that did not fit their
// bucket complete the iteration in a spill list and are re-bucketed before the
// system continues.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/fciqmc.h"
#include "engine.h"

using namespace fq;

// Determinants on the host: one 128-bit integer (bit p: spin orbital p occupied).
// The API and the device hold W = 1 or 2 64-bit words per determinant, low word
// first (Sec. 3: as many words as the spin orbitals need).
typedef unsigned __int128 hdet_t;
static inline int hpopc(hdet_t x) {
    return __builtin_popcountll((uint64_t)x) + __builtin_popcountll((uint64_t)(x >> 64));
}
static inline hdet_t hbit(int p) { return (hdet_t)1 << p; }
static inline uint64_t hlo(hdet_t x) { return (uint64_t)x; }
static inline uint64_t hhi(hdet_t x) { return (uint64_t)(x >> 64); }
static inline hdet_t hdet_in(const uint64_t *w, int W) {
    return W > 1 ? (((hdet_t)w[1] << 64) | (hdet_t)w[0]) : (hdet_t)w[0];
}
static inline void hdet_out(hdet_t d, uint64_t *w, int W) {
    w[0] = hlo(d);
    if (W > 1) w[1] = hhi(d);
}
static const hdet_t HEVEN = ((hdet_t)0x5555555555555555ull << 64) | (hdet_t)0x5555555555555555ull;
// Words per determinant for a system of n_orb spatial orbitals (det_words: 0 as needed,
// 2 forced).
static inline int words_for(int n_orb, int det_words) {
    return (2 * n_orb > 64 || det_words == 2) ? 2 : 1;
}
// The kernels' launchers of the handle's width.
#define FQ_LAUNCH(W, fn, ...) ((W) == 2 ? fq::w2::fn(__VA_ARGS__) : fq::fn(__VA_ARGS__))

// Device staging area of fciqmc_walkers_noalloc (every call on a GPU shares
// that GPU's copy). Host code never uses this name as an address: the address
// of each device's copy is taken once per device with hipGetSymbolAddress when
// the first handle on that device is created, and passed to the kernels.
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

namespace {

thread_local std::string g_err;

int set_err(int code, const std::string &msg) {
    g_err = msg;
    return code;
}

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return set_err(FCIQMC_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

// Main-list capacities: a multiple of 4 buckets, at least 4 buckets.
int64_t round_cap(int64_t x) {
    const int64_t q = 4 * CHUNK;
    return std::max<int64_t>(q, (x + q - 1) / q * q);
}

// Main-list capacity for `entries` entries at the planned mean bucket fill.
int64_t cap_for_entries(int64_t entries) {
    return round_cap((std::max<int64_t>(entries, 1) + BUCKET_FILL - 1) / BUCKET_FILL * BQ);
}

int64_t next_pow2(int64_t x) {
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

// ---------------------------------------------------------------------------
// Error bars of correlated averages by blocking (Flyvbjerg & Petersen, the
// analysis of correlated ratios the paper's conclusions cite), kept online in
// O(log n) memory. Level 0 receives every sample (x, y); each completed pair at
// level l is averaged and passed to level l + 1, so level l sees the first
// floor(n / 2^l) block means. Per level the accumulators hold sums of the
// deviations from the level's first value (dx = x - x_first, ...): dx, dy,
// dx^2, dy^2 and dx dy, from which the level's means, variances of the mean and
// covariance follow. The error of the ratio <x>/<y> is the standard error of the
// linearised ratio estimator, sqrt(var(xbar - r ybar)) / ybar with r = xbar/ybar;
// a plain mean is the case y = 1. The level reported is the first one with at
// least 16 blocks whose error the next two levels (with >= 16 blocks) do not
// exceed by more than the error's own relative uncertainty 1/sqrt(2(n - 1));
// when none qualifies, the deepest level with >= 16 blocks.
// ---------------------------------------------------------------------------
class Blocker {
  public:
    void clear() { *this = Blocker(); }
    int64_t count() const { return lev_[0].n; }

    void add(double x, double y) {
        for (int l = 0; l < kLevels; ++l) {
            Level &L = lev_[l];
            if (L.n == 0) {
                L.x0 = x;
                L.y0 = y;
            }
            const double dx = x - L.x0, dy = y - L.y0;
            L.sx += dx;
            L.sy += dy;
            L.sxx += dx * dx;
            L.syy += dy * dy;
            L.sxy += dx * dy;
            L.n += 1;
            if (!L.pending) {
                L.pending = true;
                L.px = x;
                L.py = y;
                return;
            }
            L.pending = false;
            x = (L.px + x) * 0.5;
            y = (L.py + y) * 0.5;
        }
    }

    // Mean of x / mean of y over all samples, and its error bar (NaN when no
    // level has 16 blocks).
    void result(double &mean, double &err) const {
        mean = NAN;
        err = NAN;
        const Level &L0 = lev_[0];
        if (L0.n == 0) return;
        mean = (L0.x0 + L0.sx / (double)L0.n) / (L0.y0 + L0.sy / (double)L0.n);
        double e[kLevels];
        int top = 0;   // levels with >= 16 blocks: 0 .. top-1
        while (top < kLevels && lev_[top].n >= 16) {
            e[top] = level_error(lev_[top]);
            ++top;
        }
        if (top == 0) return;
        int pick = top - 1;
        for (int l = 0; l < top; ++l) {
            const double allow = e[l] * (1.0 + 1.0 / std::sqrt(2.0 * (double)(lev_[l].n - 1)));
            const bool next_ok = l + 1 >= top || e[l + 1] <= allow;
            const bool next2_ok = l + 2 >= top || e[l + 2] <= allow;
            if (next_ok && next2_ok) {
                pick = l;
                break;
            }
        }
        err = e[pick];
    }

  private:
    static constexpr int kLevels = 64;
    struct Level {
        int64_t n = 0;
        double x0 = 0, y0 = 0, sx = 0, sy = 0, sxx = 0, syy = 0, sxy = 0;
        bool pending = false;
        double px = 0, py = 0;
    };
    static double level_error(const Level &L) {
        const double n = (double)L.n;
        const double norm = n * (n - 1.0);
        const double vx = (L.sxx - L.sx * L.sx / n) / norm;
        const double vy = (L.syy - L.sy * L.sy / n) / norm;
        const double cxy = (L.sxy - L.sx * L.sy / n) / norm;
        const double xbar = L.x0 + L.sx / n, ybar = L.y0 + L.sy / n;
        const double r = xbar / ybar;
        const double v = (vx - 2.0 * r * cxy + r * r * vy) / (ybar * ybar);
        return std::sqrt(v > 0.0 ? v : 0.0);
    }
    Level lev_[kLevels];
};

struct SysHost {
    bool active = false;
    fciqmc_params prm{};
    int M = 0, N = 0, na = 0, nb = 0;
    std::vector<double> h1, eri;
    std::vector<uint8_t> irrep;
    double e_core = 0.0, p_double = 0.0, e0 = 0.0;
    hdet_t d0 = 0;
    int W = 1;                 // 64-bit words per determinant
    int64_t cap = 0;           // main-list capacity: buckets * BQ
    void *block = nullptr;     // one device allocation for the main list + integrals
    uint64_t *key = nullptr;   // W words per entry
    int32_t *pop = nullptr;
    double *hd = nullptr;
    int32_t *bcnt = nullptr;
    double *d_h1 = nullptr, *d_eri = nullptr, *d_jk = nullptr;
    std::vector<double> jk;    // [n_so][64 W] pair table
    std::vector<double> t3;    // [n_so][64 W][64 W] single-excitation term table
    double *d_t3 = nullptr;
    std::vector<uint16_t> bound;   // [32 W][32 W] rejection bounds (SysDesc::bound)
    uint16_t *d_bound = nullptr;
    int64_t growth = 0;        // expected per-iteration increase of the entries
    double spawn_rate = 1.0;   // mean growth of the records per iteration in the last launch
    int64_t rec_r = 0;         // record slots per bucket
    bool crowded = false;      // few buckets hold most records: those get extensions,
    bool counted = false;      // from the last iteration's counts, if there are any
    double ext_factor = 1.0;   // slots per record of it
    bool no_split = false;     // no room for buckets planned by their records
    int64_t rec_peak = 0;      // most records of one bucket in the last launch (0: unknown)
    double h_max = 0.0;        // scale of the largest off-diagonal elements
    int64_t pop_max = 0;       // largest |C| of the list as loaded
    int64_t reserve_bytes = 0; // admission accounting (target footprint)
    // mirrored dynamics and statistics
    IterRecord last{};
    int64_t tot_att = 0, tot_sp = 0;
    int64_t redos = 0;         // iterations re-run after the record buffer overflowed
    int64_t spills = 0;        // iterations whose new determinants overflowed a bucket
    Blocker e_blk, s_blk;      // (num, C_0) and (S, 1) samples of the averaging window
    int fatal = 0;
};

}  // namespace

struct fciqmc_t {
    int dev = 0;
    int W = 1;                              // words per determinant of every system here
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int max_sys = 0;
    std::vector<SysHost> sys;
    std::vector<SysDesc> hdesc;
    SysDesc *d_desc = nullptr;
    IterRecord *d_rec = nullptr;            // per-iteration records: pinned host memory that
    IterRecord *h_rec = nullptr;            // k_finalize writes through d_rec, read as h_rec
    uint32_t *d_status = nullptr;           // per system ST_* bits (device)
    unsigned int *d_work = nullptr;         // dynamic work counters
    unsigned long long *d_spawns = nullptr; // per system spawn counter (device)
    std::vector<uint32_t> hstatus;          // host mirror of d_status
    std::vector<IterRecord> hrec;
    // global chunk layout
    int64_t chunk_alloc = 0, n_chunks = 0;
    int32_t *d_chunk_sys = nullptr, *d_chunk_local = nullptr;
    unsigned long long *d_total = nullptr;  // lengths of the tile lists
    uint32_t *d_unlisted = nullptr;         // buckets whose tiles did not fit
    int32_t *d_tiles = nullptr;             // the spawn tiles, 16 B each
    bool tile_map_off = false;              // its allocation failed once: whole buckets instead
    void *d_stage = nullptr;                // this device's staging area (not owned)
    // spawn records (see EngineArgs) and the spill list
    void *d_recs = nullptr;
    int64_t rec_cap = 0;                    // slots allocated
    int64_t rec_floor = 65536;              // slots a system's buckets share at least
    uint32_t *d_bhist = nullptr, *d_rec_max = nullptr, *d_bprev = nullptr;
    uint64_t *d_bext = nullptr;
    int64_t rec_base = 0;                   // slots in use before the extensions
    bool ext_on = false;                    // some bucket may have an extension
    long long *d_d0acc = nullptr;
    void *d_spill = nullptr;
    int64_t sp_cap = 0;
    unsigned long long *d_sp_count = nullptr;
    uint32_t *d_spilled = nullptr;
    int64_t tile_cap = 0;
    unsigned long long *d_step = nullptr;   // iterations run (its parity selects d_total)
    IterStat *d_acc = nullptr;              // [max_sys][ACC_SLOTS]
    int64_t *d_c0 = nullptr;                // [max_sys]
    int64_t *d_nchunks = nullptr;
    uint32_t *d_err = nullptr;
    unsigned long long *d_count = nullptr;
    int spawn_grid = 2048;
    int post_grid = 1024;
    int tile = 2048;
    bool shape_set = false;                 // the launch shape was set or tuned: used as it is
    struct Graph {
        hipGraphExec_t exec;
        int64_t used;                       // when it was last launched
    };
    std::map<std::array<int, 6>, Graph> graphs;   // by iterations, kernel variant, shape
    int64_t graph_clock = 0;
    bool use_graph = true;
    bool profiling = false;
    hipEvent_t ev[NKERN + 1] = {};
    double kms[NKERN] = {};
    int64_t kcount[NKERN] = {};
    double phase_ms[NKERN] = {};            // kernel groups of the last sampled iteration
    double ms_last = 0.0;
    bool planner = true;                    // size tables before each launch (test knob)
    int64_t tile_map_limit = -1;            // cap on the tile map (test knob; -1: none)
};

namespace {

void drop_graphs(fciqmc_t *h) {
    for (auto &kv : h->graphs) (void)hipGraphExecDestroy(kv.second.exec);
    h->graphs.clear();
}

EngineArgs make_args(fciqmc_t *h) {
    EngineArgs a{};
    a.desc = h->d_desc;
    a.max_sys = h->max_sys;
    a.chunk_sys = h->d_chunk_sys;
    a.chunk_local = h->d_chunk_local;
    a.step = h->d_step;
    a.acc = h->d_acc;
    a.c0 = h->d_c0;
    a.total = h->d_total;
    a.nchunks = h->d_nchunks;
    a.rec = h->d_rec;
    a.status = h->d_status;
    a.spawns = h->d_spawns;
    a.work = h->d_work;
    a.tiles = h->d_tiles;
    a.list_cap = h->tile_cap / NLIST;
    a.unlisted = h->d_unlisted;
    a.recs = (SpawnRec *)h->d_recs;
    a.bhist = h->d_bhist;
    a.bprev = h->d_bprev;
    a.bext = h->d_bext;
    a.rec_max = h->d_rec_max;
    a.d0acc = h->d_d0acc;
    char *q = (char *)h->d_spill;
    const size_t sc = (size_t)h->sp_cap;
    const size_t kb = 8 * (size_t)h->W;      // bytes per determinant
    a.sp_det = (uint64_t *)q;
    a.sp_hd = (double *)(q + kb * sc);
    a.sp_pop = (int32_t *)(q + (kb + 8) * sc);
    a.sp_sys = (int32_t *)(q + (kb + 12) * sc);
    a.sp_count = h->d_sp_count;
    a.sp_cap = h->sp_cap;
    a.spilled = h->d_spilled;
    a.plain = 1;
    for (int s = 0; s < h->max_sys; ++s) {
        const SysDesc &d = h->hdesc[s];
        if (h->sys[s].active && (d.n_class != 2 || d.hphf || d.space)) a.plain = 0;
    }
    return a;
}

// The launch shape of the next iterations: log2 of a wavefront's spawn tile, workgroups
// of k_spawn and of k_post. A shape set by the caller or tuned is used as it is (a
// workgroup's tile in four, one part per wavefront, of at most 512 attempts). By default a launch too small to
// give every wavefront of the chip a tile gets smaller tiles, down to one attempt per
// lane, and no more workgroups than there are tiles and chunks: a walk of few attempts
// is all latency (a tile's staging and its lanes' runs of attempts one after another),
// and idle workgroups still cost their start. Powers of two, so that a growing list
// meets few shapes (each is captured once).
// post_seg: chunks whose new determinants fill about two thirds of k_post's queue, by the
// fastest-growing list's last iteration (at most a whole window).
struct Shape {
    int wsh, spawn_grid, post_grid, post_seg;
};
Shape launch_shape(const fciqmc_t *h) {
    Shape o{std::clamp((int)std::log2((double)h->tile) - 2, 6, TILE_MAX_SH(h->W)), h->spawn_grid,
            h->post_grid, 32};
    for (int s = 0; s < h->max_sys; ++s) {
        const SysHost &S = h->sys[s];
        if (!S.active || S.fatal) continue;
        while (o.post_seg > 1 && S.last.born * o.post_seg > 700 * (S.cap / CHUNK)) o.post_seg /= 2;
    }
    if (h->shape_set) return o;
    int64_t walkers = 0;
    for (int s = 0; s < h->max_sys; ++s)
        if (h->sys[s].active && !h->sys[s].fatal) walkers += std::max<int64_t>(h->sys[s].last.nw, 0);
    const int64_t waves = 4 * (int64_t)h->spawn_grid;
    while (o.wsh > 6 && (walkers >> o.wsh) < waves) --o.wsh;
    // Two tiles for each of the grid's wavefronts, but not more than two for a bucket (each
    // stages its bucket again): with one, lists whose walkers sit on few determinants gave
    // some wavefronts three full tiles and others next to nothing (8 electrons in 20 orbitals,
    // half of 3e6 walkers on the reference: 219 -> 179 us an iteration; a ring of 14 sites, 90
    // walkers a bucket, would go from 140 to 160).
    const int64_t per_bucket = walkers / std::max<int64_t>(BPC * h->n_chunks, 1);
    while (o.wsh > 6 && (walkers >> o.wsh) < 2 * waves && per_bucket >> o.wsh) --o.wsh;
    const int64_t tiles = std::min<int64_t>(BPC * h->n_chunks, walkers) + (walkers >> o.wsh);
    o.spawn_grid = (int)std::min<int64_t>(o.spawn_grid, next_pow2(std::max<int64_t>(1, (tiles + 3) / 4)));
    o.post_grid = (int)std::min<int64_t>(o.post_grid, next_pow2(std::max<int64_t>(1, h->n_chunks)));
    return o;
}

// The spawn-record buffer for `cap` records (16 W B each). The old one is given back first
// (its records are dead, and there is seldom room for both); on failure there is none, until
// plan_launch, before the next launch, asks again.
int ensure_records(fciqmc_t *h, int64_t cap) {
    if (cap <= h->rec_cap) return 0;
    HIP_TRY(hipStreamSynchronize(h->stream));
    hipFree(h->d_recs);
    h->d_recs = nullptr;
    h->rec_cap = 0;
    drop_graphs(h);
    if (hipMalloc(&h->d_recs, (size_t)cap * (16 * h->W)) != hipSuccess) {
        (void)hipGetLastError();
        return set_err(FCIQMC_ENOMEM, "spawn-record buffer of " + std::to_string(cap) +
                                          " records does not fit in device memory");
    }
    h->rec_cap = cap;
    return 0;
}

// Slots per bucket are kept at a multiple of 8: a bucket's records then begin on a
// 128-byte line.
int64_t round_slots(double x) { return ((int64_t)std::ceil(x) + 7) / 8 * 8; }

// Fewest record slots per bucket worth having: a small list's buckets share rec_floor
// slots (early iterations multiply a handful of records), a large list's have 24 each.
int64_t min_slots(const fciqmc_t *h, int64_t nbuckets) {
    const int64_t share = h->rec_floor / std::max<int64_t>(nbuckets, 1);
    return round_slots((double)std::max<int64_t>(24, std::min<int64_t>(share, 1024)));
}

// A list of more buckets than before (old_nb) keeps its slots in all, not per bucket, until
// the next launch is planned: the few buckets of a list that starts on the reference have
// thousands each.
void share_slots(const fciqmc_t *h, SysHost &S, int64_t old_nb) {
    const int64_t nb = S.cap / BQ;
    if (!h->planner || S.rec_r <= 0 || nb <= old_nb) return;
    S.rec_r = std::max(min_slots(h, nb), round_slots((double)S.rec_r * (double)old_nb / (double)nb));
}

// Lay the active systems' record slots out one after another, each system's at its own
// count per bucket; the buffer grows when they need more.
int layout_records(fciqmc_t *h) {
    int64_t at = 0;
    for (int s = 0; s < h->max_sys; ++s) {
        SysHost &S = h->sys[s];
        if (!S.active) continue;
        if (S.rec_r <= 0) S.rec_r = min_slots(h, S.cap / BQ);
        h->hdesc[s].rec0 = at;
        h->hdesc[s].rec_r = S.rec_r;
        at += S.cap / BQ * S.rec_r;
    }
    h->rec_base = at;
    if (at > h->rec_cap) return ensure_records(h, std::max<int64_t>(at, h->rec_cap + h->rec_cap / 4));
    return 0;
}

int upload_desc(fciqmc_t *h) {
    HIP_TRY(hipMemcpyAsync(h->d_desc, h->hdesc.data(), sizeof(SysDesc) * h->max_sys,
                           hipMemcpyHostToDevice, h->stream));
    HIP_TRY(hipMemcpyAsync(h->d_status, h->hstatus.data(), sizeof(uint32_t) * h->max_sys,
                           hipMemcpyHostToDevice, h->stream));
    return 0;
}

int download_desc(fciqmc_t *h) {
    HIP_TRY(hipMemcpyAsync(h->hdesc.data(), h->d_desc, sizeof(SysDesc) * h->max_sys,
                           hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipMemcpyAsync(h->hstatus.data(), h->d_status, sizeof(uint32_t) * h->max_sys,
                           hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return 0;
}

// Clear what spawning accumulates for system s outside the records (its event
// count and its walkers onto the reference): after an abandoned iteration or a load.
int reset_spawns(fciqmc_t *h, int s) {
    HIP_TRY(hipMemsetAsync(h->d_spawns + (int64_t)s * SPAWN_SLOTS, 0,
                           SPAWN_SLOTS * sizeof(unsigned long long), h->stream));
    HIP_TRY(hipMemsetAsync(h->d_d0acc + s, 0, sizeof(long long), h->stream));
    return 0;
}

// Lay the chunks of all active systems out contiguously.
int relayout(fciqmc_t *h) {
    int64_t total = 0;
    for (int s = 0; s < h->max_sys; ++s)
        if (h->sys[s].active) total += h->sys[s].cap / CHUNK;
    if (total > h->chunk_alloc) {
        const int64_t na = next_pow2(std::max<int64_t>(total, 64));
        const struct {
            void **p;
            size_t bytes;
        } arrays[] = {{(void **)&h->d_chunk_sys, na * sizeof(int32_t)},
                      {(void **)&h->d_chunk_local, na * sizeof(int32_t)},
                      {(void **)&h->d_unlisted, BPC * na * sizeof(uint32_t)},
                      {(void **)&h->d_bhist, BPC * na * sizeof(uint32_t)},
                      {(void **)&h->d_bprev, BPC * na * sizeof(uint32_t)},
                      {(void **)&h->d_bext, BPC * na * sizeof(uint64_t)}};
        drop_graphs(h);
        h->chunk_alloc = 0;   // (without them plan_launch lays out again before a launch)
        for (const auto &x : arrays) {
            hipFree(*x.p);
            *x.p = nullptr;
        }
        for (const auto &x : arrays)
            if (hipMalloc(x.p, x.bytes) != hipSuccess) {
                (void)hipGetLastError();
                return set_err(FCIQMC_ENOMEM, "the maps of " + std::to_string(total) +
                                                  " chunks do not fit in device memory");
            }
        h->chunk_alloc = na;
    }
    // record counts start at zero (k_post keeps them so after every iteration)
    HIP_TRY(hipMemsetAsync(h->d_bhist, 0, BPC * h->chunk_alloc * sizeof(uint32_t), h->stream));
    // (the buckets are others now: their counts and extensions are void)
    HIP_TRY(hipMemsetAsync(h->d_bprev, 0, BPC * h->chunk_alloc * sizeof(uint32_t), h->stream));
    HIP_TRY(hipMemsetAsync(h->d_bext, 0, BPC * h->chunk_alloc * sizeof(uint64_t), h->stream));
    h->ext_on = false;
    for (SysHost &S : h->sys) S.counted = false;
    std::vector<int32_t> cs(total), cl(total);
    int64_t g = 0;
    for (int s = 0; s < h->max_sys; ++s) {
        SysDesc &d = h->hdesc[s];
        if (!h->sys[s].active) {
            d.gchunk0 = 0;
            d.nchunks = 0;
            d.nbuckets = 0;
            continue;
        }
        const int64_t nc = h->sys[s].cap / CHUNK;
        d.gchunk0 = g;
        d.nchunks = nc;
        d.nbuckets = h->sys[s].cap / BQ;
        for (int64_t c = 0; c < nc; ++c) {
            cs[g + c] = s;
            cl[g + c] = (int32_t)c;
        }
        g += nc;
    }
    h->n_chunks = total;
    if (total > 0) {
        HIP_TRY(hipMemcpyAsync(h->d_chunk_sys, cs.data(), total * sizeof(int32_t),
                               hipMemcpyHostToDevice, h->stream));
        HIP_TRY(hipMemcpyAsync(h->d_chunk_local, cl.data(), total * sizeof(int32_t),
                               hipMemcpyHostToDevice, h->stream));
    }
    HIP_TRY(hipMemcpyAsync(h->d_nchunks, &h->n_chunks, sizeof(int64_t), hipMemcpyHostToDevice,
                           h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return layout_records(h);
}

// The lists of spawn tiles: room in all for two tiles per bucket and for four times the
// walkers of the last iteration in whole tiles (the lists fill unevenly), grown by
// doubling (a graph holds the pointer, so growing drops the graphs). Buckets whose tiles
// do not fit are taken whole from a list of their own.
int ensure_tile_map(fciqmc_t *h) {
    int64_t walkers = 0;
    for (int s = 0; s < h->max_sys; ++s)
        if (h->sys[s].active) walkers += std::max<int64_t>(h->sys[s].last.nw, 0);
    int64_t want = 2 * BPC * h->n_chunks + ((4 * walkers) >> launch_shape(h).wsh) + 65536;
    if (h->tile_map_limit >= 0) want = std::min<int64_t>(want, h->tile_map_limit);
    if (want <= h->tile_cap || h->tile_map_off) return 0;
    int64_t cap = std::max<int64_t>(want, 2 * h->tile_cap);
    if (h->tile_map_limit >= 0) cap = std::min<int64_t>(cap, h->tile_map_limit);
    HIP_TRY(hipStreamSynchronize(h->stream));
    hipFree(h->d_tiles);
    h->d_tiles = nullptr;
    h->tile_cap = 0;
    drop_graphs(h);
    if (hipMalloc(&h->d_tiles, cap * 16) != hipSuccess) {
        (void)hipGetLastError();   // no room: every tile is found by its bucket instead
        h->d_tiles = nullptr;
        h->tile_map_off = true;
        return 0;
    }
    h->tile_cap = cap;
    return 0;
}

// Device bytes of a main list of cap entries: determinant (W words), population,
// H_DD per entry, and one count per bucket.
int64_t table_bytes(int64_t cap, int W) {
    return cap * (int64_t)(8 * W + sizeof(int32_t) + sizeof(double)) +
           (cap / BQ) * (int64_t)sizeof(int32_t) + 256;
}

// h1, the packed ERI, the pair table and the single-excitation term table, with
// rows of 64 W spin orbitals, and the rejection bounds (two bytes each).
int64_t integral_doubles(int M, int W) {
    const int64_t np = (int64_t)M * (M + 1) / 2, ns = 64 * (int64_t)W;
    return (int64_t)M * M + np * (np + 1) / 2 + ns * ns + ns * ns / 16 + (int64_t)2 * M * ns * ns;
}

int64_t integral_bytes(int M, int W) { return integral_doubles(M, W) * 8 + 256; }

void carve(SysHost &S, void *blk, int64_t cap) {
    char *p = (char *)blk;
    S.key = (uint64_t *)p;
    p += cap * 8 * S.W;
    S.hd = (double *)p;
    p += cap * sizeof(double);
    S.pop = (int32_t *)p;
    p += cap * sizeof(int32_t);
    S.bcnt = (int32_t *)p;
    p += (cap / BQ) * sizeof(int32_t);
    p = (char *)(((uintptr_t)p + 255) & ~(uintptr_t)255);
    S.d_h1 = (double *)p;
    p += (size_t)S.M * S.M * sizeof(double);
    S.d_eri = (double *)p;
    p += (size_t)S.eri.size() * sizeof(double);
    S.d_jk = (double *)p;
    p += (size_t)64 * S.W * 64 * S.W * sizeof(double);
    S.d_bound = (uint16_t *)p;
    p += (size_t)32 * S.W * 32 * S.W * sizeof(uint16_t);
    S.d_t3 = (double *)p;
    S.block = blk;
    S.cap = cap;
}

// Allocate the main list of a system with cap entries (every bucket empty) and
// room for its integrals. Old storage is released by the caller.
int alloc_tables(fciqmc_t *h, SysHost &S, int64_t cap, void **block_out) {
    const int64_t tb = table_bytes(cap, S.W), ib = integral_bytes(S.M, S.W);
    void *blk = nullptr;
    hipError_t e = hipMalloc(&blk, (size_t)(tb + ib));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_err(FCIQMC_ENOMEM, "device allocation of " + std::to_string(tb + ib) +
                                          " bytes failed: " + hipGetErrorString(e));
    }
    SysHost T = S;
    carve(T, blk, cap);
    HIP_TRY(hipMemsetAsync(T.bcnt, 0, (size_t)(cap / BQ) * sizeof(int32_t), h->stream));
    *block_out = blk;
    return 0;
}

int upload_integrals(fciqmc_t *h, SysHost &S) {
    HIP_TRY(hipMemcpyAsync(S.d_h1, S.h1.data(), S.h1.size() * 8, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(hipMemcpyAsync(S.d_eri, S.eri.data(), S.eri.size() * 8, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(hipMemcpyAsync(S.d_jk, S.jk.data(), S.jk.size() * 8, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(hipMemcpyAsync(S.d_bound, S.bound.data(), S.bound.size() * 2, hipMemcpyHostToDevice,
                           h->stream));
    HIP_TRY(hipMemcpyAsync(S.d_t3, S.t3.data(), S.t3.size() * 8, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    return 0;
}

void fill_desc_tables(fciqmc_t *h, int s) {
    SysHost &S = h->sys[s];
    SysDesc &d = h->hdesc[s];
    d.key = S.key;
    d.pop = S.pop;
    d.hdiag = S.hd;
    d.bcnt = S.bcnt;
    d.h1 = S.d_h1;
    d.eri = S.d_eri;
    d.jk = S.d_jk;
    d.t3 = S.d_t3;
    d.bound = S.d_bound;
    d.cap = (uint64_t)S.cap;
    d.nbuckets = S.cap / BQ;
}

// Move the main list of system s (and any of its entries waiting in the spill
// list) into new_cap entries' worth of buckets, in a new allocation.
int rebucket_system(fciqmc_t *h, int s, int64_t new_cap, int64_t n_spill) {
    SysHost &S = h->sys[s];
    for (int attempt = 0;; ++attempt) {
        void *blk = nullptr;
        int rc = alloc_tables(h, S, new_cap, &blk);
        if (rc) return rc == FCIQMC_ENOMEM ? FCIQMC_ECAPACITY : rc;
        SysHost T = S;
        carve(T, blk, new_cap);
        // the integrals (same layout after the list) move device to device
        const size_t ib = (size_t)((const char *)(S.d_t3 + S.t3.size()) - (const char *)S.d_h1);
        HIP_TRY(hipMemcpyAsync(T.d_h1, S.d_h1, ib, hipMemcpyDeviceToDevice, h->stream));
        // the kernel reads the destination from the descriptor
        SysDesc keep = h->hdesc[s];
        SysHost S_old = S;
        carve(S, blk, new_cap);
        fill_desc_tables(h, s);
        h->hdesc[s].nchunks = new_cap / CHUNK;
        h->hdesc[s].nbuckets = new_cap / BQ;
        rc = upload_desc(h);
        if (rc) return rc;
        HIP_TRY(hipMemsetAsync(h->d_err, 0, sizeof(uint32_t), h->stream));
        const EngineArgs a = make_args(h);
        HIP_TRY(FQ_LAUNCH(h->W, launch_rebucket, h->d_desc, s, S_old.key, S_old.pop, S_old.hd,
                          S_old.bcnt, S_old.cap / BQ, a.sp_det, a.sp_pop, a.sp_hd, a.sp_sys,
                          n_spill, h->d_err, h->stream));
        uint32_t err = 0;
        HIP_TRY(hipMemcpyAsync(&err, h->d_err, sizeof(uint32_t), hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        if (!err) {
            HIP_TRY(hipFree(S_old.block));
            S.last.used = std::max<int64_t>(S.last.used, S.last.nd + 1);
            share_slots(h, S, S_old.cap / BQ);
            rc = relayout(h);
            if (rc) return rc;
            return upload_desc(h);
        }
        // a bucket overflowed (far beyond the planned fill): back out, try twice the buckets
        HIP_TRY(hipFree(blk));
        S = S_old;
        h->hdesc[s] = keep;
        fill_desc_tables(h, s);
        rc = upload_desc(h);
        if (rc) return rc;
        if (attempt >= 4) return set_err(FCIQMC_ECAPACITY, "re-bucketing the main list failed");
        new_cap *= 2;
    }
}

// x in [0, 1] (or not finite) as a half-precision number not below it, 0 as 0, and none
// subnormal (the dot product of the kernel's test may take those as 0).
uint16_t half_up(double x) {
    if (x > 0.0 && x < 6.2e-5) x = 6.2e-5;
    _Float16 h = (_Float16)x;
    uint16_t b;
    std::memcpy(&b, &h, 2);
    if ((double)h < x) ++b;   // (positive: the next bit pattern is the next number)
    return b;
}

// Rejection bounds of double excitations: s over pairs of different spatial orbitals with
// |(pa|qb)| <= s_pa s_qb for every two of them, made small by a few sweeps of s_i =
// max_j |V_ij| / s_j, each of which keeps every inequality. (A sum over two indices
// decides most attempts: with integrals that decay as exp(-(|p-a| + |q-b|)/3), such a
// product follows them, where a single largest element would pass nearly every attempt.)
// Returns the largest s, to which the table is relative.
double double_bounds(const SysHost &S, std::vector<uint16_t> &out) {
    const int M = S.M, nt = 32 * S.W;
    std::vector<int64_t> pr;           // packed indices of the pairs p > a
    std::vector<int> pp, pa;
    for (int p = 0; p < M; ++p)
        for (int x = 0; x < p; ++x) {
            pr.push_back((int64_t)p * (p + 1) / 2 + x);
            pp.push_back(p);
            pa.push_back(x);
        }
    const int64_t n = (int64_t)pr.size();
    std::vector<double> V((size_t)n * n), s(n, 0.0), inv(n, 0.0);
    for (int64_t i = 0; i < n; ++i)
        for (int64_t j = 0; j <= i; ++j) {
            const double v = std::fabs(S.eri[pr[i] * (pr[i] + 1) / 2 + pr[j]]);
            V[(size_t)i * n + j] = V[(size_t)j * n + i] = v;
            s[i] = std::max(s[i], v);
            s[j] = std::max(s[j], v);
        }
    for (int64_t i = 0; i < n; ++i) {
        s[i] = std::sqrt(s[i]);
        inv[i] = s[i] > 0.0 ? 1.0 / s[i] : 0.0;
    }
    for (int sweep = 0; sweep < 3; ++sweep)
        for (int64_t i = 0; i < n; ++i) {
            double m = 0.0;
            const double own = V[(size_t)i * n + i];
            V[(size_t)i * n + i] = 0.0;
            for (int64_t j = 0; j < n; ++j) m = std::max(m, V[(size_t)i * n + j] * inv[j]);
            V[(size_t)i * n + i] = own;
            s[i] = std::max(m, std::sqrt(own));
            inv[i] = s[i] > 0.0 ? 1.0 / s[i] : 0.0;
        }
    double top = 0.0;
    for (int64_t i = 0; i < n; ++i) top = std::max(top, s[i]);
    out.assign((size_t)nt * nt, 0);
    for (int64_t i = 0; i < n; ++i) {
        const uint16_t b = half_up(top > 0.0 ? s[i] / top : 0.0);
        out[(size_t)pp[i] * nt + pa[i]] = out[(size_t)pa[i] * nt + pp[i]] = b;
    }
    return top;
}

// Rejection bounds of single excitations p -> a: |h_pa| plus the largest N - 1 spectator
// terms there can be, over both spins. Returns the largest, to which the table is relative.
double single_bounds(const SysHost &S, std::vector<uint16_t> &out) {
    const int M = S.M, nt = 32 * S.W, ns = 64 * S.W;
    std::vector<double> b((size_t)M * M, 0.0);
    double top = 0.0;
    for (int p = 0; p < M; ++p)
        for (int x = 0; x < M; ++x) {
            if (p == x) continue;
            double most = 0.0;
            for (int sp = 0; sp < 2; ++sp) {
                double sum = 0.0, big = 0.0;
                const double *row = &S.t3[((size_t)(2 * p + sp) * ns + (2 * x + sp)) * ns];
                for (int q = 0; q < 2 * M; ++q) {
                    if (q == 2 * p + sp || q == 2 * x + sp) continue;
                    sum += std::fabs(row[q]);
                    big = std::max(big, std::fabs(row[q]));
                }
                most = std::max(most, std::min(sum, big * (double)(S.N - 1)));
            }
            b[(size_t)p * M + x] = std::fabs(S.h1[(size_t)p * M + x]) + most;
            top = std::max(top, b[(size_t)p * M + x]);
        }
    out.assign((size_t)nt * nt, 0);
    for (int p = 0; p < M; ++p)
        for (int x = 0; x < M; ++x)
            out[(size_t)p * nt + x] = half_up(top > 0.0 ? b[(size_t)p * M + x] / top : 0.0);
    return top;
}

hdet_t aufbau(const std::vector<double> &h1, int M, int na, int nb) {
    std::vector<int> order(M);
    for (int i = 0; i < M; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return h1[a * M + a] < h1[b * M + b]; });
    hdet_t d = 0;
    for (int i = 0; i < na; ++i) d |= hbit(2 * order[i]);
    for (int i = 0; i < nb; ++i) d |= hbit(2 * order[i] + 1);
    return d;
}

// Numbers of symmetry-allowed singles and doubles from det, counted per class.
void excitation_counts(const SysHost &S, hdet_t det, int64_t &ns, int64_t &nd) {
    const int nso = 2 * S.M;
    int n_occ[NCLASS] = {0}, n_emp[NCLASS] = {0};
    auto cls = [&](int p) { return 2 * (int)S.irrep[p >> 1] + (p & 1); };
    for (int p = 0; p < nso; ++p) ((det >> p) & 1 ? n_occ : n_emp)[cls(p)]++;
    ns = 0;
    for (int c = 0; c < NCLASS; ++c) ns += (int64_t)n_occ[c] * n_emp[c];
    nd = 0;
    std::vector<int> occ;
    for (int p = 0; p < nso; ++p)
        if ((det >> p) & 1) occ.push_back(p);
    for (size_t i = 0; i < occ.size(); ++i)
        for (size_t j = i + 1; j < occ.size(); ++j) {
            const int p = occ[i], q = occ[j];
            const int g = S.irrep[p >> 1] ^ S.irrep[q >> 1];
            if ((p & 1) == (q & 1)) {
                const int sp = p & 1;
                for (int ga = 0; ga < 8; ++ga) {
                    const int gb = ga ^ g;
                    if (gb < ga) continue;
                    const int na_ = n_emp[2 * ga + sp], nb_ = n_emp[2 * gb + sp];
                    nd += (ga == gb) ? (int64_t)na_ * (na_ - 1) / 2 : (int64_t)na_ * nb_;
                }
            } else {
                for (int ga = 0; ga < 8; ++ga)
                    nd += (int64_t)n_emp[2 * ga + 0] * n_emp[2 * (ga ^ g) + 1];
            }
        }
}

int validate(const fciqmc_hamiltonian *ham, const fciqmc_params *prm) {
    if (!ham || !prm) return set_err(FCIQMC_EINVAL, "null hamiltonian or params");
    if (ham->n_orb < 1 || ham->n_orb > 64)
        return set_err(FCIQMC_EINVAL, "n_orb must be in 1..64 (2*n_orb <= 128)");
    if (prm->det_words < 0 || prm->det_words > 2 || (prm->det_words == 1 && 2 * ham->n_orb > 64))
        return set_err(FCIQMC_EINVAL, "det_words must be 0, 1 (at most 64 spin orbitals) or 2");
    if (ham->n_alpha < 0 || ham->n_beta < 0 || ham->n_alpha > ham->n_orb ||
        ham->n_beta > ham->n_orb || ham->n_alpha + ham->n_beta == 0)
        return set_err(FCIQMC_EINVAL, "bad electron counts");
    if (!ham->h1 || !ham->eri) return set_err(FCIQMC_EINVAL, "missing integrals");
    if (!(prm->tau > 0.0)) return set_err(FCIQMC_EINVAL, "tau must be positive");
    if (prm->shift_update_every < 1) return set_err(FCIQMC_EINVAL, "shift_update_every must be >= 1");
    if (ham->p_double > 1.0) return set_err(FCIQMC_EINVAL, "p_double > 1");
    if (prm->initial_walkers < 0 || prm->initial_walkers > 2147483647)
        return set_err(FCIQMC_EINVAL, "initial_walkers out of range");
    if (ham->orb_irrep)
        for (int i = 0; i < ham->n_orb; ++i)
            if (ham->orb_irrep[i] > 7) return set_err(FCIQMC_EINVAL, "irrep labels must be 0..7");
    if (prm->space & ~(FCIQMC_SPACE_EXCITATION | FCIQMC_SPACE_SENIORITY | FCIQMC_SPACE_FROZEN))
        return set_err(FCIQMC_EINVAL, "unknown space restriction");
    if (((prm->space & FCIQMC_SPACE_EXCITATION) && prm->max_excitation < 0) ||
        ((prm->space & FCIQMC_SPACE_SENIORITY) && prm->max_seniority < 0) ||
        ((prm->space & FCIQMC_SPACE_FROZEN) &&
         ((prm->frozen_occupied & prm->frozen_empty) ||
          (prm->frozen_occupied_hi & prm->frozen_empty_hi))))
        return set_err(FCIQMC_EINVAL, "inconsistent space restriction");
    if (prm->hphf != 0 && prm->hphf != 1 && prm->hphf != -1)
        return set_err(FCIQMC_EINVAL, "hphf must be 0, 1 or -1");
    if (prm->hphf && ham->n_alpha != ham->n_beta)
        return set_err(FCIQMC_EINVAL, "spin-coupled functions need n_alpha = n_beta");
    if (prm->hphf && prm->space)
        return set_err(FCIQMC_EINVAL, "spin-coupled functions with a restricted space are not supported");
    return 0;
}

hdet_t host_spin_flip(hdet_t D) { return ((D & HEVEN) << 1) | ((D >> 1) & HEVEN); }

// Whether det lies in the run's restricted space (host check of the reference).
bool host_in_space(const fciqmc_params *prm, hdet_t d0, hdet_t det) {
    if ((prm->space & FCIQMC_SPACE_EXCITATION) && hpopc(det & ~d0) > prm->max_excitation)
        return false;
    if ((prm->space & FCIQMC_SPACE_SENIORITY) && hpopc((det ^ (det >> 1)) & HEVEN) > prm->max_seniority)
        return false;
    const hdet_t fo = ((hdet_t)prm->frozen_occupied_hi << 64) | (hdet_t)prm->frozen_occupied;
    const hdet_t fe = ((hdet_t)prm->frozen_empty_hi << 64) | (hdet_t)prm->frozen_empty;
    if ((prm->space & FCIQMC_SPACE_FROZEN) && ((det & fo) != fo || (det & fe))) return false;
    return true;
}

int64_t initial_capacity(const fciqmc_params *prm) {
    return prm->det_capacity > 0 ? round_cap(prm->det_capacity)
                                 : cap_for_entries(4 * std::max<int64_t>(prm->initial_walkers, 1024));
}

// Device bytes reserved for a system at its walker target: a main list of twice
// the target in entries, and its integrals.
int64_t target_footprint(const fciqmc_hamiltonian *ham, const fciqmc_params *prm) {
    const int64_t cap = round_cap(2 * std::max<int64_t>(prm->target_walkers, 1));
    const int W = words_for(ham->n_orb, prm->det_words);
    return table_bytes(cap, W) + integral_bytes(ham->n_orb, W);
}

int load_list(fciqmc_t *h, int s, const std::vector<hdet_t> &det, const std::vector<int32_t> &pop);

// Admit a system into slot s (slot must be free).
int admit(fciqmc_t *h, int s, const fciqmc_hamiltonian *ham, const fciqmc_params *prm) {
    int rc = validate(ham, prm);
    if (rc) return rc;
    SysHost &S = h->sys[s];
    S = SysHost();
    S.prm = *prm;
    S.M = ham->n_orb;
    S.na = ham->n_alpha;
    S.nb = ham->n_beta;
    S.N = S.na + S.nb;
    S.e_core = ham->e_core;
    S.h1.assign(ham->h1, ham->h1 + (size_t)S.M * S.M);
    const int64_t np = (int64_t)S.M * (S.M + 1) / 2;
    S.eri.assign(ham->eri, ham->eri + np * (np + 1) / 2);
    S.irrep.assign(S.M, 0);
    if (ham->orb_irrep) S.irrep.assign(ham->orb_irrep, ham->orb_irrep + S.M);
    const int nso = 2 * S.M;
    S.W = words_for(S.M, prm->det_words);
    if (S.W != h->W)
        return set_err(FCIQMC_EINVAL, "a batch holds determinants of one width: this system takes " +
                                          std::to_string(S.W) + " 64-bit words, the batch " +
                                          std::to_string(h->W));
    const hdet_t valid = nso == 128 ? ~(hdet_t)0 : (hbit(nso) - 1);
    if (ham->ref_det) {
        S.d0 = hdet_in(ham->ref_det, S.W);
        int a = 0, b = 0;
        for (int p = 0; p < 128; ++p)
            if ((S.d0 >> p) & 1) (p & 1 ? b : a)++;
        if ((S.d0 & ~valid) || a != S.na || b != S.nb)
            return set_err(FCIQMC_EINVAL, "reference determinant does not match the electron counts");
    } else {
        S.d0 = aufbau(S.h1, S.M, S.na, S.nb);
    }
    if (!host_in_space(prm, S.d0, S.d0))
        return set_err(FCIQMC_EINVAL, "the reference lies outside the restricted space");
    if (ham->p_double >= 0.0) {
        S.p_double = ham->p_double;
    } else {
        int64_t ns, nd;
        excitation_counts(S, S.d0, ns, nd);
        S.p_double = (ns + nd) > 0 ? (double)nd / (double)(ns + nd) : 0.0;
    }
    if (prm->hphf) {   // the reference function, stored as the smaller determinant of its pair
        const hdet_t f = host_spin_flip(S.d0);
        if (f == S.d0 && prm->hphf < 0)
            return set_err(FCIQMC_EINVAL, "a closed-shell reference has no odd-spin function");
        S.d0 = std::min(S.d0, f);
    }
    S.reserve_bytes = target_footprint(ham, prm);
    // free-memory admission
    size_t fr = 0, tot = 0;
    HIP_TRY(hipMemGetInfo(&fr, &tot));
    int64_t reserved = 0;
    for (int t = 0; t < h->max_sys; ++t)
        if (t != s && h->sys[t].active)
            reserved += std::max<int64_t>(0, h->sys[t].reserve_bytes - table_bytes(h->sys[t].cap, h->W));
    const int64_t need = S.reserve_bytes;
    if ((int64_t)fr - reserved < need + (int64_t)(1ull << 30))
        return set_err(FCIQMC_ENOMEM, "system footprint " + std::to_string(need) +
                                          " B does not fit in free device memory");
    // Pair table for the diagonal elements: (pp|qq) - (pq|qp) over spin orbitals p < q,
    // rows of ns = 64 W entries.
    const int ns = 64 * S.W;
    S.jk.assign((size_t)ns * ns, 0.0);
    auto eri_sp = [&](int i, int j, int k, int l) {
        auto tri = [](int x, int y) { return x >= y ? (int64_t)x * (x + 1) / 2 + y : (int64_t)y * (y + 1) / 2 + x; };
        const int64_t a = tri(i, j), b = tri(k, l);
        return S.eri[a >= b ? a * (a + 1) / 2 + b : b * (b + 1) / 2 + a];
    };
    for (int p = 0; p < nso; ++p)
        for (int q = p + 1; q < nso; ++q) {
            const double coul = eri_sp(p >> 1, p >> 1, q >> 1, q >> 1);
            const double exch = ((p ^ q) & 1) ? 0.0 : eri_sp(p >> 1, q >> 1, q >> 1, p >> 1);
            S.jk[(size_t)p * ns + q] = coul - exch;
        }
    // Single-excitation terms: for p -> a (same spin) and each spectator q,
    // (pa|qq) - [same spin](pq|qa), the difference the Slater-Condon sum adds.
    S.t3.assign((size_t)nso * ns * ns, 0.0);
    for (int p = 0; p < nso; ++p)
        for (int a = 0; a < nso; ++a) {
            if ((p ^ a) & 1) continue;
            for (int q = 0; q < nso; ++q) {
                const double coul = eri_sp(p >> 1, a >> 1, q >> 1, q >> 1);
                const double exch = ((p ^ q) & 1) ? 0.0 : eri_sp(p >> 1, q >> 1, q >> 1, a >> 1);
                S.t3[((size_t)p * ns + a) * ns + q] = coul - exch;
            }
        }
    {
        double h1m = 0.0, em = 0.0;
        for (int p = 0; p < S.M; ++p)
            for (int q = 0; q < p; ++q) h1m = std::max(h1m, std::fabs(S.h1[(size_t)p * S.M + q]));
        // (pa|qb) with p != a and q != b: the diagonal pairs p = a are the last of each row
        std::vector<char> diag((size_t)np, 0);
        for (int p = 0; p < S.M; ++p) diag[(size_t)p * (p + 1) / 2 + p] = 1;
        for (int64_t i = 0, k = 0; i < np; ++i)
            for (int64_t j = 0; j <= i; ++j, ++k)
                if (!diag[i] && !diag[j]) em = std::max(em, std::fabs(S.eri[k]));
        S.h_max = h1m + 2.0 * em;
    }
    const bool defer = S.p_double >= 0.5;
    const double scale = defer ? double_bounds(S, S.bound) : single_bounds(S, S.bound);
    const int64_t cap = initial_capacity(prm);
    void *blk = nullptr;
    rc = alloc_tables(h, S, cap, &blk);
    if (rc) return rc;
    carve(S, blk, cap);
    rc = upload_integrals(h, S);
    if (rc) return rc;
    S.growth = cap / 16;
    S.active = true;
    SysDesc &d = h->hdesc[s];
    std::memset(&d, 0, sizeof d);
    d.active = 1;
    d.M = S.M;
    d.N = S.N;
    d.n_so = nso;
    {
        int mx = 0;
        for (int i = 0; i < S.M; ++i) mx = std::max<int>(mx, S.irrep[i]);
        d.n_class = 2 * (mx + 1);
    }
    d.A = prm->shift_update_every;
    d.n_a = prm->initiator_threshold;
    d.tau = prm->tau;
    d.zeta = prm->shift_damping;
    d.e_core = S.e_core;
    d.p_double = S.p_double;
    d.p_single = 1.0 - S.p_double;
    d.inv_p_double = d.p_double > 0.0 ? 1.0 / d.p_double : 0.0;
    d.inv_p_single = d.p_single > 0.0 ? 1.0 / d.p_single : 0.0;
    {
        // pgen of a double excitation without a point group, by the same operations
        // as the general branch of the kernels' excitation generator
        const int ne[2] = {S.M - hpopc(S.d0 & HEVEN), S.M - hpopc(S.d0 & (HEVEN << 1))};
        d.n_emp[0] = ne[0];
        d.n_emp[1] = ne[1];
        auto pg = [&](int nba, int nbb, int nal) {
            return (2.0 * d.p_double * (1.0 / (double)nba + 1.0 / (double)nbb)) /
                   (double)((int64_t)S.N * (int64_t)(S.N - 1) * (int64_t)nal);
        };
        const int nal_u = (ne[1] > 0 ? ne[0] : 0) + (ne[0] > 0 ? ne[1] : 0);
        for (int sp = 0; sp < 2; ++sp) {
            d.pgen_c1[sp] = ne[sp] >= 2 && S.N >= 2 ? pg(ne[sp] - 1, ne[sp] - 1, ne[sp]) : 0.0;
            d.pgen_c1[2 + sp] =
                ne[sp] > 0 && ne[1 - sp] > 0 && S.N >= 2 ? pg(ne[1 - sp], ne[sp], nal_u) : 0.0;
        }
    }
    {
        // The margin covers every rounding of the bound's single-precision arithmetic
        // (a few 1e-7) and of the exact test's.
        constexpr double margin = 1.0 + 1e-5;
        d.defer = defer ? 1 : 0;
        d.has_double = d.p_double > 0.0 ? 1 : 0;
        d.dbl_thr = d.has_double ? (uint32_t)((uint64_t)std::ceil(d.p_double * 4294967296.0) - 1ull) : 0u;
        // w0 / 2^32 / P_double is a double's uniform
        const double u1 = d.inv_p_double / 4294967296.0;
        if (defer) {
            d.bound_ft = (float)(prm->tau * scale * scale / u1 * margin);
            for (int c = 0; c < 4; ++c)
                d.bound_f[c] = d.pgen_c1[c] > 0.0
                                   ? (float)(prm->tau * scale * scale / d.pgen_c1[c] / u1 * margin)
                                   : INFINITY;
        } else {
            d.bound_ft = (float)(prm->tau * scale / d.p_single * margin);
            d.sg_mul = (float)(d.inv_p_single / 4294967296.0);
            d.sg_sub = (float)(d.p_double * d.inv_p_single + 1e-5);
        }
    }
    d.target = prm->target_walkers;
    d.seed = prm->seed;
    d.d0 = hlo(S.d0);
    d.d0_hi = hhi(S.d0);
    d.det_words = S.W;
    d.space = prm->space;
    d.max_ex = prm->max_excitation;
    d.max_sen = prm->max_seniority;
    d.frz_occ = prm->frozen_occupied;
    d.frz_emp = prm->frozen_empty;
    d.frz_occ_hi = prm->frozen_occupied_hi;
    d.frz_emp_hi = prm->frozen_empty_hi;
    d.hphf = prm->hphf;
    d.lam = ((S.N / 2) & 1) ? -prm->hphf : prm->hphf;
    d.valid = hlo(valid);
    d.valid_hi = hhi(valid);
    for (int p = 0; p < nso; ++p) {
        const int c = 2 * S.irrep[p >> 1] + (p & 1);
        if (p < 64)
            d.cmask[c] |= 1ull << p;
        else
            d.cmask_hi[c] |= 1ull << (p - 64);
    }
    for (int i = 0; i < S.M; ++i) {
        uint64_t *w = i < 32 ? d.irr_packed : d.irr_packed_hi;
        w[(i >> 4) & 1] |= (uint64_t)S.irrep[i] << (4 * (i & 15));
    }
    d.shift = prm->initial_shift;
    fill_desc_tables(h, s);
    rc = relayout(h);
    if (rc) return rc;
    const int64_t n0 = prm->initial_walkers > 0 ? prm->initial_walkers : 10;
    rc = load_list(h, s, {S.d0}, {(int32_t)n0});
    if (rc) return rc;
    S.last.shift = prm->initial_shift;
    return 0;
}

// Replace the list of system s by the n entries (dd, dp) on the device, of which `held`
// have walkers (at most `most` each; the others are skipped), and the reference without
// walkers if it is not among them.
int load_entries(fciqmc_t *h, int s, const uint64_t *dd, const int32_t *dp, int64_t n, int64_t held,
                 bool have_ref, int64_t most) {
    SysHost &S = h->sys[s];
    const int64_t entries = held + (have_ref ? 0 : 1);
    int64_t need = std::max<int64_t>(S.cap, cap_for_entries(entries));
    for (int attempt = 0;; ++attempt) {
        if (need > S.cap) {
            void *blk = nullptr;
            int rc = alloc_tables(h, S, need, &blk);
            if (rc) return rc;
            SysHost T = S;
            carve(T, blk, need);
            rc = upload_integrals(h, T);
            if (rc) return rc;
            HIP_TRY(hipFree(S.block));
            const int64_t old_nb = S.cap / BQ;
            carve(S, blk, need);
            share_slots(h, S, old_nb);
            fill_desc_tables(h, s);
            rc = relayout(h);
            if (rc) return rc;
        } else {
            HIP_TRY(hipMemsetAsync(S.bcnt, 0, (size_t)(S.cap / BQ) * sizeof(int32_t), h->stream));
        }
        h->hstatus[s] = 0;
        int rc = reset_spawns(h, s);
        if (rc) return rc;
        rc = upload_desc(h);
        if (rc) return rc;
        HIP_TRY(hipMemsetAsync(h->d_err, 0, sizeof(uint32_t), h->stream));
        HIP_TRY(FQ_LAUNCH(h->W, launch_load, h->d_desc, s, dd, dp, n, have_ref ? 0 : 1, h->d_err,
                          h->stream));
        uint32_t err = 0;
        HIP_TRY(hipMemcpyAsync(&err, h->d_err, 4, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        if (!err) break;
        // a bucket overflowed: twice the buckets
        if (attempt >= 4) return set_err(FCIQMC_ECAPACITY, "walker list does not fit the buckets");
        need = 2 * S.cap;
    }
    S.growth = std::max<int64_t>(256, entries / 8);
    S.spawn_rate = 1.0;
    S.rec_peak = 0;
    S.counted = false;
    S.pop_max = most;
    return 0;
}

// A caller's list of n entries on the device for the length of a call.
struct ListBuf {
    uint64_t *det = nullptr;
    int32_t *pop = nullptr;
    ListCheck *check = nullptr;
    ~ListBuf() {
        hipFree(det);
        hipFree(pop);
        hipFree(check);
    }
    int upload(fciqmc_t *h, const uint64_t *d, const int32_t *p, int64_t n) {
        const size_t kb = (size_t)n * 8 * h->W;
        HIP_TRY(hipMalloc(&det, std::max<size_t>(kb, 8)));
        HIP_TRY(hipMalloc(&pop, std::max<int64_t>(n, 1) * 4));
        if (n == 0) return 0;
        HIP_TRY(hipMemcpyAsync(det, d, kb, hipMemcpyHostToDevice, h->stream));
        HIP_TRY(hipMemcpyAsync(pop, p, n * 4, hipMemcpyHostToDevice, h->stream));
        return 0;
    }
};

// Replace the list of system s by (det, pop), a list the engine made itself.
int load_list(fciqmc_t *h, int s, const std::vector<hdet_t> &det, const std::vector<int32_t> &pop) {
    SysHost &S = h->sys[s];
    const int64_t n = (int64_t)det.size();
    std::vector<uint64_t> words((size_t)n * S.W);
    int64_t held = 0, most = 0;
    bool have_ref = false;
    for (int64_t i = 0; i < n; ++i) {
        hdet_out(det[i], &words[(size_t)i * S.W], S.W);
        if (pop[i] == 0) continue;
        held++;
        have_ref |= det[i] == S.d0;
        most = std::max<int64_t>(most, pop[i] < 0 ? -(int64_t)pop[i] : pop[i]);
    }
    ListBuf b;
    int rc = b.upload(h, words.data(), pop.data(), n);
    if (rc) return rc;
    return load_entries(h, s, b.det, b.pop, n, held, have_ref, most);
}

// Whether the list (det, pop; on the device b, which this reorders) has walkers twice on
// one determinant: sorted on the device in the record buffer or a second list of the call's
// own, on the host where there is room for neither.
int holds_twice(fciqmc_t *h, ListBuf &b, const uint64_t *det, const int32_t *pop, int64_t n,
                ListCheck &c) {
    const size_t kb = (size_t)n * 8 * h->W, vb = ((size_t)n * 4 + 15) / 16 * 16;
    const size_t bytes = kb + vb + (size_t)sort_hist_words(n) * 4;
    void *own = nullptr;
    char *blk = nullptr;
    if (n <= SORT_MAX) {
        if ((size_t)h->rec_cap * 16 * h->W >= bytes) blk = (char *)h->d_recs;
        else if (hipMalloc(&own, bytes) == hipSuccess) blk = (char *)own;
        else (void)hipGetLastError();
    }
    if (!blk) {
        std::vector<hdet_t> v;
        v.reserve(n);
        for (int64_t i = 0; i < n; ++i)
            if (pop[i] != 0) v.push_back(hdet_in(det + i * h->W, h->W));
        std::sort(v.begin(), v.end());
        c.twice = std::adjacent_find(v.begin(), v.end()) != v.end();
        return 0;
    }
    auto body = [&]() -> int {
        // every digit: entries without walkers may hold any word
        HIP_TRY(FQ_LAUNCH(h->W, launch_sort, b.det, b.pop, (uint64_t *)blk, (int32_t *)(blk + kb),
                          (uint32_t *)(blk + kb + vb), n, 8 * h->W, h->stream));
        HIP_TRY(FQ_LAUNCH(h->W, launch_twice, b.det, b.pop, n, b.check, h->stream));
        HIP_TRY(hipMemcpyAsync(&c, b.check, sizeof c, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        return 0;
    };
    const int rc = body();
    if (own) {
        if (rc) (void)hipStreamSynchronize(h->stream);
        hipFree(own);
    }
    return rc;
}

int compute_e0(fciqmc_t *h, int s);

struct Walkers {
    std::vector<hdet_t> det;
    std::vector<int32_t> pop;
};

// The list of system s in ascending order of determinants: the number of its entries in
// *n, the first `cap` of them in det (W words each), pop and flags (any may be null).
// Compacted, sorted and flagged on the device; the lists live for the call only, in the
// record buffer where they fit (its records are dead between launches). The host's sort was
// nearly all of an export: a count and an export of 1.35e6 determinants took 220 ms with it.
int list_out(fciqmc_t *h, int s, uint64_t *det, int32_t *pop, uint32_t *flags, int64_t cap,
             int64_t *n_out) {
    SysHost &S = h->sys[s];
    const int64_t nb = S.cap / BQ;
    unsigned long long n = 0;
    HIP_TRY(hipMemsetAsync(h->d_count, 0, 8, h->stream));
    HIP_TRY(FQ_LAUNCH(h->W, launch_compact, S.key, S.pop, S.bcnt, nb, nullptr, nullptr, h->d_count,
                      0, h->stream));
    HIP_TRY(hipMemcpyAsync(&n, h->d_count, 8, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    *n_out = (int64_t)n;
    const int64_t m = std::min<int64_t>((int64_t)n, cap);
    if (m <= 0 || (!det && !pop && !flags)) return 0;
    // two lists and the digit counts; one list only where the device has no room for two
    // (or the sort no positions): those are sorted on the host
    const size_t kb = (size_t)n * 8 * S.W, vb = ((size_t)n * 4 + 15) / 16 * 16;
    const size_t both = 2 * (kb + vb) + (size_t)sort_hist_words((int64_t)n) * 4;
    char *blk = nullptr;
    void *own = nullptr;
    bool on_device = (int64_t)n <= SORT_MAX;
    if (on_device) {
        if ((size_t)h->rec_cap * 16 * h->W >= both) blk = (char *)h->d_recs;
        else if (hipMalloc(&own, both) == hipSuccess) blk = (char *)own;
        else {
            (void)hipGetLastError();
            on_device = false;
        }
    }
    if (!on_device) {
        HIP_TRY(hipMalloc(&own, kb + vb));
        blk = (char *)own;
    }
    auto body = [&]() -> int {
        uint64_t *k1 = (uint64_t *)blk;
        int32_t *v1 = (int32_t *)(blk + kb);
        HIP_TRY(hipMemsetAsync(h->d_count, 0, 8, h->stream));
        HIP_TRY(FQ_LAUNCH(h->W, launch_compact, S.key, S.pop, S.bcnt, nb, k1, v1, h->d_count,
                          (int64_t)n, h->stream));
        if (on_device) {
            uint64_t *k2 = (uint64_t *)(blk + kb + vb);
            int32_t *v2 = (int32_t *)(blk + 2 * kb + vb);
            const int passes = (2 * S.M + 7) / 8;
            HIP_TRY(FQ_LAUNCH(h->W, launch_sort, k1, v1, k2, v2, (uint32_t *)(blk + 2 * (kb + vb)),
                              (int64_t)n, passes, h->stream));
            if (passes & 1) {
                std::swap(k1, k2);
                std::swap(v1, v2);
            }
            if (flags) {   // into the other list's populations
                HIP_TRY(FQ_LAUNCH(h->W, launch_flags, k1, v1, m, S.prm.initiator_threshold,
                                  hlo(S.d0), hhi(S.d0), (uint32_t *)v2, h->stream));
                HIP_TRY(hipMemcpyAsync(flags, v2, m * 4, hipMemcpyDeviceToHost, h->stream));
            }
            if (det) HIP_TRY(hipMemcpyAsync(det, k1, m * 8 * S.W, hipMemcpyDeviceToHost, h->stream));
            if (pop) HIP_TRY(hipMemcpyAsync(pop, v1, m * 4, hipMemcpyDeviceToHost, h->stream));
            HIP_TRY(hipStreamSynchronize(h->stream));
            return 0;
        }
        std::vector<uint64_t> words(n * S.W);
        std::vector<int32_t> pv(n);
        HIP_TRY(hipMemcpyAsync(words.data(), k1, kb, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipMemcpyAsync(pv.data(), v1, n * 4, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        std::vector<std::pair<hdet_t, int32_t>> v(n);
        for (size_t i = 0; i < n; ++i) v[i] = {hdet_in(&words[i * S.W], S.W), pv[i]};
        std::sort(v.begin(), v.end());
        for (int64_t i = 0; i < m; ++i) {
            const int64_t a = v[i].second < 0 ? -(int64_t)v[i].second : v[i].second;
            if (det) hdet_out(v[i].first, det + i * S.W, S.W);
            if (pop) pop[i] = v[i].second;
            if (flags) flags[i] = (a > S.prm.initiator_threshold || v[i].first == S.d0) ? 1u : 0u;
        }
        return 0;
    };
    const int rc = body();
    if (own) {
        if (rc) (void)hipStreamSynchronize(h->stream);
        hipFree(own);
    }
    return rc;
}

int export_walkers(fciqmc_t *h, int s, Walkers &w) {
    const int W = h->sys[s].W;
    int64_t n = 0, m = 0;
    int rc = list_out(h, s, nullptr, nullptr, nullptr, 0, &n);
    if (rc) return rc;
    std::vector<uint64_t> words((size_t)n * W);
    w.det.resize(n);
    w.pop.resize(n);
    rc = list_out(h, s, words.data(), w.pop.data(), nullptr, n, &m);
    if (rc) return rc;
    for (int64_t i = 0; i < n; ++i) w.det[i] = hdet_in(&words[(size_t)i * W], W);
    return 0;
}

int fill_estimates(fciqmc_t *h, int s, fciqmc_estimates *o) {
    SysHost &S = h->sys[s];
    if (!S.active) return set_err(FCIQMC_ESTATE, "slot is not active");
    const IterRecord &r = S.last;
    std::memset(o, 0, sizeof *o);
    o->iteration = h->hdesc[s].iter;
    o->n_walkers = r.nw;
    o->n_dets = r.nd;
    o->ref_pop = r.c0;
    o->attempts = r.attempts;
    o->spawns = r.spawns;
    o->merged = r.merged;
    o->aborted = r.aborted;
    o->born = r.born;
    o->total_attempts = S.tot_att;
    o->total_spawns = S.tot_sp;
    o->n_samples = S.e_blk.count();
    o->n_var = h->hdesc[s].n_var;
    o->n_prev = h->hdesc[s].n_prev;
    o->table_slots = S.cap;
    o->table_used = std::max<int64_t>(r.used, r.nd);
    o->shift = h->hdesc[s].shift;
    o->e_ref = S.e0;
    o->p_double = S.p_double;
    o->proj_num = r.num;
    o->e_proj_inst = r.c0 != 0 ? S.e0 + r.num / (double)r.c0 : NAN;
    double m, e;
    S.e_blk.result(m, e);
    o->e_proj_mean = S.e0 + m;
    o->e_proj_err = e;
    S.s_blk.result(m, e);
    o->shift_mean = S.e0 + m;
    o->shift_err = e;
    o->ms_last_call = h->ms_last;
    o->redos = S.redos;
    o->spills = S.spills;
    o->ms_spawn = h->phase_ms[0] + h->phase_ms[1] + h->phase_ms[2];
    o->ms_death = 0.0;   // death runs inside the annihilation pass
    o->ms_annihilate = h->phase_ms[3];
    o->ms_estimators = h->phase_ms[4];
    o->shift_varying = h->hdesc[s].varying;
    o->status = S.fatal;
    return 0;
}

// Captured graphs a handle keeps (up to 64 iterations of three kernels each): a list that
// grows, or calls of changing lengths, would otherwise leave one for every combination of
// length and launch shape it has met.
constexpr size_t MAX_GRAPHS = 64;

int capture_or_get(fciqmc_t *h, int L, hipGraphExec_t *out) {
    // one graph per length, spawning variant and launch shape
    const Shape sh = launch_shape(h);
    EngineArgs a = make_args(h);
    a.wsh = sh.wsh;
    a.post_seg = sh.post_seg;
    const std::array<int, 6> key = {L, a.plain, sh.wsh, sh.spawn_grid, sh.post_grid, sh.post_seg};
    auto it = h->graphs.find(key);
    if (it != h->graphs.end()) {
        it->second.used = ++h->graph_clock;
        *out = it->second.exec;
        return 0;
    }
    if (h->graphs.size() >= MAX_GRAPHS) {   // the one not launched for longest (none is running)
        auto old = h->graphs.begin();
        for (auto k = h->graphs.begin(); k != h->graphs.end(); ++k)
            if (k->second.used < old->second.used) old = k;
        (void)hipGraphExecDestroy(old->second.exec);
        h->graphs.erase(old);
    }
    hipGraph_t g = nullptr;
    HIP_TRY(hipStreamBeginCapture(h->stream, hipStreamCaptureModeRelaxed));
    for (int i = 0; i < L; ++i)
        FQ_LAUNCH(h->W, launch_iteration, a, sh.post_grid, sh.spawn_grid, i == 0, h->stream, nullptr);
    HIP_TRY(hipStreamEndCapture(h->stream, &g));
    hipGraphExec_t ex = nullptr;
    HIP_TRY(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0));
    HIP_TRY(hipGraphDestroy(g));
    h->graphs[key] = {ex, ++h->graph_clock};
    *out = ex;
    return 0;
}

// The extensions of crowded systems' buckets, anew before each launch (the record buffer is
// dead between launches): what they need in all, room for it, their places.
int extend_buckets(fciqmc_t *h) {
    bool any = false;
    for (const SysHost &S : h->sys) any |= S.active && S.crowded && S.counted;
    if (!any && !h->ext_on) return 0;
    HIP_TRY(hipMemsetAsync(h->d_bext, 0, BPC * h->chunk_alloc * sizeof(uint64_t), h->stream));
    h->ext_on = any;
    int64_t pool = 0;
    for (int pass = 0; any && pass < 2; ++pass) {
        HIP_TRY(hipMemsetAsync(h->d_count, 0, 8, h->stream));
        for (int s = 0; s < h->max_sys; ++s) {
            const SysHost &S = h->sys[s];
            if (!S.active || !S.crowded || !S.counted) continue;
            const int64_t b0 = h->hdesc[s].gchunk0 * BPC;
            HIP_TRY(FQ_LAUNCH(h->W, launch_extend, h->d_bprev + b0, h->d_bext + b0, S.cap / BQ,
                              (uint32_t)S.rec_r, (float)S.ext_factor, h->rec_base, pool, h->d_count,
                              h->stream));
        }
        if (pass == 0) {
            unsigned long long need = 0;
            HIP_TRY(hipMemcpyAsync(&need, h->d_count, 8, hipMemcpyDeviceToHost, h->stream));
            HIP_TRY(hipStreamSynchronize(h->stream));
            pool = (int64_t)need;
            if (h->rec_base + pool > h->rec_cap) {
                const int rc = ensure_records(h, h->rec_base + pool + pool / 4);
                if (rc) return rc;
            }
        }
    }
    return 0;
}

// Whether list S may have nc entries' worth of buckets for its records' sake: they save time
// only, so the table and the slots that BUCKET_RECS records a bucket come to (120, with the
// planner's slack over the fullest of many) may take half of the free memory, the old ones
// still in place. The rest is for what lists cannot do without.
int split_fits(const fciqmc_t *h, const SysHost &S, int64_t nc, bool *fits) {
    size_t fr = 0, tot = 0;
    HIP_TRY(hipMemGetInfo(&fr, &tot));
    const int64_t need = table_bytes(nc, S.W) + integral_bytes(S.M, S.W) +
                         nc / BQ * (int64_t)(128 * 16 * h->W);
    *fits = need <= (int64_t)(fr / 2);
    return 0;
}

// Before a launch of up to L iterations: re-bucket any main list whose buckets
// would pass 5/8 full on average during the launch (each iteration adds at most
// `growth` entries, the largest increase seen, with slack), size the record slots per
// bucket for the launch (the fullest bucket of the last launch growing at the largest
// rate seen), and return how many iterations that headroom allows. Whatever the
// estimates miss is caught on the device: overflowing record slots abandon the
// iteration for a re-run, an overflowing bucket of the main list spills.
int plan_launch(fciqmc_t *h, int L, int *L_out) {
    int allowed = L;
    bool relaid = false;
    if (h->n_chunks > h->chunk_alloc) {   // (an earlier call had no room for the chunks' maps)
        const int rc = relayout(h);
        if (rc) return rc;
    }
    for (int s = 0; s < h->max_sys; ++s) {
        SysHost &S = h->sys[s];
        if (!S.active || S.fatal) continue;
        const SysDesc &d = h->hdesc[s];
        if (d.iter >= d.stop_at) continue;
        if (!h->planner) continue;   // overflows are left to the redo and spill paths
        const int64_t g = std::max<int64_t>(S.growth, 256);
        int64_t used = std::max<int64_t>(S.last.used, S.last.nd + 1);
        if (used + 4 * g > S.cap * 5 / 8) {
            const int64_t nc = std::max<int64_t>(cap_for_entries(used + 8 * g),
                                                 round_cap(S.cap + S.cap / 2));
            const int rc = rebucket_system(h, s, nc, 0);
            if (rc) return rc;
        }
        // Many records per determinant (a lattice: one to twenty) would make buckets planned
        // by their entries merge in several rounds, from memory: more buckets then, unless
        // the device has no room for them.
        if (S.last.spawns > S.cap / BQ * (BUCKET_RECS + BUCKET_RECS / 2) && !S.no_split) {
            const int64_t nc = round_cap(S.last.spawns / BUCKET_RECS * BQ);
            bool fits = false;
            int rc = split_fits(h, S, nc, &fits);
            if (rc) return rc;
            if (fits) rc = rebucket_system(h, s, nc, 0);
            if (!fits || rc == FCIQMC_ECAPACITY) S.no_split = true;
            else if (rc) return rc;
        }
        const int64_t room = (S.cap * 5 / 8 - used) / g;
        allowed = (int)std::max<int64_t>(1, std::min<int64_t>(allowed, room));
        // Record slots per bucket: the fullest bucket of the last launch with half as much
        // again, growing at the launch's largest rate. Before anything is known: one per
        // walker, spread over the buckets, and what the list's largest population sends to
        // one child, tau |H| |C| (a list that starts on the reference sends thousands to
        // each of its few neighbours on a lattice; a re-run costs a system the rest of the
        // launch). Given back when four times too many.
        const int64_t nb = S.cap / BQ;
        const double peak = S.rec_peak > 0 ? (double)S.rec_peak
                                           : (double)std::max<int64_t>(S.last.nw, 1) / (double)nb +
                                                 S.prm.tau * S.h_max * (double)S.pop_max;
        const double grow = std::min(std::pow(S.spawn_rate, (double)std::min(allowed, 8)), 4.0);
        const double fullest = 1.5 * peak * grow + 16.0;
        int64_t want = std::max(min_slots(h, nb), round_slots(std::min(fullest, 1e12)));
        // As many for every bucket as the fullest needs, up to 8 slots (128 B) per walker or
        // 2^21 in all; where records crowd into few buckets, those get the rest as extensions
        // (a pass over the buckets before the launch), by what each received in the last
        // iteration. Without such a count (the buckets are new) one iteration is tried: if
        // it overflows it is re-run, from its own counts.
        const int64_t most = std::max<int64_t>((int64_t)1 << 21, 8 * S.last.nw) / nb / 8 * 8;
        S.crowded = want > std::max(most, min_slots(h, nb));
        if (S.crowded) {
            want = std::max(most, min_slots(h, nb));
            S.ext_factor = 1.5 * grow;
            if (!S.counted) allowed = 1;
        }
        if (want > S.rec_r || 4 * want < S.rec_r) {
            S.rec_r = want;
            relaid = true;
        }
        if (S.spawn_rate > 1.0) {
            const double fit = std::log((S.crowded ? fullest : (double)S.rec_r) / (1.25 * peak)) /
                               std::log(S.spawn_rate);
            allowed = (int)std::max<double>(1.0, std::min<double>((double)allowed, std::floor(fit)));
        }
    }
    // (a buffer that an earlier call could not make larger is gone: asked for again, so that
    // no launch runs without the slots its descriptors name)
    if (relaid || h->rec_base > h->rec_cap) {
        const int rc = layout_records(h);
        if (rc) return rc;
    }
    const int rc = extend_buckets(h);
    if (rc) return rc;
    *L_out = allowed;
    return 0;
}

// Launch L iterations (graph or direct), then read records and statuses. With
// `sample` the last iteration runs as direct launches bracketed by events, which
// gives the per-phase device times of one iteration on the graph path too.
int run_iterations(fciqmc_t *h, int L, bool sample) {
    std::vector<int> redo;
    std::vector<int> spilled;
    std::vector<int64_t> before(h->max_sys);
    for (int s = 0; s < h->max_sys; ++s) before[s] = h->hdesc[s].iter;
    int rc = ensure_tile_map(h);
    if (rc) return rc;
    for (int s = 0; s < h->max_sys; ++s)
        if (h->sys[s].active) h->hdesc[s].nw = h->sys[s].last.nw;
    rc = upload_desc(h);
    if (rc) return rc;
    const Shape sh = launch_shape(h);
    EngineArgs a = make_args(h);
    a.wsh = sh.wsh;
    a.post_seg = sh.post_seg;
    if (h->profiling) {
        for (int i = 0; i < L; ++i) {
            FQ_LAUNCH(h->W, launch_iteration, a, sh.post_grid, sh.spawn_grid, i == 0, h->stream, h->ev);
            HIP_TRY(hipEventSynchronize(h->ev[NKERN]));
            for (int k = 0; k < NKERN; ++k) {
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, h->ev[k], h->ev[k + 1]));
                h->kms[k] += ms;
                h->kcount[k]++;
            }
        }
        HIP_TRY(hipGetLastError());
    } else if (h->use_graph) {
        const int Lg = sample ? L - 1 : L;
        if (Lg > 0) {
            hipGraphExec_t ex = nullptr;
            rc = capture_or_get(h, Lg, &ex);
            if (rc) return rc;
            HIP_TRY(hipGraphLaunch(ex, h->stream));
        }
        if (sample) {
            FQ_LAUNCH(h->W, launch_iteration, a, sh.post_grid, sh.spawn_grid, true, h->stream, h->ev);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipEventSynchronize(h->ev[NKERN]));
            for (int k = 0; k < NKERN; ++k) {
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, h->ev[k], h->ev[k + 1]));
                h->phase_ms[k] = ms;
            }
        }
    } else {
        for (int i = 0; i < L; ++i)
        FQ_LAUNCH(h->W, launch_iteration, a, sh.post_grid, sh.spawn_grid, i == 0, h->stream, nullptr);
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipStreamSynchronize(h->stream));
    rc = download_desc(h);
    if (rc) return rc;
    for (int s = 0; s < h->max_sys; ++s) {
        SysHost &S = h->sys[s];
        if (!S.active) continue;
        SysDesc &d = h->hdesc[s];
        S.counted = true;   // (an abandoned iteration counts its records as well)
        const int64_t n_new = d.iter - before[s];
        if (n_new > 0) {
            // the stream has been synchronised: the records are in host memory
            const IterRecord *rr = h->h_rec + (int64_t)s * REC_CAP;
            int64_t prev_used = S.last.used, seen = 0;
            for (int64_t it = before[s] + 1; it <= d.iter; ++it) {
                const IterRecord &r = rr[it % REC_CAP];
                seen = std::max<int64_t>(seen, r.used - prev_used);
                prev_used = r.used;
                S.tot_att += r.attempts;
                S.tot_sp += r.spawns;
                if (r.varying && r.iter - r.n_var >= S.prm.avg_start) {
                    S.e_blk.add(r.num, (double)r.c0);
                    S.s_blk.add(r.shift, 1.0);
                }
                S.last = r;
            }
            // headroom estimates for the next launch: the largest growth of the entries in
            // this one, with 25 % slack, its fullest bucket of records and the mean growth
            // of the record count per iteration
            S.growth = std::max<int64_t>(256, seen + seen / 4);
            S.rec_peak = 1;
            for (int64_t it = before[s] + 1; it <= d.iter; ++it)
                S.rec_peak = std::max(S.rec_peak, rr[it % REC_CAP].rec_max);
            const int64_t sp0 = rr[(before[s] + 1) % REC_CAP].spawns, sp1 = S.last.spawns;
            S.spawn_rate = 1.0;
            if (n_new > 1 && sp0 > 0 && sp1 > sp0)
                S.spawn_rate = std::min(std::pow((double)sp1 / (double)sp0, 1.0 / (double)(n_new - 1)), 4.0);
        }
        uint32_t &st = h->hstatus[s];
        if (st & ST_TABLE_FULL) {
            // a bucket's record slots overflowed: this iteration was abandoned and runs again
            st &= ~ST_TABLE_FULL;
            S.redos += 1;
            rc = reset_spawns(h, s);
            if (rc) return rc;
            redo.push_back(s);
        }
        if (st & ST_SPILLED) {
            st &= ~ST_SPILLED;
            S.spills += 1;
            spilled.push_back(s);
        }
        if (st) {
            S.fatal = (st & ST_SPILL_FULL) ? FCIQMC_ECAPACITY : FCIQMC_EOVERFLOW;
            return set_err(S.fatal,
                           "system " + std::to_string(s) + ": status " + std::to_string(st) +
                               ((st & ST_DIED) ? " (walkers died out)"
                                : (st & ST_SPILL_FULL) ? " (more new determinants than the spill list holds)"
                                                       : " (population overflow)"));
        }
    }
    for (int s : redo) {
        // the abandoned iteration counted its dropped records: slots for the fullest bucket
        uint32_t most = 0;
        HIP_TRY(hipMemcpyAsync(&most, h->d_rec_max + s, sizeof most, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipMemsetAsync(h->d_rec_max + s, 0, sizeof most, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        h->sys[s].rec_peak = most;
        if (h->planner) continue;   // (plan_launch lays them out)
        h->sys[s].rec_r = std::max(h->sys[s].rec_r + 8, round_slots(1.5 * (double)most + 16.0));
        rc = layout_records(h);
        if (rc) return rc;
    }
    if (!spilled.empty()) {
        unsigned long long n_sp = 0;
        HIP_TRY(hipMemcpyAsync(&n_sp, h->d_sp_count, sizeof n_sp, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        const int64_t n_take = std::min<int64_t>((int64_t)n_sp, h->sp_cap);
        for (int s : spilled) {
            SysHost &S = h->sys[s];
            const int64_t used = std::max<int64_t>(S.last.used, S.last.nd + 1) + n_take;
            const int64_t nc = std::max<int64_t>(cap_for_entries(used + 8 * S.growth),
                                                 round_cap(2 * S.cap));
            rc = rebucket_system(h, s, nc, n_take);
            if (rc) return rc;
        }
        HIP_TRY(hipMemsetAsync(h->d_sp_count, 0, sizeof(unsigned long long), h->stream));
    }
    return 0;
}

int iterate_each(fciqmc_t *h, const std::vector<int64_t> &n) {
    hipEvent_t t0, t1;
    HIP_TRY(hipEventCreate(&t0));
    HIP_TRY(hipEventCreate(&t1));
    HIP_TRY(hipEventRecord(t0, h->stream));
    for (int s = 0; s < h->max_sys; ++s)
        if (h->sys[s].active) h->hdesc[s].stop_at = h->hdesc[s].iter + std::max<int64_t>(n[s], 0);
    for (;;) {
        int64_t rem = 0;
        for (int s = 0; s < h->max_sys; ++s)
            if (h->sys[s].active && !h->sys[s].fatal)
                rem = std::max<int64_t>(rem, h->hdesc[s].stop_at - h->hdesc[s].iter);
        if (rem <= 0) break;
        int L = 0;
        int rc = plan_launch(h, (int)std::min<int64_t>(rem, MAX_GRAPH_ITERS), &L);
        if (rc) return rc;
        // the launch that ends the call samples the per-phase times of its last iteration
        rc = run_iterations(h, L, L >= rem);
        if (rc) return rc;
    }
    HIP_TRY(hipEventRecord(t1, h->stream));
    HIP_TRY(hipEventSynchronize(t1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, t0, t1));
    h->ms_last = ms;
    hipEventDestroy(t0);
    hipEventDestroy(t1);
    return 0;
}

// Entries of the spill list (new determinants that did not fit their bucket).
constexpr int64_t SPILL_CAP = (int64_t)1 << 16;

// Address of the staging area on each device (resolved once per device, with
// that device current).
constexpr int MAX_DEVICES = 64;
std::mutex g_stage_mu;
void *g_stage_ptr[MAX_DEVICES] = {};

int resolve_stage(int dev, void **out) {
    if (dev < 0 || dev >= MAX_DEVICES) return set_err(FCIQMC_EDEVICE, "device index out of range");
    std::lock_guard<std::mutex> lock(g_stage_mu);
    if (!g_stage_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return set_err(FCIQMC_EDEVICE, "staging area has no device address");
        g_stage_ptr[dev] = p;
    }
    *out = g_stage_ptr[dev];
    return 0;
}

int create_handle(int max_slots, void *stream, int W, fciqmc_t **out) {
    fciqmc_t *h = new (std::nothrow) fciqmc_t();
    if (!h) return set_err(FCIQMC_ENOMEM, "host allocation failed");
    h->W = W;
    HIP_TRY(hipGetDevice(&h->dev));
    {
        const int rc = resolve_stage(h->dev, &h->d_stage);
        if (rc) {
            delete h;
            return rc;
        }
    }
    if (stream) {
        h->stream = (hipStream_t)stream;
    } else {
        HIP_TRY(hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking));
        h->own_stream = true;
    }
    h->max_sys = max_slots;
    h->sys.resize(max_slots);
    h->hdesc.assign(max_slots, SysDesc{});
    h->hstatus.assign(max_slots, 0u);
    HIP_TRY(hipMalloc(&h->d_desc, sizeof(SysDesc) * max_slots));
    HIP_TRY(hipMalloc(&h->d_status, sizeof(uint32_t) * max_slots));
    HIP_TRY(hipMalloc(&h->d_work, sizeof(unsigned int) * N_WORK));
    HIP_TRY(hipMemsetAsync(h->d_work, 0, sizeof(unsigned int) * N_WORK, h->stream));
    HIP_TRY(hipMalloc(&h->d_spawns, sizeof(unsigned long long) * SPAWN_SLOTS * max_slots));
    HIP_TRY(hipMemsetAsync(h->d_spawns, 0, sizeof(unsigned long long) * SPAWN_SLOTS * max_slots,
                           h->stream));
    HIP_TRY(hipHostMalloc((void **)&h->h_rec, sizeof(IterRecord) * REC_CAP * max_slots,
                          hipHostMallocDefault));
    std::memset(h->h_rec, 0, sizeof(IterRecord) * REC_CAP * max_slots);
    HIP_TRY(hipHostGetDevicePointer((void **)&h->d_rec, h->h_rec, 0));
    HIP_TRY(hipMalloc(&h->d_total, N_TOTAL * sizeof(unsigned long long)));
    HIP_TRY(hipMemsetAsync(h->d_total, 0, N_TOTAL * sizeof(unsigned long long), h->stream));
    HIP_TRY(hipMalloc(&h->d_nchunks, sizeof(int64_t)));
    HIP_TRY(hipMalloc(&h->d_step, sizeof(unsigned long long)));
    HIP_TRY(hipMemsetAsync(h->d_step, 0, sizeof(unsigned long long), h->stream));
    HIP_TRY(hipMalloc(&h->d_acc, sizeof(IterStat) * ACC_SLOTS * max_slots));
    HIP_TRY(hipMemsetAsync(h->d_acc, 0, sizeof(IterStat) * ACC_SLOTS * max_slots, h->stream));
    HIP_TRY(hipMalloc(&h->d_c0, sizeof(int64_t) * max_slots));
    HIP_TRY(hipMalloc(&h->d_err, sizeof(uint32_t)));
    HIP_TRY(hipMalloc(&h->d_count, sizeof(unsigned long long)));
    HIP_TRY(hipMalloc(&h->d_rec_max, sizeof(uint32_t) * max_slots));
    HIP_TRY(hipMemsetAsync(h->d_rec_max, 0, sizeof(uint32_t) * max_slots, h->stream));
    HIP_TRY(hipMalloc(&h->d_d0acc, sizeof(long long) * max_slots));
    HIP_TRY(hipMemsetAsync(h->d_d0acc, 0, sizeof(long long) * max_slots, h->stream));
    h->sp_cap = SPILL_CAP;
    HIP_TRY(hipMalloc(&h->d_spill, (size_t)h->sp_cap * (16 + 8 * h->W)));
    HIP_TRY(hipMalloc(&h->d_sp_count, sizeof(unsigned long long)));
    HIP_TRY(hipMemsetAsync(h->d_sp_count, 0, sizeof(unsigned long long), h->stream));
    HIP_TRY(hipMalloc(&h->d_spilled, sizeof(uint32_t) * max_slots));
    HIP_TRY(hipMemsetAsync(h->d_spilled, 0, sizeof(uint32_t) * max_slots, h->stream));
    for (int k = 0; k <= NKERN; ++k) HIP_TRY(hipEventCreate(&h->ev[k]));
    h->spawn_grid = spawn_grid_size(W);
    h->post_grid = post_grid_size();
    int rc = upload_desc(h);
    if (rc) return rc;
    rc = relayout(h);
    if (rc) return rc;
    *out = h;
    return 0;
}

}  // namespace

namespace {
int compute_e0(fciqmc_t *h, int s) {
    double *d_out = nullptr;
    HIP_TRY(hipMalloc(&d_out, 8));
    int rc = upload_desc(h);
    if (rc) return rc;
    HIP_TRY(FQ_LAUNCH(h->W, launch_e0, h->d_desc, s, hlo(h->sys[s].d0), hhi(h->sys[s].d0), d_out,
                      h->stream));
    double e0 = 0;
    HIP_TRY(hipMemcpyAsync(&e0, d_out, 8, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    hipFree(d_out);
    h->sys[s].e0 = e0;
    h->hdesc[s].e0 = e0;
    return 0;
}

int admit_full(fciqmc_t *h, int s, const fciqmc_hamiltonian *ham, const fciqmc_params *prm) {
    const int64_t floor0 = h->rec_floor;
    int rc = admit(h, s, ham, prm);
    if (!rc) rc = compute_e0(h, s);
    if (!rc && prm->spawn_capacity > 0) {   // the record buffer is shared by the handle's systems
        h->rec_floor = std::max(h->rec_floor, prm->spawn_capacity);
        rc = ensure_records(h, prm->spawn_capacity);
    }
    if (rc) {   // the slot is free again
        const std::string keep = g_err;
        SysHost &S = h->sys[s];
        if (S.block) {
            (void)hipStreamSynchronize(h->stream);
            hipFree(S.block);
        }
        S = SysHost();
        h->rec_floor = floor0;
        h->hdesc[s] = SysDesc{};
        h->hstatus[s] = 0;
        relayout(h);
        upload_desc(h);
        g_err = keep;
        return rc;
    }
    const int64_t n0 = prm->initial_walkers > 0 ? prm->initial_walkers : 10;
    h->sys[s].last = IterRecord{};
    h->sys[s].last.nw = n0;
    h->sys[s].last.nd = 1;
    h->sys[s].last.c0 = n0;
    h->sys[s].last.shift = prm->initial_shift;
    return upload_desc(h);
}

void release(fciqmc_t *h) {
    if (!h) return;
    hipStreamSynchronize(h->stream);
    drop_graphs(h);
    for (auto &S : h->sys)
        if (S.block) hipFree(S.block);
    hipFree(h->d_desc);
    if (h->h_rec) hipHostFree(h->h_rec);
    hipFree(h->d_status);
    hipFree(h->d_work);
    hipFree(h->d_spawns);
    hipFree(h->d_total);
    hipFree(h->d_nchunks);
    hipFree(h->d_step);
    hipFree(h->d_acc);
    hipFree(h->d_c0);
    hipFree(h->d_err);
    hipFree(h->d_count);
    hipFree(h->d_chunk_sys);
    hipFree(h->d_chunk_local);
    hipFree(h->d_unlisted);
    hipFree(h->d_tiles);
    hipFree(h->d_recs);
    hipFree(h->d_rec_max);
    hipFree(h->d_bhist);
    hipFree(h->d_bprev);
    hipFree(h->d_bext);
    hipFree(h->d_d0acc);
    hipFree(h->d_spill);
    hipFree(h->d_sp_count);
    hipFree(h->d_spilled);
    for (auto &e : h->ev)
        if (e) hipEventDestroy(e);
    if (h->own_stream) hipStreamDestroy(h->stream);
    delete h;
}

int64_t walkers_out(fciqmc_t *h, int s, uint64_t *det, int32_t *pop, uint32_t *flags, int64_t cap) {
    if (!h || s < 0 || s >= h->max_sys || !h->sys[s].active)
        return set_err(FCIQMC_ESTATE, "slot is not active");
    int64_t n = 0;
    const int rc = list_out(h, s, det, pop, flags, cap, &n);
    return rc ? rc : n;
}
}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *fciqmc_last_error(void) { return g_err.c_str(); }

int fciqmc_batch_create(int32_t max_slots, int32_t n, const fciqmc_hamiltonian *hams,
                        const fciqmc_params *prms, void *hip_stream, fciqmc_t **out) {
    if (!out) return set_err(FCIQMC_EINVAL, "null output handle");
    *out = nullptr;
    if (max_slots < 1 || n < 0 || n > max_slots) return set_err(FCIQMC_EINVAL, "bad slot counts");
    if (n > 0 && (!hams || !prms)) return set_err(FCIQMC_EINVAL, "null hamiltonians or params");
    for (int i = 0; i < n; ++i) {
        int rc = validate(&hams[i], &prms[i]);
        if (rc) return rc;
    }
    // one determinant width for the batch: the first system's (one word when empty)
    const int W = n > 0 ? words_for(hams[0].n_orb, prms[0].det_words) : 1;
    for (int i = 1; i < n; ++i)
        if (words_for(hams[i].n_orb, prms[i].det_words) != W)
            return set_err(FCIQMC_EINVAL, "a batch holds determinants of one width (64-bit words)");
    fciqmc_t *h = nullptr;
    int rc = create_handle(max_slots, hip_stream, W, &h);
    if (rc) {
        release(h);
        return rc;
    }
    for (int i = 0; i < n; ++i) {
        rc = admit_full(h, i, &hams[i], &prms[i]);
        if (rc) {
            std::string keep = g_err;
            release(h);
            g_err = keep;
            return rc;
        }
    }
    *out = h;
    return 0;
}

int fciqmc_init(const fciqmc_hamiltonian *ham, const fciqmc_params *prm, void *hip_stream,
                fciqmc_t **out) {
    return fciqmc_batch_create(1, 1, ham, prm, hip_stream, out);
}

int fciqmc_free(fciqmc_t *h) {
    release(h);
    return 0;
}

int fciqmc_iterate(fciqmc_t *h, int32_t n_iterations) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (n_iterations < 0) return set_err(FCIQMC_EINVAL, "negative iteration count");
    std::vector<int64_t> n(h->max_sys, n_iterations);
    return iterate_each(h, n);
}

int fciqmc_batch_iterate(fciqmc_t *h, int32_t n_iterations) { return fciqmc_iterate(h, n_iterations); }

int fciqmc_batch_iterate_each(fciqmc_t *h, const int32_t *n_iter) {
    if (!h || !n_iter) return set_err(FCIQMC_EINVAL, "null argument");
    std::vector<int64_t> n(h->max_sys);
    for (int s = 0; s < h->max_sys; ++s) n[s] = n_iter[s];
    return iterate_each(h, n);
}

int fciqmc_estimators(fciqmc_t *h, fciqmc_estimates *out) {
    if (!h || !out) return set_err(FCIQMC_EINVAL, "null argument");
    return fill_estimates(h, 0, out);
}

int fciqmc_batch_slot_estimators(fciqmc_t *h, int32_t slot, fciqmc_estimates *out) {
    if (!h || !out || slot < 0 || slot >= h->max_sys) return set_err(FCIQMC_EINVAL, "bad argument");
    return fill_estimates(h, slot, out);
}

int32_t fciqmc_det_words(const fciqmc_t *h) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    return h->W;
}

int64_t fciqmc_walkers(fciqmc_t *h, uint64_t *det, int32_t *pop, uint32_t *flags, int64_t cap) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    return walkers_out(h, 0, det, pop, flags, cap);
}

int64_t fciqmc_batch_slot_walkers(fciqmc_t *h, int32_t slot, uint64_t *det, int32_t *pop,
                                  uint32_t *flags, int64_t cap) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    return walkers_out(h, slot, det, pop, flags, cap);
}

int fciqmc_load_walkers(fciqmc_t *h, const uint64_t *det, const int32_t *pop, int64_t n,
                        int64_t iteration, double shift, int64_t n_prev, int32_t varying,
                        int64_t n_var) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (n < 0 || (n > 0 && (!det || !pop)) || iteration < 0)
        return set_err(FCIQMC_EINVAL, "bad walker list");
    const int s = 0;
    SysHost &S = h->sys[s];
    if (!S.active) return set_err(FCIQMC_ESTATE, "slot is not active");
    // Checked, summed and (if it does not ascend) searched for repeats on the device: reading
    // out and loading back 1.35e6 determinants took 220 ms with the checks on the host, 5.6
    // with them here.
    ListBuf b;
    ListCheck c;
    int rc = b.upload(h, det, pop, n);
    if (rc) return rc;
    HIP_TRY(hipMalloc(&b.check, sizeof c));
    HIP_TRY(hipMemcpyAsync(b.check, &c, sizeof c, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(FQ_LAUNCH(h->W, launch_check_list, h->d_desc, s, b.det, b.pop, n, S.na, S.nb, b.check,
                      h->stream));
    HIP_TRY(hipMemcpyAsync(&c, b.check, sizeof c, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    if (c.bad != ~0ull) switch (c.bad & 7) {
        case LIST_COUNTS:
            return set_err(FCIQMC_EINVAL, "determinant with wrong electron counts in walker list");
        case LIST_RANGE:
            return set_err(FCIQMC_EINVAL, "population out of range");
        case LIST_SPACE:
            return set_err(FCIQMC_EINVAL, "determinant outside the restricted space in walker list");
        default:
            return set_err(FCIQMC_EINVAL, "a list of spin-coupled functions holds each as the "
                                          "smaller determinant of its pair");
    }
    if (c.unsorted && c.nd > 1) {
        rc = holds_twice(h, b, det, pop, n, c);
        if (rc) return rc;
        if (c.twice) return set_err(FCIQMC_EINVAL, "duplicate determinant in walker list");
    }
    SysDesc &d = h->hdesc[s];
    d.iter = iteration;
    d.shift = shift;
    d.n_prev = n_prev;
    d.varying = varying ? 1 : 0;
    d.n_var = n_var;
    rc = load_entries(h, s, b.det, b.pop, n, (int64_t)c.nd, c.have_ref != 0, c.most);
    if (rc) return rc;
    S.e_blk.clear();
    S.s_blk.clear();
    S.fatal = 0;
    IterRecord r{};
    r.c0 = c.c0;
    r.nw = (int64_t)c.nw;
    r.nd = (int64_t)c.nd;
    r.num = NAN;
    r.shift = d.shift;
    S.last = r;
    return upload_desc(h);
}

int fciqmc_set_shift(fciqmc_t *h, double shift, int32_t varying) {
    if (!h || !h->sys[0].active) return set_err(FCIQMC_EINVAL, "null handle");
    SysDesc &d = h->hdesc[0];
    d.shift = shift;
    d.varying = varying ? 1 : 0;
    if (varying) {
        d.n_prev = h->sys[0].last.nw;
        d.n_var = d.iter;
    }
    h->sys[0].e_blk.clear();
    h->sys[0].s_blk.clear();
    return upload_desc(h);
}

int fciqmc_reserve(fciqmc_t *h, int64_t slots) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (slots < 0) return set_err(FCIQMC_EINVAL, "slots must be >= 0");
    const int64_t want = round_cap(slots);
    for (int s = 0; s < h->max_sys; ++s) {
        SysHost &S = h->sys[s];
        if (!S.active || S.fatal || S.cap >= want) continue;
        const int rc = rebucket_system(h, s, want, 0);
        if (rc) return rc;
    }
    return 0;
}

int fciqmc_batch_admit(fciqmc_t *h, const fciqmc_hamiltonian *ham, const fciqmc_params *prm,
                       int32_t *slot) {
    if (!h || !slot) return set_err(FCIQMC_EINVAL, "null argument");
    int s = -1;
    for (int i = 0; i < h->max_sys; ++i)
        if (!h->sys[i].active) {
            s = i;
            break;
        }
    if (s < 0) return set_err(FCIQMC_ESTATE, "no free slot");
    int rc = admit_full(h, s, ham, prm);
    if (rc) return rc;
    *slot = s;
    return 0;
}

int fciqmc_batch_retire(fciqmc_t *h, int32_t slot) {
    if (!h || slot < 0 || slot >= h->max_sys || !h->sys[slot].active)
        return set_err(FCIQMC_ESTATE, "slot is not active");
    HIP_TRY(hipStreamSynchronize(h->stream));
    SysHost &S = h->sys[slot];
    if (S.block) HIP_TRY(hipFree(S.block));
    S = SysHost();
    h->hdesc[slot] = SysDesc{};
    h->hstatus[slot] = 0;
    int rc = relayout(h);
    if (rc) return rc;
    return upload_desc(h);
}

int32_t fciqmc_batch_active(fciqmc_t *h) {
    if (!h) return 0;
    int32_t n = 0;
    for (auto &S : h->sys) n += S.active ? 1 : 0;
    return n;
}

int64_t fciqmc_footprint_bytes(const fciqmc_hamiltonian *ham, const fciqmc_params *prm) {
    if (!ham || !prm) return set_err(FCIQMC_EINVAL, "null argument");
    return target_footprint(ham, prm);
}

int fciqmc_set_profiling(fciqmc_t *h, int32_t on) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    h->profiling = on != 0;
    for (int k = 0; k < NKERN; ++k) {
        h->kms[k] = 0.0;
        h->kcount[k] = 0;
    }
    return 0;
}

int fciqmc_set_launch(fciqmc_t *h, int32_t spawn_grid, int32_t tile, int32_t post_grid) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (spawn_grid < 1 || post_grid < 1 || tile < 256 || tile > (1 << 20) || (tile & (tile - 1)))
        return set_err(FCIQMC_EINVAL, "launch shape out of range (tile: a power of two, 256..2^20)");
    h->spawn_grid = spawn_grid;
    h->post_grid = post_grid;
    h->tile = tile;
    h->shape_set = true;
    drop_graphs(h);
    return 0;
}

int fciqmc_get_launch(fciqmc_t *h, int32_t *spawn_grid, int32_t *tile, int32_t *post_grid) {
    if (!h || !spawn_grid || !tile || !post_grid) return set_err(FCIQMC_EINVAL, "null argument");
    *spawn_grid = h->spawn_grid;
    *tile = h->tile;
    *post_grid = h->post_grid;
    return 0;
}

// What an autotuning trial advances of one system, restored after the trials: the
// walker list, the dynamics, the statistics and the per-iteration records.
struct SysSnapshot {
    int s = 0;
    std::vector<hdet_t> det;
    std::vector<int32_t> pop;
    SysDesc desc{};
    IterRecord last{};
    int64_t tot_att = 0, tot_sp = 0, redos = 0, spills = 0, growth = 0, rec_peak = 0;
    double spawn_rate = 1.0;
    Blocker e_blk, s_blk;
    std::vector<IterRecord> ring;
};

int take_snapshot(fciqmc_t *h, int s, SysSnapshot &o) {
    SysHost &S = h->sys[s];
    Walkers w;
    const int rc = export_walkers(h, s, w);
    if (rc) return rc;
    o.s = s;
    o.det = std::move(w.det);
    o.pop = std::move(w.pop);
    o.desc = h->hdesc[s];
    o.last = S.last;
    o.tot_att = S.tot_att;
    o.tot_sp = S.tot_sp;
    o.redos = S.redos;
    o.spills = S.spills;
    o.growth = S.growth;
    o.rec_peak = S.rec_peak;
    o.spawn_rate = S.spawn_rate;
    o.e_blk = S.e_blk;
    o.s_blk = S.s_blk;
    o.ring.assign(h->h_rec + (int64_t)s * REC_CAP, h->h_rec + (int64_t)(s + 1) * REC_CAP);
    return 0;
}

int restore_snapshot(fciqmc_t *h, const SysSnapshot &o) {
    const int s = o.s;
    SysHost &S = h->sys[s];
    SysDesc &d = h->hdesc[s];
    d.iter = o.desc.iter;
    d.stop_at = o.desc.iter;
    d.shift = o.desc.shift;
    d.varying = o.desc.varying;
    d.n_prev = o.desc.n_prev;
    d.n_var = o.desc.n_var;
    const int rc = load_list(h, s, o.det, o.pop);
    if (rc) return rc;
    S.last = o.last;
    S.tot_att = o.tot_att;
    S.tot_sp = o.tot_sp;
    S.redos = o.redos;
    S.spills = o.spills;
    S.growth = o.growth;
    S.rec_peak = o.rec_peak;
    S.spawn_rate = o.spawn_rate;
    S.e_blk = o.e_blk;
    S.s_blk = o.s_blk;
    S.fatal = 0;
    std::copy(o.ring.begin(), o.ring.end(), h->h_rec + (int64_t)s * REC_CAP);
    return upload_desc(h);
}

int fciqmc_autotune(fciqmc_t *h, int32_t iters_per_trial) {
    if (!h || iters_per_trial < 1) return set_err(FCIQMC_EINVAL, "bad argument");
    int cus = fq::post_grid_size() / 4;   // (four post workgroups per CU)
    // The trials run on the live systems; their state is saved first and restored
    // afterwards, so tuning leaves every trajectory where it was.
    std::vector<SysSnapshot> snaps;
    for (int s = 0; s < h->max_sys; ++s) {
        if (!h->sys[s].active || h->sys[s].fatal) continue;
        snaps.emplace_back();
        const int rc = take_snapshot(h, s, snaps.back());
        if (rc) return rc;
    }
    const bool was = h->profiling, shape_was_set = h->shape_set;
    const int sg0 = h->spawn_grid, tl0 = h->tile, pg0 = h->post_grid;
    h->profiling = true;
    h->shape_set = true;   // (each trial runs at its own shape)
    auto give_up = [&](int rc) {   // a trial failed: the shape is again what it was
        h->spawn_grid = sg0;
        h->tile = tl0;
        h->post_grid = pg0;
        h->shape_set = shape_was_set;
        h->profiling = was;
        return rc;
    };
    auto trial = [&](int sg, int tl, int pg, double &spawn_ns, double &post_ns) -> int {
        h->spawn_grid = sg;
        h->tile = tl;
        h->post_grid = pg;
        for (int k = 0; k < NKERN; ++k) {
            h->kms[k] = 0.0;
            h->kcount[k] = 0;
        }
        int64_t a0 = 0;
        for (auto &S : h->sys) a0 += S.active ? S.tot_att : 0;
        std::vector<int64_t> n(h->max_sys, iters_per_trial);
        int rc = iterate_each(h, n);
        if (rc) return rc;
        int64_t a1 = 0;
        for (auto &S : h->sys) a1 += S.active ? S.tot_att : 0;
        spawn_ns = h->kms[2] * 1e6 / (double)std::max<int64_t>(a1 - a0, 1);
        post_ns = h->kms[3] * 1e6 / (double)iters_per_trial;   // per iteration
        return 0;
    };
    int best_sg = h->spawn_grid, best_tl = h->tile, best_pg = h->post_grid;
    double best_s = 1e300, best_p = 1e300;
    // (k_post is compiled for four resident workgroups per CU)
    const int sgs[4] = {2, 4, 8, 16}, tls[3] = {1024, 2048, 4096}, pgs[5] = {2, 3, 4, 6, 8};
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 3; ++j) {
            double sn, pn;
            int rc = trial(sgs[i] * cus, tls[j], best_pg, sn, pn);
            if (rc) return give_up(rc);
            if (sn < best_s) {
                best_s = sn;
                best_sg = sgs[i] * cus;
                best_tl = tls[j];
            }
        }
    for (int i = 0; i < 5; ++i) {
        double sn, pn;
        int rc = trial(best_sg, best_tl, pgs[i] * cus, sn, pn);
        if (rc) return give_up(rc);
        if (pn < best_p) {
            best_p = pn;
            best_pg = pgs[i] * cus;
        }
    }
    h->spawn_grid = best_sg;
    h->tile = best_tl;
    h->post_grid = best_pg;
    h->profiling = was;
    for (int k = 0; k < NKERN; ++k) {
        h->kms[k] = 0.0;
        h->kcount[k] = 0;
    }
    drop_graphs(h);
    for (const SysSnapshot &o : snaps) {
        const int rc = restore_snapshot(h, o);
        if (rc) return rc;
    }
    return 0;
}

int64_t fciqmc_history(fciqmc_t *h, int32_t slot, int64_t first, int64_t n, fciqmc_iteration *out) {
    if (!h || slot < 0 || slot >= h->max_sys || n < 0 || (n > 0 && !out))
        return set_err(FCIQMC_EINVAL, "bad argument");
    if (!h->sys[slot].active) return set_err(FCIQMC_ESTATE, "slot is not active");
    const int64_t cur = h->hdesc[slot].iter;
    const int64_t lo = std::max<int64_t>(1, cur - REC_CAP + 1);
    if (first < lo || first + n - 1 > cur) return set_err(FCIQMC_EINVAL, "iterations not in the log");
    for (int64_t i = 0; i < n; ++i) {
        const IterRecord &r = h->h_rec[(int64_t)slot * REC_CAP + (first + i) % REC_CAP];
        fciqmc_iteration &o = out[i];
        o.iteration = r.iter;
        o.n_walkers = r.nw;
        o.n_dets = r.nd;
        o.ref_pop = r.c0;
        o.attempts = r.attempts;
        o.spawns = r.spawns;
        o.merged = r.merged;
        o.aborted = r.aborted;
        o.born = r.born;
        o.entries = r.used;
        o.proj_num = r.num;
        o.shift = r.shift;
        o.shift_varying = r.varying;
        o.status = r.status;
    }
    return n;
}

int fciqmc_blocking(const double *num, const double *den, int64_t n, double *mean, double *err) {
    if (n < 0 || (n > 0 && !num) || !mean || !err) return set_err(FCIQMC_EINVAL, "bad argument");
    Blocker b;
    for (int64_t t = 0; t < n; ++t) b.add(num[t], den ? den[t] : 1.0);
    b.result(*mean, *err);
    return 0;
}

int fciqmc_set_test_options(fciqmc_t *h, int32_t planner, int64_t tile_map_limit,
                            int64_t record_capacity) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (tile_map_limit < -1) return set_err(FCIQMC_EINVAL, "tile_map_limit must be >= -1");
    if (record_capacity < 0) return set_err(FCIQMC_EINVAL, "record_capacity must be >= 0");
    h->planner = planner != 0;
    if (record_capacity > 0) {
        HIP_TRY(hipStreamSynchronize(h->stream));
        hipFree(h->d_recs);
        h->d_recs = nullptr;
        h->rec_cap = 0;
        int rc = ensure_records(h, record_capacity);
        if (rc) return rc;
        // every bucket of the handle gets its share of them
        for (SysHost &S : h->sys)
            if (S.active)
                S.rec_r = std::max<int64_t>(1, record_capacity / std::max<int64_t>(1, BPC * h->n_chunks));
        rc = layout_records(h);
        if (rc) return rc;
    }
    if (tile_map_limit != h->tile_map_limit) {
        HIP_TRY(hipStreamSynchronize(h->stream));
        hipFree(h->d_tiles);
        h->d_tiles = nullptr;
        h->tile_cap = 0;
        h->tile_map_off = false;
        h->tile_map_limit = tile_map_limit;
        drop_graphs(h);
    }
    return 0;
}

int64_t fciqmc_walkers_noalloc(fciqmc_t *h, uint64_t *det, int32_t *pop, uint32_t *flags,
                               int64_t cap) {
    if (!h) return set_err(FCIQMC_EINVAL, "null handle");
    if (cap < 0) return set_err(FCIQMC_EINVAL, "cap must be >= 0");
    const int s = 0;
    const SysHost &S = h->sys[s];
    if (!S.active) return set_err(FCIQMC_ESTATE, "slot is not active");
    if (h->W != 1)
        return set_err(FCIQMC_ESTATE, "the staging export holds one-word determinants only");
    HIP_TRY(launch_stage_compact(S.key, S.pop, S.bcnt, S.cap / BQ, h->d_stage, h->stream));
    unsigned long long n = 0;
    HIP_TRY(hipMemcpyAsync(&n, h->d_stage, sizeof n, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(hipStreamSynchronize(h->stream));
    if ((int64_t)n > NOALLOC_MAX_DETS)
        return set_err(FCIQMC_ECAPACITY, "walker list of " + std::to_string(n) +
                                             " determinants exceeds the staging limit of " +
                                             std::to_string(NOALLOC_MAX_DETS));
    const int64_t m = std::min<int64_t>((int64_t)n, cap);
    if (m > 0 && (det || pop || flags)) {
        HIP_TRY(launch_stage_sort(h->d_stage, (int64_t)n, h->stream));
        if (flags)
            HIP_TRY(launch_stage_flags(h->d_stage, m, S.prm.initiator_threshold, hlo(S.d0), h->stream));
        const char *p = (const char *)h->d_stage;
        if (det)
            HIP_TRY(hipMemcpyAsync(det, p + NOALLOC_KEYS_OFF, (size_t)m * 8, hipMemcpyDeviceToHost,
                                   h->stream));
        if (pop)
            HIP_TRY(hipMemcpyAsync(pop, p + NOALLOC_VALS_OFF, (size_t)m * 4, hipMemcpyDeviceToHost,
                                   h->stream));
        if (flags)
            HIP_TRY(hipMemcpyAsync(flags, p + NOALLOC_FLAGS_OFF, (size_t)m * 4,
                                   hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
    }
    return (int64_t)n;
}

int fciqmc_kernel_times(fciqmc_t *h, double ms[5], int64_t counts[5]) {
    if (!h || !ms || !counts) return set_err(FCIQMC_EINVAL, "null argument");
    for (int k = 0; k < NKERN; ++k) {
        ms[k] = h->kms[k];
        counts[k] = h->kcount[k];
    }
    return 0;
}

}  // extern "C"
