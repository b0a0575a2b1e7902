// Internal layout shared by the kernels and the host engine of libfciqmc.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fq {

constexpr int BQ = 256;              // entries per bucket of the main list (a wavefront's unit
                                     // in annihilation: four per lane)
constexpr int CHUNK = 1024;          // four consecutive buckets: one workgroup's unit in
                                     // annihilation
constexpr int BPC = CHUNK / BQ;      // buckets per chunk
constexpr int BUCKET_FILL = 128;     // planned mean entries per bucket (half full)
constexpr int BUCKET_RECS = 32;      // planned mean spawn records per bucket at most: a
                                     // wavefront merges 64 in one round
constexpr int NCLASS = 16;           // symmetry classes: 2 spins x up to 8 abelian irreps
constexpr int REC_CAP = 256;         // per-system ring of per-iteration records
constexpr int MAX_GRAPH_ITERS = 64;  // iterations captured in one graph launch
// Lists of work (spawn tiles, windows of chunks) with a counter each, and where the
// counters lie: each on a 128-byte line of its own. Tiles: three sets of lists (even and
// odd steps, a launch's first), and per set the buckets whose tiles were not listed.
constexpr int NLIST = 32;
constexpr int CTR_STRIDE = 32;                                    // unsigned ints
constexpr int CTR_SPAWN(int l) { return l * CTR_STRIDE; }
constexpr int CTR_POST(int l) { return (NLIST + l) * CTR_STRIDE; }
constexpr int CTR_FALLBACK = 2 * NLIST * CTR_STRIDE;
constexpr int N_WORK = CTR_FALLBACK + CTR_STRIDE;
constexpr int CTR_TILES(int h, int l) { return (h * NLIST + l) * (CTR_STRIDE / 2); }
constexpr int CTR_UNLISTED(int h) { return (3 * NLIST + h) * (CTR_STRIDE / 2); }
constexpr int N_TOTAL = CTR_UNLISTED(3);
constexpr int TILE_MAX_SH(int W) { return W == 1 ? 9 : 8; }   // log2 of a wavefront's largest
                                     // spawn tile (W words per determinant)
constexpr int SPAWN_SLOTS = 16;      // shares of a system's spawning-event counter
constexpr int ACC_SLOTS = 64;        // shares of a system's iteration statistics

// Status bits set on the device.
constexpr uint32_t ST_TABLE_FULL = 1u;     // the spawn-record buffer overflowed: the iteration
                                           // is abandoned, the buffer grown, the iteration redone
constexpr uint32_t ST_POP_OVERFLOW = 2u;   // a population left int32
constexpr uint32_t ST_DIED = 4u;           // N_w reached zero
constexpr uint32_t ST_SPAWN_OVERFLOW = 8u; // one spawning event would create > 2^30 walkers
constexpr uint32_t ST_SPILLED = 16u;       // new determinants did not fit their bucket: the
                                           // iteration completed with them in the spill list,
                                           // the system pauses until the host re-buckets
constexpr uint32_t ST_SPILL_FULL = 32u;    // the spill list itself overflowed (fatal)


struct IterRecord {
    int64_t iter;      // completed iterations after this one
    int64_t nw, nd, c0, attempts, spawns, merged, aborted;
    int64_t born;      // determinants that entered the main list
    int64_t used;      // entries in the buckets after the iteration (occupied + the reference)
    int64_t n_var, n_prev;
    int64_t rec_max;   // most spawn records of one bucket
    double num, shift;
    int32_t varying, status;
};

// Statistics of an iteration (a share of them). In k_post's lanes three of the counts are
// kept in one word, each below 2^21: entries | merged spawn targets << 21 | occupied << 42.
struct __attribute__((aligned(128))) IterStat {
    int64_t nw, nd, merged, aborted, used, born;
    double num;
};
constexpr int CNT_SHIFT_MERGED = 21, CNT_SHIFT_ND = 42;
constexpr int POST_WAVES = BPC;   // wavefronts of a k_post workgroup: one bucket and one
                                   // of a chunk each
constexpr uint64_t CNT_FIELD = (1ull << 21) - 1;

// Per-system descriptor, resident in device memory. The first block is
// written by the host at admission / growth; the second block is updated by
// the finalize kernel every iteration.
struct SysDesc {
    // --- set by the host
    int32_t active, M, N, n_so;
    int32_t A, n_a, n_class, pad1;  // n_class: 2 x (largest irrep label + 1)
    double tau, zeta, e0, e_core, p_double, p_single;
    double inv_p_double, inv_p_single;   // 1/P_double, 1/P_single (0 when the type is impossible)
    // With no point group (two classes, the spins) every determinant has n_emp[s]
    // empty orbitals of spin s, and a double excitation's pgen is pgen_c1[s] (both
    // electrons of spin s) or pgen_c1[2 + s] (unlike spins, first hole of spin s);
    // 0 where the case cannot occur.
    double pgen_c1[4];
    int32_t n_emp[2];
    int64_t target;
    uint64_t seed, d0, valid;
    uint64_t cmask[NCLASS];
    uint64_t irr_packed[2];          // 4 bits per spatial orbital
    const double *h1, *eri;
    const double *jk;                // [n_so][64]: (pp|qq) - (pq|qp) for p < q, spin orbitals
    const double *t3;                // [n_so][64][64]: (pa|qq) - d(s_p,s_q)(pq|qa), same-spin p, a
    // Rejection bounds of the spawning kernel, over spatial orbital pairs [32 W][32 W] in
    // half precision, rounded up, relative to their largest. With mostly double
    // excitations (p_double >= 1/2): s with |(pa|qb)| <= s_pa s_qb. Otherwise: the largest
    // |<D'|H|D>| of a single excitation p -> a.
    const uint16_t *bound;
    // A double with type word w0 is rejected when (float)w0 > bound x bound_f[pgen index]
    // (no point group) or (float)w0 pgen > bound x bound_ft; a single of nt choices when
    // (float)w0 sg_mul - sg_sub (its uniform, rounded down) > bound x nt x bound_ft.
    float bound_f[4], bound_ft, sg_mul, sg_sub;
    uint32_t dbl_thr;                // w0 <= dbl_thr: a double excitation (U < P_double)
    int32_t has_double, defer;       // P_double > 0; single excitations are rare (>= 1/2)
    // Main list: nb buckets of BQ entries (structure of arrays); a determinant lives
    // in bucket floor(mix64(D) nb / 2^64), the entries of bucket b are the first
    // bcnt[b] of [b BQ, (b+1) BQ), every one occupied (the reference may sit at 0).
    uint64_t *key;                   // determinant
    int32_t *pop;                    // signed walker count
    double *hdiag;                   // stored H_DD
    int32_t *bcnt;                   // entries per bucket
    uint64_t cap;                    // nb * BQ
    int64_t nbuckets;                // nb
    int64_t nchunks, gchunk0;        // chunks (nb / BPC) of this system and the first global one
    // Spawn records: bucket b's go to slots [rec0 + b rec_r, rec0 + (b + 1) rec_r) of the
    // handle's record buffer.
    int64_t rec0, rec_r;
    int64_t stop_at;                 // iterate while iter < stop_at
    // Restricted space (FCIQMC_SPACE_* bits; children outside it are null excitations).
    int32_t space, max_ex, max_sen, pad2;
    uint64_t frz_occ, frz_emp;
    // Spin-coupled functions (Sec. 5.3): hphf = 0 (determinants), +1 / -1 (even / odd
    // total spin); lam = hphf (-1)^{N/2}, the relative sign of a pair's determinants.
    int32_t hphf, lam;
    // --- updated on the device
    int64_t iter;
    double shift;
    int32_t varying, pad3;
    int64_t n_prev, n_var;
    int64_t nw;                      // walkers, i.e. the next iteration's attempts
    // --- set by the host: determinants of more than 64 spin orbitals (two words,
    // Sec. 3): the high words of d0, valid, cmask, frz_occ and frz_emp, and the irreps
    // of spatial orbitals 32-63 (4 bits each); det_words = 1 or 2 selects the width.
    uint64_t d0_hi, valid_hi;
    uint64_t cmask_hi[NCLASS];
    uint64_t irr_packed_hi[2];
    uint64_t frz_occ_hi, frz_emp_hi;
    int32_t det_words, pad5;
};

// A spawn record (16 B, written and read with one vector access): child determinant,
// signed walkers, and a tag word (bit 0: from an initiator; bits 1-3: k_post's marks).
struct __attribute__((aligned(16))) SpawnRec {
    uint64_t det;
    int32_t w;
    uint32_t tag;
};

constexpr int EXT_BITS = 28;

struct EngineArgs {
    SysDesc *desc;
    int32_t max_sys;
    int32_t wsh;                     // log2 of a spawn tile's attempts
    int32_t post_seg;                // chunks between k_post's looks at its queue of new dets
    unsigned int *work;              // [N_WORK] shares taken of each list (reset per iteration)
    uint32_t *status;                // per system: ST_* bits (kept apart from the read-only
    unsigned long long *spawns;      // descriptors); [SPAWN_SLOTS] spawning events each
    const int32_t *chunk_sys;        // system of each global chunk (-1: unused)
    const int32_t *chunk_local;      // chunk index inside its system's table
    unsigned long long *step;        // iterations run by this handle (its parity selects total)
    IterStat *acc;                   // [max_sys][ACC_SLOTS] the iteration's statistics
    int64_t *c0;                     // [max_sys] population on the reference after the iteration
    unsigned long long *total;       // [N_TOTAL] lengths of the lists of spawn tiles
    const int64_t *nchunks;          // global chunks in use
    IterRecord *rec;                 // [max_sys][REC_CAP]
    int32_t *tiles;                  // [NLIST][list_cap][4] the spawn tiles (see put_tile)
    int64_t list_cap;
    uint32_t *unlisted;              // [BPC chunk_cap] buckets whose tiles did not fit a list
    // Spawn records of the iteration (the per-destination blocks of Sec. 4.1, with the
    // bucket as destination): k_spawn writes a record straight into its child's bucket's
    // slots (SysDesc::rec0, rec_r), at the place the bucket's counter gives it. Writing
    // them unsorted and grouping them afterwards (a counting sort in five launches) cost
    // 115 us of a 3.3 ms iteration and 23 us of a 118 us one.
    SpawnRec *recs;
    uint32_t *bhist;                 // [BPC chunk_cap] records per bucket (k_post clears them)
    uint32_t *bprev;                 // [BPC chunk_cap] the same, the last count above zero
    // [BPC chunk_cap] slots of a bucket beyond its system's rec_r: their first << EXT_BITS |
    // how many (0: none). For lists whose records crowd into few buckets (the reference's
    // neighbours): with as many slots for every bucket as the fullest one needs, a list
    // grown from walkers on the reference asked for 8e9.
    uint64_t *bext;
    uint32_t *rec_max;               // [max_sys] most records of one bucket this iteration
    long long *d0acc;                // [max_sys] walkers spawned onto the reference (kept out of
                                     // the records: the reference is the hot spot of Sec. 4.1)
    // New determinants that did not fit their bucket (completed, then re-bucketed by the host).
    uint64_t *sp_det;
    int32_t *sp_pop, *sp_sys;
    double *sp_hd;
    unsigned long long *sp_count;
    int64_t sp_cap;
    uint32_t *spilled;               // [max_sys] set by k_post when a bucket spilled
    // Every system of the launch draws plain determinants with no point group and no
    // restricted space: the spawning kernel is then launched in its variant that
    // leaves those cases out.
    int32_t plain;
};

// Staging area of the export that allocates nothing (fciqmc_walkers_noalloc): a
// 64-bit counter, then keys, populations and initiator flags of up to
// NOALLOC_MAX_DETS entries (32 MiB + 256 B).
constexpr int64_t NOALLOC_MAX_DETS = (int64_t)1 << 21;
constexpr size_t NOALLOC_KEYS_OFF = 256;
constexpr size_t NOALLOC_VALS_OFF = NOALLOC_KEYS_OFF + 8 * (size_t)NOALLOC_MAX_DETS;
constexpr size_t NOALLOC_FLAGS_OFF = NOALLOC_VALS_OFF + 4 * (size_t)NOALLOC_MAX_DETS;
constexpr size_t NOALLOC_BYTES = NOALLOC_FLAGS_OFF + 4 * (size_t)NOALLOC_MAX_DETS;

// Kernel launchers (kernels.hip, compiled once per determinant width: one word in fq,
// two words in fq::w2). Determinant arrays hold the width's words per entry.
constexpr int NKERN = 5;   // profiled kernel groups: tile listing, (unused), spawn,
                           // annihilation, statistics/shift
// Device sort: longest list (32-bit positions), and the words its digit counts take (a
// total per digit, then one count per digit and run of 1024 entries).
constexpr int64_t SORT_MAX = (int64_t)1 << 31;
constexpr int64_t sort_hist_words(int64_t n) { return 256 * (1 + (n + 1023) / 1024); }

// What the check of a walker list finds. `bad`: the first entry the system cannot hold, as
// its number * 8 + the reason.
enum { LIST_COUNTS = 1, LIST_RANGE = 2, LIST_SPACE = 3, LIST_PAIR = 4 };
struct ListCheck {
    unsigned long long bad = ~0ull;
    unsigned long long nw = 0, nd = 0;   // walkers, entries with walkers
    uint32_t most = 0;                   // largest |population|
    int32_t c0 = 0, have_ref = 0;        // the reference's population, whether it has walkers
    int32_t unsorted = 0;                // not strictly ascending, or an entry without walkers
    int32_t twice = 0;
};

#define FQ_WIDTH_LAUNCHERS                                                                     \
    /* first: the spawn tiles are listed from the tables (the first iteration of a launch,    \
       after any host-side change); later iterations use the list the previous iteration's    \
       k_post wrote. */                                                                       \
    void launch_iteration(const EngineArgs &a, int post_grid, int spawn_grid, bool first,      \
                          hipStream_t s, hipEvent_t *ev /* NKERN + 1 events or nullptr */);     \
    hipError_t launch_load(SysDesc *d_desc, int32_t sys, const uint64_t *det,                 \
                           const int32_t *pop, int64_t n, int add_ref, uint32_t *d_err,        \
                           hipStream_t s);                                                     \
    /* The checks and sums of a list to be loaded, into *out (which begins as the host's     \
       ListCheck{}); na, nb: electrons of either spin. */                                     \
    hipError_t launch_check_list(const SysDesc *desc, int32_t sys, const uint64_t *det,       \
                                 const int32_t *pop, int64_t n, int na, int nb,               \
                                 ListCheck *out, hipStream_t s);                              \
    /* Sets out->twice if a sorted list has walkers twice on one determinant. */              \
    hipError_t launch_twice(const uint64_t *det, const int32_t *pop, int64_t n,               \
                            ListCheck *out, hipStream_t s);                                   \
    /* Move every entry of the buckets (src_*, src_nb buckets, counts src_cnt) and the spill  \
       entries of system sys into the descriptor's (empty) buckets. */                        \
    hipError_t launch_rebucket(SysDesc *d_desc, int32_t sys, const uint64_t *src_key,         \
                               const int32_t *src_pop, const double *src_hd,                  \
                               const int32_t *src_cnt, int64_t src_nb, const uint64_t *sp_det, \
                               const int32_t *sp_pop, const double *sp_hd,                    \
                               const int32_t *sp_sys, int64_t n_sp, uint32_t *d_err,          \
                               hipStream_t s);                                                 \
    /* Adds the occupied entries of nb buckets to *count and writes the first `limit`. */     \
    hipError_t launch_compact(const uint64_t *key, const int32_t *pop, const int32_t *cnt,    \
                              int64_t nb, uint64_t *out_det, int32_t *out_pop,                \
                              unsigned long long *count, int64_t limit, hipStream_t s);       \
    /* Stable sort of n (<= SORT_MAX) entries by the low `passes` bytes of the determinant;   \
       the result is in key2/val2 if passes is odd. hist: sort_hist_words(n) words. */        \
    hipError_t launch_sort(uint64_t *key, int32_t *val, uint64_t *key2, int32_t *val2,        \
                           uint32_t *hist, int64_t n, int passes, hipStream_t s);             \
    /* Initiator flag of each of n entries: |pop| > n_a, or the reference. */                 \
    hipError_t launch_flags(const uint64_t *key, const int32_t *val, int64_t n, int32_t n_a,  \
                            uint64_t d0, uint64_t d0_hi, uint32_t *flags, hipStream_t s);     \
    /* Gives nb buckets of rec_r slots (arrays bprev and bext at the first) their places in \
       the extension [pool0, pool0 + pool) of the record buffer, for `factor` times the       \
       records of the last iteration and 16 more; *used gets what all of them need. */        \
    hipError_t launch_extend(const uint32_t *bprev, uint64_t *bext, int64_t nb, uint32_t rec_r, \
                             float factor, int64_t pool0, int64_t pool,                       \
                             unsigned long long *used, hipStream_t s);                        \
    /* H_DD (or the function's diagonal) of one determinant, words lo and hi. */              \
    hipError_t launch_e0(const SysDesc *desc, int32_t sys, uint64_t lo, uint64_t hi,          \
                         double *out, hipStream_t s);
FQ_WIDTH_LAUNCHERS
namespace w2 {
FQ_WIDTH_LAUNCHERS
}  // namespace w2
// Export into the staging area `stage` (NOALLOC layout): compaction of the occupied
// slots (entries past NOALLOC_MAX_DETS are counted, not written), then a bitonic
// sort by determinant of the first n entries padded to a power of two.
hipError_t launch_stage_compact(const uint64_t *key, const int32_t *pop, const int32_t *cnt,
                                int64_t nb, void *stage, hipStream_t s);
hipError_t launch_stage_sort(void *stage, int64_t n, hipStream_t s);
// Initiator flag of each of the n sorted entries: |pop| > n_a, or the reference.
hipError_t launch_stage_flags(void *stage, int64_t n, int32_t n_a, uint64_t d0, hipStream_t s);
int spawn_grid_size(int W);
int post_grid_size();

}  // namespace fq
