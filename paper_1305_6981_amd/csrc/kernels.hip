// HIP kernels of the FCIQMC iteration (Booth, Smart & Alavi, arXiv:1305.6981)
// for gfx950.
//
// The main list of a system is hash-partitioned into buckets of at most 256
// densely packed entries (determinant, population, stored H_DD): the paper's
// distribution of determinants over processes by a hash (Sec. 4.1), with a
// wavefront in the role of a process. Four consecutive buckets form a chunk,
// one workgroup's unit in annihilation. One iteration of every active system is
// three launches (four in the first iteration of a launch sequence):
//
//   k_tiles       lists the spawn tiles, runs of attempts of one bucket (first iteration
//                 of a launch sequence only; afterwards k_post does)
//   k_spawn       one spawning attempt per walker (Sec. 2, Eq. pspawn): random
//                 excitation with its pgen (Sec. 5), Slater-Condon element,
//                 acceptance; each accepted spawn becomes a record (child,
//                 signed walkers, initiator flag) in the slots of the child's
//                 bucket -- the per-destination blocks of Sec. 4.1
//   k_post        per bucket, by one wavefront: the records merged per child in
//                 an LDS hash (the sort and compress of Sec. 4.1); death/cloning
//                 of every entry (Eq. pdeath); annihilation with the initiator
//                 test for children that are unoccupied after death (Sec. 4.2);
//                 new determinants placed into the holes left by emptied
//                 entries, the bucket re-packed, H_DD of new determinants from a
//                 pair table staged in LDS; estimator partial sums (Eq. ProjE);
//                 the next iteration's spawn tiles
//   k_finalize    per system, one wavefront: the iteration's statistics, which k_post's
//                 workgroups add up in a few shares, the shift update, the record
//
// All floating-point decisions follow the same operation order as the CPU
// oracle and are compiled with -ffp-contract=off.
#include "engine.h"

#include <utility>

#ifndef FQ_DET_WORDS
#define FQ_DET_WORDS 1
#endif

namespace fq {
#if FQ_DET_WORDS == 2
namespace w2 {
#endif

// ---------------------------------------------------------------------------
// Determinants (Sec. 3): bit p set when spin orbital p is occupied, in as many
// 64-bit words as the spin orbitals need. This file is compiled once per width:
// one word (up to 64 spin orbitals, det_t = uint64_t) into namespace fq, two
// words (up to 128, det_t = a 128-bit integer with the operations used here)
// into fq::w2.
// ---------------------------------------------------------------------------
#if FQ_DET_WORDS == 1
typedef uint64_t det_t;
__device__ __forceinline__ uint64_t lo64(det_t x) { return x; }
__device__ __forceinline__ uint64_t hi64(det_t) { return 0ull; }
__device__ __forceinline__ det_t make_det(uint64_t lo, uint64_t) { return lo; }
__device__ __forceinline__ int dpopc(det_t x) { return __popcll(x); }
__device__ __forceinline__ int dctz(det_t x) { return __builtin_ctzll(x); }      // lowest set bit
__device__ __forceinline__ int dhib(det_t x) { return 63 - __builtin_clzll(x); } // highest set bit
#else
struct det_t {
    unsigned __int128 v;
    det_t() = default;
    __device__ constexpr explicit det_t(unsigned long long x) : v(x) {}
    __device__ explicit operator bool() const { return v != 0; }
};
__device__ __forceinline__ det_t det_raw(unsigned __int128 v) {
    det_t r;
    r.v = v;
    return r;
}
__device__ __forceinline__ det_t operator&(det_t a, det_t b) { return det_raw(a.v & b.v); }
__device__ __forceinline__ det_t operator|(det_t a, det_t b) { return det_raw(a.v | b.v); }
__device__ __forceinline__ det_t operator^(det_t a, det_t b) { return det_raw(a.v ^ b.v); }
__device__ __forceinline__ det_t operator~(det_t a) { return det_raw(~a.v); }
__device__ __forceinline__ det_t operator<<(det_t a, int k) { return det_raw(a.v << k); }
__device__ __forceinline__ det_t operator>>(det_t a, int k) { return det_raw(a.v >> k); }
__device__ __forceinline__ det_t operator-(det_t a, unsigned long long b) { return det_raw(a.v - b); }
__device__ __forceinline__ det_t &operator&=(det_t &a, det_t b) { a.v &= b.v; return a; }
__device__ __forceinline__ det_t &operator|=(det_t &a, det_t b) { a.v |= b.v; return a; }
__device__ __forceinline__ det_t &operator^=(det_t &a, det_t b) { a.v ^= b.v; return a; }
__device__ __forceinline__ bool operator==(det_t a, det_t b) { return a.v == b.v; }
__device__ __forceinline__ bool operator!=(det_t a, det_t b) { return a.v != b.v; }
__device__ __forceinline__ bool operator<(det_t a, det_t b) { return a.v < b.v; }
__device__ __forceinline__ uint64_t lo64(det_t x) { return (uint64_t)x.v; }
__device__ __forceinline__ uint64_t hi64(det_t x) { return (uint64_t)(x.v >> 64); }
__device__ __forceinline__ det_t make_det(uint64_t lo, uint64_t hi) {
    return det_raw(((unsigned __int128)hi << 64) | (unsigned __int128)lo);
}
__device__ __forceinline__ int dpopc(det_t x) { return __popcll(lo64(x)) + __popcll(hi64(x)); }
__device__ __forceinline__ int dctz(det_t x) {
    const uint64_t l = lo64(x);
    return l ? __builtin_ctzll(l) : 64 + __builtin_ctzll(hi64(x));
}
__device__ __forceinline__ int dhib(det_t x) {
    const uint64_t h = hi64(x);
    return h ? 127 - __builtin_clzll(h) : 63 - __builtin_clzll(lo64(x));
}
#endif
constexpr int NSO_MAX = 64 * FQ_DET_WORDS;   // spin orbitals a determinant holds
#define DBIT(p) (det_t(1ull) << (p))
__device__ __forceinline__ det_t even_bits() {
    return make_det(0x5555555555555555ull, 0x5555555555555555ull);
}
__device__ __forceinline__ det_t odd_bits() {
    return make_det(0xAAAAAAAAAAAAAAAAull, 0xAAAAAAAAAAAAAAAAull);
}
// The determinant-valued fields of a system's descriptor.
__device__ __forceinline__ det_t ref_of(const SysDesc &d) { return make_det(d.d0, d.d0_hi); }
__device__ __forceinline__ det_t valid_of(const SysDesc &d) { return make_det(d.valid, d.valid_hi); }
__device__ __forceinline__ det_t cmask_of(const SysDesc &d, int c) {
    return make_det(d.cmask[c], d.cmask_hi[c]);
}
__device__ __forceinline__ det_t *keys_of(const SysDesc &d) { return (det_t *)d.key; }

// ---------------------------------------------------------------------------
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11).
// Counter (bits 0-31 of D, bits 32-63 of D, k, ((iter mod 2^24) << 8) | block),
// key = seed XOR (bits 64-127 of D), i.e. the seed up to 64 spin orbitals.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32->64 product per multiplier gives both halves
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c.z;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        // three-input XORs (0x96 is the truth table of a ^ b ^ c)
        c = make_uint4(__builtin_amdgcn_bitop3_b32(hi1, c.y, k0, 0x96), lo1,
                       __builtin_amdgcn_bitop3_b32(hi0, c.w, k1, 0x96), lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ void draw2(uint64_t seed, det_t det, uint32_t k, int64_t iter,
                                      uint32_t block, uint64_t &x0, uint64_t &x1) {
    const uint64_t lo = lo64(det), key = seed ^ hi64(det);
    const uint4 ctr = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), k,
                                 ((uint32_t)((uint64_t)iter & 0xFFFFFFu) << 8) | block);
    const uint4 w = philox10(ctr, (uint32_t)key, (uint32_t)(key >> 32));
    x0 = ((uint64_t)w.y << 32) | (uint64_t)w.x;
    x1 = ((uint64_t)w.w << 32) | (uint64_t)w.z;
}

__device__ __forceinline__ double u01(uint64_t x) {
    return (double)(x >> 11) * (1.0 / 9007199254740992.0);
}

// w / 2^32, exact in double.
__device__ __forceinline__ double u01_32(uint32_t w) {
    return (double)w * (1.0 / 4294967296.0);
}

// floor(w n / 2^32): an index in [0, n).
__device__ __forceinline__ uint32_t pick(uint32_t w, uint32_t n) { return __umulhi(w, n); }

// Position of the k-th (0-based) set bit of byte b (k below its bit count), the entries
// [k][b] of the table sel8 (2 KB, staged in LDS).
__device__ __forceinline__ uint8_t sel8_entry(uint32_t k, uint32_t b) {
    for (uint32_t i = 0; i < k; ++i) b &= b - 1u;
    return (uint8_t)(b ? __builtin_ctz(b) : 0);
}

// j (j - 1) / 2 for j < 2^12 (0 for j = 0): the index of the first pair (i, j).
__device__ __forceinline__ uint32_t pair_base(uint32_t j) {
    return (uint32_t)__umul24(j, j - 1u) >> 1;
}

// Position of the k-th (0-based) set bit of x (k < popcount(x)): halving with
// popcounts down to one byte, then the table. (min(k, k - c) is k - c exactly when
// k >= c.)
__device__ __forceinline__ int select_bit(uint64_t x, uint32_t k, const uint8_t *sel8) {
    uint32_t c = (uint32_t)__popc((uint32_t)x);
    uint32_t w = k >= c ? (uint32_t)(x >> 32) : (uint32_t)x;
    uint32_t pos = k >= c ? 32u : 0u;
    k = k - c < k ? k - c : k;
    c = (uint32_t)__popc(w & 0xFFFFu);
    uint32_t sh = k >= c ? 16u : 0u;
    k = k - c < k ? k - c : k;
    w >>= sh;
    pos += sh;
    c = (uint32_t)__popc(w & 0xFFu);
    sh = k >= c ? 8u : 0u;
    k = k - c < k ? k - c : k;
    w >>= sh;
    return (int)(pos + sh + sel8[(k << 8) | (w & 0xFFu)]);
}
#if FQ_DET_WORDS == 2
__device__ __forceinline__ int select_bit(det_t x, uint32_t k, const uint8_t *sel8) {
    const uint32_t c = (uint32_t)__popcll(lo64(x));
    return k < c ? select_bit(lo64(x), k, sel8) : 64 + select_bit(hi64(x), k - c, sel8);
}
#endif

// 64-bit finaliser of MurmurHash3 (public domain): table placement only.
__device__ __forceinline__ uint64_t mix64(uint64_t h) {
    h ^= h >> 33;
    h *= 0xff51afd7ed558ccdull;
    h ^= h >> 33;
    h *= 0xc4ceb9fe1a85ec53ull;
    h ^= h >> 33;
    return h;
}

// Bucket of a determinant among nb buckets: the high word of mix64(D) * nb, i.e.
// the hash scaled onto [0, nb) (the placement of Sec. 4.1's process hash; the
// paper's Algorithm 1 is kept in the CPU oracle, results do not depend on it).
__device__ __forceinline__ uint32_t bucket_of(det_t D, uint64_t nb) {
#if FQ_DET_WORDS == 1
    return (uint32_t)__umul64hi(mix64(D), nb);
#else
    return (uint32_t)__umul64hi(mix64(lo64(D) ^ mix64(hi64(D) ^ 0x9E3779B97F4A7C15ull)), nb);
#endif
}

// ---------------------------------------------------------------------------
// Hamiltonian (spin orbital p = 2 s + sigma).
// ---------------------------------------------------------------------------
// Packed-pair index; operands stay below 2^24, so 24-bit multiplies are exact.
__device__ __forceinline__ int tri(int i, int j) {
    const int hi = i >= j ? i : j, lo = i >= j ? j : i;
    return (int)(__umul24((unsigned)hi, (unsigned)(hi + 1)) >> 1) + lo;
}

// The integral tables live in global memory; saying so lets the compiler use
// global (not flat) loads, which do not hold up the LDS wait counter.
typedef __attribute__((address_space(1))) const double gdouble;
__device__ __forceinline__ const gdouble *gptr(const double *p) { return (const gdouble *)p; }
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gp(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}
// A load through the constant address space: for a uniform address the compiler
// issues a scalar load (scalar cache, scalar registers). Only for values this kernel
// reads before (or never) writing them.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T *p) {
    return *(const __attribute__((address_space(4))) T *)p;
}

// 16-byte global loads and stores through plain vector types.
typedef int v4i32 __attribute__((ext_vector_type(4)));
typedef unsigned long long v2u64 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int4 gload_i4(const int32_t *p) {
    const v4i32 v = *gp(reinterpret_cast<const v4i32 *>(p));
    return make_int4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ ulonglong2 gload_u2(const uint64_t *p) {
    const v2u64 v = *gp(reinterpret_cast<const v2u64 *>(p));
    return make_ulonglong2(v.x, v.y);
}
__device__ __forceinline__ void gstore_i4(void *p, int x, int y, int z, int w) {
    v4i32 v;
    v.x = x;
    v.y = y;
    v.z = z;
    v.w = w;
    *gp(reinterpret_cast<v4i32 *>(p)) = v;
}

// Main-list keys in global memory (one 16-byte access for two words).
#if FQ_DET_WORDS == 1
__device__ __forceinline__ det_t ldk(const det_t *p) { return *gp(p); }
__device__ __forceinline__ void stk(det_t *p, det_t v) { *gp(p) = v; }
#else
__device__ __forceinline__ det_t ldk(const det_t *p) {
    const ulonglong2 w = gload_u2((const uint64_t *)p);
    return make_det(w.x, w.y);
}
__device__ __forceinline__ void stk(det_t *p, det_t v) {
    v2u64 w;
    w.x = lo64(v);
    w.y = hi64(v);
    *gp(reinterpret_cast<v2u64 *>(p)) = w;
}
#endif

// Spawn records: one 16-byte access each (two for two-word determinants, whose
// records take 32 bytes).
#if FQ_DET_WORDS == 1
typedef SpawnRec rec_t;
__device__ __forceinline__ void put_rec(rec_t *p, det_t D, int32_t w, uint32_t tag) {
    gstore_i4(p, (int)(uint32_t)D, (int)(uint32_t)(D >> 32), w, (int)tag);
}
__device__ __forceinline__ rec_t get_rec(const rec_t *p) {
    const int4 x = gload_i4((const int32_t *)p);
    rec_t r;
    r.det = (uint64_t)(uint32_t)x.x | ((uint64_t)(uint32_t)x.y << 32);
    r.w = x.z;
    r.tag = (uint32_t)x.w;
    return r;
}
#else
struct __attribute__((aligned(16))) rec_t {
    det_t det;
    int32_t w;
    uint32_t tag;
    uint64_t pad;
};
static_assert(sizeof(rec_t) == 32, "two-word spawn records take 32 bytes");
__device__ __forceinline__ void put_rec(rec_t *p, det_t D, int32_t w, uint32_t tag) {
    const uint64_t lo = lo64(D), hi = hi64(D);
    gstore_i4(p, (int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi,
              (int)(uint32_t)(hi >> 32));
    gstore_i4((char *)p + 16, w, (int)tag, 0, 0);
}
__device__ __forceinline__ rec_t get_rec(const rec_t *p) {
    const int4 x = gload_i4((const int32_t *)p);
    const int4 y = gload_i4((const int32_t *)p + 4);
    rec_t r;
    r.det = make_det((uint64_t)(uint32_t)x.x | ((uint64_t)(uint32_t)x.y << 32),
                     (uint64_t)(uint32_t)x.z | ((uint64_t)(uint32_t)x.w << 32));
    r.w = y.x;
    r.tag = (uint32_t)y.y;
    return r;
}
#endif
static_assert(sizeof(rec_t) == 16 * FQ_DET_WORDS, "record size");
__device__ __forceinline__ rec_t *recs_of(const EngineArgs &a) { return (rec_t *)a.recs; }
__device__ __forceinline__ det_t *spill_dets(const EngineArgs &a) { return (det_t *)a.sp_det; }

__device__ __forceinline__ double eri_so(const SysDesc &d, int p, int q, int r, int s) {
    if (((p ^ q) | (r ^ s)) & 1) return 0.0;
    return gptr(d.eri)[tri(tri(p >> 1, q >> 1), tri(r >> 1, s >> 1))];
}

__device__ __forceinline__ double h_so(const SysDesc &d, int p, int q) {
    if ((p ^ q) & 1) return 0.0;
    return gptr(d.h1)[(p >> 1) * d.M + (q >> 1)];
}

// Both words are read at uniform addresses (scalar loads); the lane's label is
// then picked out with ALU operations only.
__device__ __forceinline__ int irrep_of(const SysDesc &d, int s) {
#if FQ_DET_WORDS == 1
    const uint64_t w0 = d.irr_packed[0], w1 = d.irr_packed[1];
#else
    const uint64_t w0 = (s & 32) ? d.irr_packed_hi[0] : d.irr_packed[0];
    const uint64_t w1 = (s & 32) ? d.irr_packed_hi[1] : d.irr_packed[1];
#endif
    return (int)((((s & 16) ? w1 : w0) >> (4 * (s & 15))) & 0xFull);
}

__device__ __forceinline__ int class_of(const SysDesc &d, int p) {
    return 2 * irrep_of(d, p >> 1) + (p & 1);
}

// The orbitals strictly between p and a, and the parity of the occupied ones.
__device__ __forceinline__ det_t between_mask(int p, int a) {
    const int lo = p < a ? p : a, hi = p < a ? a : p;
    return (DBIT(hi) - 1ull) & ~((det_t(2ull) << lo) - 1ull);
}
__device__ __forceinline__ int between_parity(det_t det, int p, int a) {
    return dpopc(det & between_mask(p, a)) & 1;
}

__device__ double hdiag_of(const SysDesc &d, det_t det) {
    double acc = d.e_core;
    for (det_t m = det; m; m &= m - 1ull) {
        const int p = dctz(m);
        acc = acc + h_so(d, p, p);
    }
    for (det_t m1 = det; m1; m1 &= m1 - 1ull) {
        const int p = dctz(m1);
        for (det_t m2 = m1 & (m1 - 1ull); m2; m2 &= m2 - 1ull) {
            const int q = dctz(m2);
            acc = acc + (eri_so(d, p, p, q, q) - eri_so(d, p, q, q, p));
        }
    }
    return acc;
}

// Single excitation p -> a: h_pa + sum over occupied q != p (ascending) of
// (pa|qq) - [same spin](pq|qa), each term read from the precomputed row
// t3[p][a][*]; four loads are issued before they are added, in order.
__device__ double hel_single(const SysDesc &d, det_t det, int p, int a) {
    double acc = h_so(d, p, a);
    const gdouble *row = gptr(d.t3) + ((p * NSO_MAX + a) * NSO_MAX);
    det_t m = det & ~DBIT(p);
    while (m) {
        const int q0 = dctz(m);
        m &= m - 1ull;
        const int q1 = m ? dctz(m) : q0;
        m &= m - 1ull;
        const int q2 = m ? dctz(m) : q0;
        m &= m - 1ull;
        const int q3 = m ? dctz(m) : q0;
        const int n = 1 + (q1 != q0) + (q2 != q0) + (q3 != q0);
        m &= m - 1ull;
        const double v0 = row[q0], v1 = row[q1], v2 = row[q2], v3 = row[q3];
        acc = acc + v0;
        if (n > 1) acc = acc + v1;
        if (n > 2) acc = acc + v2;
        if (n > 3) acc = acc + v3;
    }
    return between_parity(det, p, a) ? -acc : acc;
}

// p < q occupied, a, b empty. Pairing: unlike spins -> a' carries p's spin;
// like spins -> a' = min(a, b). Sign: q -> b' on det, then p -> a'.
__device__ double hel_double(const SysDesc &d, det_t det, int p, int q, int a, int b) {
    int ap, bp;
    if ((p ^ q) & 1) {
        const bool a_with_p = ((a ^ p) & 1) == 0;
        ap = a_with_p ? a : b;
        bp = a_with_p ? b : a;
    } else {
        ap = a < b ? a : b;
        bp = a < b ? b : a;
    }
    // the two parities at once: parity(x) ^ parity(y) = parity(x ^ y)
    const det_t d1 = (det & ~DBIT(q)) | DBIT(bp);
    const int par = dpopc((det & between_mask(q, bp)) ^ (d1 & between_mask(p, ap))) & 1;
    const double v = eri_so(d, p, ap, q, bp) - eri_so(d, p, bp, q, ap);
    return par ? -v : v;
}

// Whether a child lies in the system's restricted space (Sec. 5: outside it the
// excitation is null). Excitation level: electrons outside the reference's
// orbitals; seniority: spatial orbitals holding exactly one electron.
__device__ __forceinline__ bool in_space(const SysDesc &d, det_t det) {
    const int sp = d.space;
    if ((sp & 1) && dpopc(det & ~ref_of(d)) > d.max_ex) return false;
    if ((sp & 2) && dpopc((det ^ (det >> 1)) & even_bits()) > d.max_sen) return false;
    const det_t fo = make_det(d.frz_occ, d.frz_occ_hi), fe = make_det(d.frz_emp, d.frz_emp_hi);
    if ((sp & 4) && ((det & fo) != fo || (det & fe))) return false;
    return true;
}

// <det|H|d0> for det != d0 within two excitations of d0 (d0 is the source).
__device__ double hel_to_ref(const SysDesc &d, det_t det) {
    const det_t d0 = ref_of(d);
    const det_t from = d0 & ~det, to = det & ~d0;
    const int nd = dpopc(from);
    if (nd == 1) return hel_single(d, d0, dctz(from), dctz(to));
    const int p = dctz(from), q = dhib(from);
    const int a = dctz(to), b = dhib(to);
    return hel_double(d, d0, p, q, a, b);
}

// ---------------------------------------------------------------------------
// Excitation generation (Sec. 5). Symmetry classes are (irrep, spin) with
// class id 2*irrep + spin; cmask[c] holds the spin orbitals of class c.
// Returns false for a null excitation.
// ---------------------------------------------------------------------------
struct Excit {
    det_t det;
    double pgen;
    double hel;
    int p, a;
    uint32_t nt;   // single excitation: movable electrons times targets
};


// Symmetry classes seen from the excitation generator. With no point group
// (every orbital in irrep 0, two classes: the spins) everything is bit
// arithmetic; otherwise the class masks are read from an LDS copy, since the
// class index differs between lanes.
template <bool C1>
struct ClassView {
    det_t valid;
    const det_t *cm;      // LDS copy of SysDesc::cmask (unused when C1)
    __device__ __forceinline__ det_t mask(int c) const {
        if (C1) return valid & ((c & 1) ? odd_bits() : even_bits());
        return cm[c];
    }
    __device__ __forceinline__ int irrep(const SysDesc &d, int s) const {
        return C1 ? 0 : irrep_of(d, s);
    }
    __device__ __forceinline__ int cls(const SysDesc &d, int p) const {
        return C1 ? (p & 1) : class_of(d, p);
    }
};

// Single excitation (Sec. 5.1) from the electron word w1 and the hole word w2:
// renormalised over the electrons that have an allowed target. Returns false
// for a null excitation; otherwise the child, pgen and the orbitals p -> a.
template <bool C1>
__device__ __forceinline__ bool excite_single(const SysDesc &d, const ClassView<C1> &cv,
                                              det_t det, uint32_t w1, uint32_t w2,
                                              const uint8_t *sel8, Excit &ex) {
    const det_t emp = ~det & valid_of(d);
    const int n_class = C1 ? 2 : d.n_class;
    det_t movable = det_t(0ull);
    for (int c = 0; c < n_class; ++c) {
        const det_t cm = C1 ? cv.mask(c) : cmask_of(d, c);
        if (emp & cm) movable |= det & cm;
    }
    const uint32_t nmov = (uint32_t)dpopc(movable);
    if (nmov == 0) return false;
    const int p = select_bit(movable, pick(w1, nmov), sel8);
    const det_t tg = emp & cv.mask(cv.cls(d, p));
    const uint32_t nal = (uint32_t)dpopc(tg);
    const int a = select_bit(tg, pick(w2, nal), sel8);
    ex.det = det ^ DBIT(p) ^ DBIT(a);
    ex.pgen = d.p_single / (double)((int64_t)nal * (int64_t)nmov);
    ex.p = p;
    ex.a = a;
    ex.nt = nal * nmov;
    return true;
}

// pgen of a single excitation from orbital p of det that has a target (Sec. 5.1): the
// value excite_single gives, from the electron alone.
template <bool C1>
__device__ __forceinline__ double single_pgen(const SysDesc &d, const ClassView<C1> &cv, det_t det,
                                              int p) {
    const det_t emp = ~det & valid_of(d);
    const int n_class = C1 ? 2 : d.n_class;
    det_t movable = det_t(0ull);
    for (int c = 0; c < n_class; ++c) {
        const det_t cm = C1 ? cv.mask(c) : cmask_of(d, c);
        if (emp & cm) movable |= det & cm;
    }
    const uint32_t nal = (uint32_t)dpopc(emp & cv.mask(cv.cls(d, p)));
    return d.p_single / (double)((int64_t)nal * (int64_t)dpopc(movable));
}

// What the spawning kernel's attempts need of a system, kept in scalar registers while it
// works on the system (read from the descriptor at each attempt, these were a dozen
// dependent scalar loads: most of a short wavefront's time).
struct SpawnSys {
    uint64_t seed;
    det_t valid;
    uint32_t iterw;          // iteration, as in the Philox counter
    uint32_t dbl_thr, npairs;
    uint32_t n0, n1, nl0, nl1, nu;   // empty orbitals per spin; first-hole choices for like
                                     // spins (0, 1) and unlike spins; 0: none
    uint64_t mu;             // orbitals that may be the first hole for unlike spins
    float f0, f1, f2, f3, ft;   // rejection: (float)w0 > bound x f (SysDesc::bound_f)
    float sg_mul, sg_sub;    // a single's acceptance uniform, rounded down
    int32_t has_double, defer, c1, coupled;
};
// Values made uniform explicitly (the compiler then keeps them in scalar registers).
__device__ __forceinline__ uint32_t uni(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
__device__ __forceinline__ uint64_t uni(uint64_t x) {
    return (uint64_t)uni((uint32_t)x) | ((uint64_t)uni((uint32_t)(x >> 32)) << 32);
}
__device__ __forceinline__ float uni(float x) { return __uint_as_float(uni(__float_as_uint(x))); }
__device__ __forceinline__ SpawnSys spawn_sys(const SysDesc &d) {
    SpawnSys h;
    h.seed = uni(d.seed);
    h.valid = make_det(uni(d.valid), uni(d.valid_hi));
    h.iterw = uni(((uint32_t)((uint64_t)d.iter & 0xFFFFFFu)) << 8);
    h.dbl_thr = uni(d.dbl_thr);
    h.npairs = uni((uint32_t)(d.N * (d.N - 1) / 2));
    h.n0 = uni((uint32_t)d.n_emp[0]);
    h.n1 = uni((uint32_t)d.n_emp[1]);
    // (one electron: the type word still picks a double, which has no choice: null)
    h.nl0 = d.N >= 2 && h.n0 >= 2u ? h.n0 : 0u;
    h.nl1 = d.N >= 2 && h.n1 >= 2u ? h.n1 : 0u;
    h.nu = d.N >= 2 ? (h.n1 > 0u ? h.n0 : 0u) + (h.n0 > 0u ? h.n1 : 0u) : 0u;
    h.mu = (h.n1 > 0u ? 0x5555555555555555ull : 0ull) | (h.n0 > 0u ? 0xAAAAAAAAAAAAAAAAull : 0ull);
    h.f0 = uni(d.bound_f[0]);
    h.f1 = uni(d.bound_f[1]);
    h.f2 = uni(d.bound_f[2]);
    h.f3 = uni(d.bound_f[3]);
    h.ft = uni(d.bound_ft);
    h.sg_mul = uni(d.sg_mul);
    h.sg_sub = uni(d.sg_sub);
    h.has_double = (int32_t)uni((uint32_t)d.has_double);
    h.defer = (int32_t)uni((uint32_t)d.defer);
    h.c1 = (int32_t)uni(d.n_class == 2 ? 1u : 0u);
    h.coupled = (int32_t)uni((uint32_t)d.hphf);
    return h;
}
// c ? a : b of values (a conditional between two members would select an address and keep
// the whole struct in memory).
template <typename T>
__device__ __forceinline__ T pick_if(bool c, T a, T b) {
    return c ? a : b;
}
// The four words of one Philox block of a spawning attempt: word 0 picks the
// type and, rescaled within the chosen type's interval, is the acceptance
// uniform; words 1-3 pick the orbitals.
__device__ __forceinline__ uint4 spawn_words(const SpawnSys &h, det_t det, uint32_t k) {
    const uint64_t lo = lo64(det), key = h.seed ^ hi64(det);
    return philox10(make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), k, h.iterw), (uint32_t)key,
                    (uint32_t)(key >> 32));
}

// The orbitals of a double excitation (Sec. 5.2) from the words of one Philox block: the
// electrons p < q from w.y, the holes a and b, in the order drawn, from w.z and w.w.
// Returns false for a null excitation (p, q, a and b are orbital numbers all the same, below
// NSO_MAX: the bounds are looked up for every lane that picked a double). pgen: with no point
// group one of the four per-system values, given as its index pc; else computed here.
// recip[k] = 1.0 / k, filled by IEEE division (same bits as dividing in place).
struct DoubleDraw {
    int p, q, a, b, pc;
    double pgen;
};
// A unique pair of electrons by inverse triangular indexing.
__device__ __forceinline__ void draw_pair(uint32_t npairs, det_t det, uint32_t w, const uint8_t *sel8,
                                          DoubleDraw &x) {
    const uint32_t K = pick(w, npairs);   // < 2016
    // The estimate from the hardware square root is within one of j (the largest
    // j with j (j - 1) / 2 <= K); one exact integer correction each way.
    // (float)(8 K + 1), exact below 2^23, by the mantissa trick
    const float xf = __int_as_float((int)(0x4B000000u | (8u * K + 1u))) - 8388608.0f;
    uint32_t j = (uint32_t)((1.0f + __builtin_amdgcn_sqrtf(xf)) * 0.5f);
    j -= pair_base(j) > K ? 1u : 0u;
    j += pair_base(j + 1) <= K ? 1u : 0u;
    x.p = select_bit(det, K - pair_base(j), sel8);
    x.q = select_bit(det, j, sel8);
}
// No point group: every determinant has the same number of empty orbitals of each spin, so
// the allowed sets and their sizes follow from the spins alone, and pgen is one of four
// per-system values (the general draw below gives the same sets, counts and pgen). Like
// spins: both holes from the empty orbitals of that spin, the second by its rank without
// the first. Unlike spins: the first from all empty orbitals that leave the other spin a
// choice. Free of branches (a null excitation selects from an empty set, harmlessly).
__device__ __forceinline__ bool draw_double_c1(const SpawnSys &h, det_t det, uint4 w,
                                               const uint8_t *sel8, DoubleDraw &x) {
    const det_t emp = ~det & h.valid;
    draw_pair(h.npairs, det, w.y, sel8, x);
    const bool same = ((x.p ^ x.q) & 1) == 0, sp = (x.p & 1) != 0;
    const uint64_t ev = 0x5555555555555555ull, od = 0xAAAAAAAAAAAAAAAAull;
    const uint64_t ms = sp ? od : ev, ma = pick_if(same, ms, h.mu);
    const uint32_t nal = pick_if(same, pick_if(sp, h.nl1, h.nl0), h.nu);
    const uint32_t ka = pick(w.z, nal);
    x.a = select_bit(emp & make_det(ma, ma), ka, sel8);
    const bool sa = (x.a & 1) != 0;
    const uint64_t mb = same ? ms : sa ? ev : od;
    const uint32_t nb = pick_if(same, nal ? nal - 1u : 0u, pick_if(sa, h.n0, h.n1));
    uint32_t kb = pick(w.w, nb);
    kb += same && kb >= ka ? 1u : 0u;
    x.b = select_bit(emp & make_det(mb, mb), kb, sel8);
    x.pc = same ? (int)sp : 2 + (int)sa;
    return nal != 0u;
}
__device__ __forceinline__ bool draw_double(const SysDesc &d, const ClassView<false> &cv, det_t det,
                                            uint4 w, const double *recip, const uint8_t *sel8,
                                            DoubleDraw &x) {
    const det_t emp = ~det & valid_of(d);
    const int N = d.N, n_class = d.n_class;
    draw_pair((uint32_t)(N * (N - 1) / 2), det, w.y, sel8, x);
    const int p = x.p;
    const bool same = ((p ^ x.q) & 1) == 0;
    const det_t A = same ? (emp & ((p & 1) ? odd_bits() : even_bits())) : emp;
    const int gpq = cv.irrep(d, p >> 1) ^ cv.irrep(d, x.q >> 1);
    // a orbitals whose partner class (Eq. sym1 plus spin) has an empty orbital besides a: an
    // irrep's two spins together, without a branch on the lanes (which kept the LDS reads of
    // the partners' masks one behind the other). Like spins take the partner of their own
    // spin (the other spin's class has no orbital in A).
    det_t allowed = det_t(0ull);
    const int self = same && gpq == 0 ? 1 : 0;   // a is in its own partner class
#pragma unroll 2
    for (int g = 0; 2 * g < n_class; ++g) {
        const det_t even = cv.mask(2 * (gpq ^ g)), odd = cv.mask(2 * (gpq ^ g) + 1);
        const int ne = dpopc(emp & even), no = dpopc(emp & odd);
        if ((same ? ne : no) > self) allowed |= A & cmask_of(d, 2 * g);
        if ((same ? no : ne) > self) allowed |= A & cmask_of(d, 2 * g + 1);
    }
    const uint32_t nal = (uint32_t)dpopc(allowed);
    if (nal == 0 || N < 2) {
        // null: any orbitals will do, but the caller looks their bounds up (p and q are set)
        x.a = x.b = x.pc = 0;
        x.pgen = 0.0;
        return false;
    }
    const int a = select_bit(allowed, pick(w.z, nal), sel8);
    const int ca = cv.cls(d, a);
    const int pca = 2 * (gpq ^ (ca >> 1)) + (same ? (p & 1) : 1 - (ca & 1));
    const det_t bset = emp & cv.mask(pca) & ~DBIT(a);
    const uint32_t nba = (uint32_t)dpopc(bset);
    const int b = select_bit(bset, pick(w.w, nba), sel8);
    const int cb = cv.cls(d, b);
    const int pcb = 2 * (gpq ^ (cb >> 1)) + (same ? (p & 1) : 1 - (cb & 1));
    const int nbb = dpopc(emp & cv.mask(pcb)) - (pcb == cb ? 1 : 0);
    x.a = a;
    x.b = b;
    x.pc = 0;
    x.pgen = (2.0 * d.p_double * (recip[nba] + recip[nbb])) /
             (double)((int64_t)N * (int64_t)(N - 1) * (int64_t)nal);
    return true;
}

// ---------------------------------------------------------------------------
// Spin-coupled functions (Sec. 5.3, Eqs. EqualCoeffs and SpinCoup). With spin
// orbitals interleaved, exchanging alpha and beta in every spatial orbital maps
// |D> to (-1)^{n2(D)} |D~> (n2: doubly occupied orbitals); the function of the
// pair {D, D~} is (|D> + lam (-1)^{n2(D)} |D~>)/sqrt2, lam = (-1)^S (-1)^{N/2}
// (SysDesc::lam), or |D> for a closed pair D = D~ (even S only). A function is
// stored as min(D, D~); excitations are drawn from that determinant only.
// ---------------------------------------------------------------------------
__device__ __forceinline__ det_t spin_flip(det_t D) {
    return ((D & even_bits()) << 1) | ((D >> 1) & even_bits());
}
__device__ __forceinline__ det_t fn_rep(det_t D) {
    const det_t f = spin_flip(D);
    return f < D ? f : D;
}
__device__ __forceinline__ int pair_sign(const SysDesc &d, det_t D) {
    return (dpopc(D & (D >> 1) & even_bits()) & 1) ? -d.lam : d.lam;
}

// <bra|H|ket> for a single or double excitation with ket the source (0 beyond).
__device__ double hel_between(const SysDesc &d, det_t bra, det_t ket) {
    const det_t from = ket & ~bra, to = bra & ~ket;
    const int n = dpopc(from);
    if (n == 1) return hel_single(d, ket, dctz(from), dctz(to));
    if (n == 2) return hel_double(d, ket, dctz(from), dhib(from), dctz(to), dhib(to));
    return 0.0;
}

// <Phi_j|H|Phi_i> for the stored functions Dj != Di, Di the source: both open,
// <Dj|H|Di> + lam (-1)^{n2(Dj)} <Dj~|H|Di>; one closed, sqrt2 <Dj|H|Di>; both
// closed, <Dj|H|Di>.
__device__ double fn_hel(const SysDesc &d, det_t Di, det_t Dj) {
    const det_t fi = spin_flip(Di), fj = spin_flip(Dj);
    const double h = hel_between(d, Dj, Di);
    if (fi != Di && fj != Dj) return h + (double)pair_sign(d, Dj) * hel_between(d, fj, Di);
    if (fi != Di || fj != Dj) return 1.4142135623730951 * h;
    return h;
}

// Diagonal element of a stored function from its determinant's diagonal hd.
__device__ __forceinline__ double fn_diag_from(const SysDesc &d, det_t D, double hd) {
    if (!d.hphf) return hd;
    const det_t f = spin_flip(D);
    if (f == D) return hd;
    return hd + (double)pair_sign(d, D) * hel_between(d, f, D);
}
__device__ double fn_diag(const SysDesc &d, det_t D) { return fn_diag_from(d, D, hdiag_of(d, D)); }

// The same, with nothing to add for determinants (PLAIN: EngineArgs::plain).
template <bool PLAIN>
__device__ __forceinline__ double diag_from(const SysDesc &d, det_t D, double hd) {
    return PLAIN ? hd : fn_diag_from(d, D, hd);
}

// Projected-energy element <Phi_0|H|Phi_D> (Eq. ProjE) and whether it can be
// nonzero (D within a double excitation of the reference, or its partner).
// (PLAIN: determinants, EngineArgs::plain.)
template <bool PLAIN>
__device__ __forceinline__ bool near_ref(const SysDesc &d, det_t D) {
    return dpopc(D ^ ref_of(d)) <= 4 || (!PLAIN && d.hphf && dpopc(spin_flip(D) ^ ref_of(d)) <= 4);
}
template <bool PLAIN>
__device__ __forceinline__ double ref_hel(const SysDesc &d, det_t D) {
    return !PLAIN && d.hphf ? fn_hel(d, ref_of(d), D) : hel_to_ref(d, D);
}

// The probability that excite() draws T from det (Secs. 5.1, 5.2) by the same
// operations as the draw, 0 when it cannot draw T. recip[k] = 1/k.
__device__ double pgen_target(const SysDesc &d, const det_t *cm, const double *recip,
                              det_t det, det_t T) {
    const det_t from = det & ~T, to = T & ~det;
    const int nf = dpopc(from);
    if (nf != dpopc(to)) return 0.0;
    const det_t emp = ~det & valid_of(d);
    const bool c1 = d.n_class == 2;
    auto mask = [&](int c) -> det_t {
        return c1 ? (valid_of(d) & ((c & 1) ? odd_bits() : even_bits())) : cm[c];
    };
    auto cls = [&](int p) -> int { return c1 ? (p & 1) : class_of(d, p); };
    if (nf == 1) {
        const int p = dctz(from), a = dctz(to);
        if (cls(a) != cls(p)) return 0.0;
        det_t movable = det_t(0ull);
        for (int c = 0; c < (c1 ? 2 : d.n_class); ++c) {
            const det_t m = mask(c);
            if (emp & m) movable |= det & m;
        }
        const uint32_t nmov = (uint32_t)dpopc(movable);
        const uint32_t nal = (uint32_t)dpopc(emp & mask(cls(p)));
        return d.p_single / (double)((int64_t)nal * (int64_t)nmov);
    }
    if (nf != 2) return 0.0;
    const int p = dctz(from), q = dhib(from);
    const int a = dctz(to), b = dhib(to);
    const bool same = ((p ^ q) & 1) == 0;
    if (same ? (((a ^ p) & 1) || ((b ^ p) & 1)) : (((a ^ b) & 1) == 0)) return 0.0;
    if (c1) return same ? d.pgen_c1[p & 1] : d.pgen_c1[2 + (a & 1)];
    const int gpq = irrep_of(d, p >> 1) ^ irrep_of(d, q >> 1);
    const int ca = class_of(d, a), cb = class_of(d, b);
    const int pca = 2 * (gpq ^ (ca >> 1)) + (same ? (p & 1) : 1 - (ca & 1));
    if (cb != pca) return 0.0;
    const det_t A = same ? (emp & ((p & 1) ? odd_bits() : even_bits())) : emp;
    det_t allowed = det_t(0ull);
    for (int c = 0; c < d.n_class; ++c) {
        const det_t memb = A & cm[c];
        if (!memb) continue;
        const int sb = same ? (p & 1) : 1 - (c & 1);
        const int pc = 2 * (gpq ^ (c >> 1)) + sb;
        const int nb = dpopc(emp & cm[pc]) - (pc == c ? 1 : 0);
        if (nb > 0) allowed |= memb;
    }
    const uint32_t nal = (uint32_t)dpopc(allowed);
    const int pcb = 2 * (gpq ^ (cb >> 1)) + (same ? (p & 1) : 1 - (cb & 1));
    const uint32_t nba = (uint32_t)dpopc(emp & cm[pca] & ~DBIT(a));
    const int nbb = dpopc(emp & cm[pcb]) - (pcb == cb ? 1 : 0);
    return (2.0 * d.p_double * (recip[nba] + recip[nbb])) /
           (double)((int64_t)d.N * (int64_t)(d.N - 1) * (int64_t)nal);
}

// A drawn excitation as a spawn between stored functions: the target is the
// function holding the child, reached through the child or its partner (their
// probabilities add); the pair of the source itself is diagonal (null), and so is a
// closed pair in an odd-spin run. Returns false for a null excitation.
__device__ bool to_function(const SysDesc &d, const det_t *cm, const double *recip,
                            det_t D, Excit &ex) {
    const det_t Dj = fn_rep(ex.det), fx = spin_flip(ex.det);
    if (Dj == D || (d.hphf < 0 && spin_flip(Dj) == Dj)) return false;
    if (fx != ex.det) ex.pgen = ex.pgen + pgen_target(d, cm, recip, D, fx);
    ex.hel = fn_hel(d, D, Dj);
    ex.det = Dj;
    return true;
}

// Natural log for the shift update: x = m 2^e with m in (1/sqrt2, sqrt2],
// ln x = e ln2 + 2 atanh((m-1)/(m+1)), the atanh series summed by Horner's
// rule through the z^25 term. Fixed operation order (no contraction), so any
// IEEE-double implementation of the same method returns the same bits.
__device__ double shift_log(double x) {
    const uint64_t bits = (uint64_t)__double_as_longlong(x);
    int e = (int)((bits >> 52) & 0x7FFull) - 1023;
    double m = __longlong_as_double((long long)((bits & 0x000FFFFFFFFFFFFFull) |
                                                0x3FF0000000000000ull));
    if (m > 1.4142135623730951) {
        m = m * 0.5;
        e = e + 1;
    }
    const double z = (m - 1.0) / (m + 1.0);
    const double z2 = z * z;
    double sum = 1.0 / 27.0;
    for (int k = 25; k >= 1; k -= 2) sum = sum * z2 + 1.0 / (double)k;
    return (double)e * 0.6931471805599453 + 2.0 * z * sum;
}

__device__ __forceinline__ bool participating(const SysDesc &d, uint32_t status) {
    return d.active && status == 0 && d.iter < d.stop_at;
}

// Sum over the 64 lanes of a wavefront with a fixed butterfly (deterministic).
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    for (int o = 32; o > 0; o >>= 1) v = v + __shfl_xor(v, o, 64);
    return v;
}

// Orders the LDS accesses of a wavefront's lanes around it (LDS operations of one
// wavefront complete in issue order, so no wait is needed, only no code motion).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive prefix sum over the 64 lanes of a wavefront by data-parallel primitives
// (DPP): shifts within rows of 16 lanes, then row broadcasts (no LDS traffic).
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_move(unsigned long long v) {
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
    return (unsigned long long)(uint32_t)lo | ((unsigned long long)(uint32_t)hi << 32);
}
__device__ __forceinline__ unsigned long long wave_incl_scan(unsigned long long x) {
    const int lane = threadIdx.x & 63, r = lane & 15;
    unsigned long long y = dpp_move<0x111>(x);   // row_shr:1
    if (r >= 1) x += y;
    y = dpp_move<0x112>(x);                      // row_shr:2
    if (r >= 2) x += y;
    y = dpp_move<0x114>(x);                      // row_shr:4
    if (r >= 4) x += y;
    y = dpp_move<0x118>(x);                      // row_shr:8
    if (r >= 8) x += y;
    y = dpp_move<0x142>(x);                      // row_bcast:15 (last lane of the row below)
    if (lane & 16) x += y;
    y = dpp_move<0x143>(x);                      // row_bcast:31 (lane 31, to the upper half)
    if (lane >= 32) x += y;
    return x;
}

// The same for 32-bit sums and maxima (one instruction a step: lanes without a source
// take the 0 given as the old value).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_incl_sum32(uint32_t x) {
    x += dpp_or_0<0x111, 0xF>(x);
    x += dpp_or_0<0x112, 0xF>(x);
    x += dpp_or_0<0x114, 0xF>(x);
    x += dpp_or_0<0x118, 0xF>(x);
    x += dpp_or_0<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
    x += dpp_or_0<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_incl_max32(uint32_t x) {
    auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    x = mx(x, dpp_or_0<0x111, 0xF>(x));
    x = mx(x, dpp_or_0<0x112, 0xF>(x));
    x = mx(x, dpp_or_0<0x114, 0xF>(x));
    x = mx(x, dpp_or_0<0x118, 0xF>(x));
    x = mx(x, dpp_or_0<0x142, 0xA>(x));
    x = mx(x, dpp_or_0<0x143, 0xC>(x));
    return x;
}

// ---------------------------------------------------------------------------
// Handing out work. One counter for the whole chip serves about 100 grabs per
// microsecond, which 6144 wavefronts exceed (a kernel of 100 us spent most of it in 28000
// grabs of one tile); so work is kept in NLIST lists with a counter each, on lines of
// their own. A taker begins with a share of its home list fixed by its number (no atomic),
// goes on by its home list's counter and then takes from lists that still hold work,
// found by reading all the counters at once. With one share per taker or less there is no
// atomic at all.
// ---------------------------------------------------------------------------
struct Handout {
    unsigned int *work;          // the lists' counters (CTR_STRIDE apart)
    const unsigned int *len;     // the lists' lengths, in LDS
    unsigned int takers;         // per workgroup
    unsigned int share;
    int list;                    // list being taken from
    bool begin;
};
// Items of list l that are handed out by number: one share to every taker of the
// workgroups congruent to l.
__device__ __forceinline__ unsigned int handout_fixed(const Handout &h, unsigned int l) {
    const unsigned int g = gridDim.x;
    return l < g ? h.takers * ((g - l + NLIST - 1) / NLIST) * h.share : 0u;
}
// The next share: items [at, at + count) of list h.list. rank: this taker's number among
// those at home in its list. Returns false when every list is empty. Whole wavefront;
// uniform results.
__device__ __forceinline__ bool handout_next(Handout &h, unsigned int rank, unsigned int &at,
                                             unsigned int &count) {
    const unsigned int lane = threadIdx.x & 63u;
    unsigned int n = (unsigned int)__builtin_amdgcn_readfirstlane((int)h.len[h.list]);
    if (h.begin) {
        h.begin = false;
        at = rank * h.share;
        if (at < n) {
            count = n - at < h.share ? n - at : h.share;
            return true;
        }
    }
    for (;;) {
        const unsigned int f = handout_fixed(h, (unsigned int)h.list);
        if (f < n) {
            unsigned int g = 0;
            if (lane == 0) g = atomicAdd(&h.work[h.list * CTR_STRIDE], h.share);
            at = f + (unsigned int)__builtin_amdgcn_readfirstlane((int)g);
            if (at < n) {
                count = n - at < h.share ? n - at : h.share;
                return true;
            }
        }
        // another list that still holds work, the nearest after this one
        const unsigned int nl = h.len[lane & (NLIST - 1)], fl = handout_fixed(h, lane & (NLIST - 1));
        const bool open = lane < NLIST && fl < nl;
        if (!__ballot(open)) return false;
        unsigned int w = 0xFFFFFFFFu;
        if (open) w = __hip_atomic_load(&h.work[lane * CTR_STRIDE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t m = __ballot(open && w < nl - fl);
        if (!m) return false;
        const uint64_t after = m & ~((2ull << h.list) - 1ull);
        h.list = __builtin_ctzll(after ? after : m);
        n = (unsigned int)__builtin_amdgcn_readfirstlane((int)h.len[h.list]);
    }
}

// ---------------------------------------------------------------------------
// Spawn tiles. A tile is a run of at most 2^wsh consecutive attempts (walkers) of one
// bucket, the unit of work of a wavefront in k_spawn; the tiles of all buckets form NLIST
// lists in no particular order (results do not depend on it), written by k_post as it
// finishes its windows, or by k_tiles before the first iteration of a launch. A tile
// holds its system, the bucket in the system, its number among the bucket's tiles, and
// its attempts | the bucket's entries << 20 | whether the bucket holds 2^30 walkers or more.
// ---------------------------------------------------------------------------
constexpr int TILE_ENT_SHIFT = 20;
constexpr uint32_t TILE_BIG = 1u << 31;

__device__ __forceinline__ void put_tile(const EngineArgs &a, int list, unsigned long long at, int s,
                                         uint32_t lb, uint32_t j, unsigned long long x, int n) {
    const unsigned long long done = (unsigned long long)j << a.wsh, wt = 1ull << a.wsh;
    const unsigned long long left = x > done ? x - done : 0ull;
    const uint32_t n_t = (uint32_t)(left < wt ? left : wt);
    gstore_i4(a.tiles + 4 * ((int64_t)list * a.list_cap + (int64_t)at), s, (int)lb, (int)j,
              (int)(n_t | ((uint32_t)n << TILE_ENT_SHIFT) | (x >> 30 ? TILE_BIG : 0u)));
}

// A bucket whose tiles do not fit their list: k_spawn takes it whole from a list of its
// own (any of its tiles' places that were reserved get empty tiles).
__device__ __forceinline__ void put_unlisted(const EngineArgs &a, int h, int64_t gb) {
    const unsigned long long u = atomicAdd(&a.total[CTR_UNLISTED(h)], 1ull);
    a.unlisted[u] = (uint32_t)gb;
}

// Append the tiles of one bucket per lane (x walkers, n entries; x = 0: none; call with
// the whole wavefront) to the lists of half h: one reservation in the given list for all
// buckets of at most 64 tiles (callers deal their groups of buckets out to the lists in
// turn, so that all lists hold much the same of every system); a bucket with more (the reference's can have thousands)
// is spread over several lists, in runs of at least 64 (in a batch a list of short runs
// of many systems makes every wavefront change system at nearly every tile).
__device__ __forceinline__ void emit_tiles(const EngineArgs &a, int h, int list, int64_t gb, int s,
                                           uint32_t lb, unsigned long long x, int n) {
    const int lane = threadIdx.x & 63;
    const unsigned long long cap = (unsigned long long)a.list_cap;
    const unsigned long long nt = (x + (1ull << a.wsh) - 1ull) >> a.wsh;
    const bool few = nt <= 64ull;
    const unsigned long long mine = few ? nt : 0ull, incl = wave_incl_scan(mine);
    unsigned long long base = 0;
    if (lane == 63 && incl) base = atomicAdd(&a.total[CTR_TILES(h, list)], incl);
    base = __shfl(base, 63, 64);
    const unsigned long long at = base + incl - mine;
    const bool fits = mine == 0ull || at + mine <= cap;   // (empty buckets and idle lanes fit)
    for (unsigned long long k = 0; k < mine && at + k < cap; ++k)
        put_tile(a, list, at + k, s, lb, (uint32_t)k, fits ? x : 0ull, n);
    if (!fits) put_unlisted(a, h, gb);
    for (uint64_t big = __ballot(!few); big; big &= big - 1) {
        const int l = __builtin_ctzll(big);
        const unsigned long long nl = __shfl(nt, l, 64), xl = __shfl(x, l, 64);
        const int sl = __shfl(s, l, 64), ml = __shfl(n, l, 64);
        const uint32_t bl = (uint32_t)__shfl((int)lb, l, 64);
        // over as many lists as give each 64 tiles, from the given one on: lane i fills the
        // part of list i, tiles i, i + lists, ...
        const int lists = nl < 64ull * NLIST ? (int)((nl + 63ull) / 64ull) : NLIST;
        const int to = (list + lane) & (NLIST - 1);
        const bool fill = lane < lists;
        const unsigned long long part = fill ? (nl + (unsigned)(lists - 1 - lane)) / (unsigned)lists : 0ull;
        const unsigned long long b = fill ? atomicAdd(&a.total[CTR_TILES(h, to)], part) : 0ull;
        const bool all = !__ballot(fill && b + part > cap);
        for (unsigned long long k = 0; k < part && b + k < cap; ++k)
            put_tile(a, to, b + k, sl, bl, (uint32_t)(k * (unsigned)lists + (unsigned)lane), all ? xl : 0ull, ml);
        if (!all && lane == l) put_unlisted(a, h, gb);
    }
}

// The tile lists of an iteration: half step & 1, the next one's in the other; those of a
// launch's first iteration in 2.
__device__ __forceinline__ int cur_half(const EngineArgs &a) { return (int)(*a.step & 1ull); }

// Sum of |C| over a bucket's n entries by a wavefront.
__device__ __forceinline__ unsigned long long abs_sum4(int4 v) {
    return (unsigned long long)(abs(v.x)) + (unsigned long long)(abs(v.y)) +
           (unsigned long long)(abs(v.z)) + (unsigned long long)(abs(v.w));
}
__device__ __forceinline__ unsigned long long bucket_walkers(const SysDesc &d, int64_t lb, int n) {
    const int e = 4 * (threadIdx.x & 63);
    int4 q = make_int4(0, 0, 0, 0);
    if (e < n) {
        q = gload_i4(d.pop + lb * BQ + e);
        if (e + 1 >= n) q.y = 0;
        if (e + 2 >= n) q.z = 0;
        if (e + 3 >= n) q.w = 0;
    }
    return wave_sum(abs_sum4(q));
}

// ---------------------------------------------------------------------------
// K1: the tiles of the current list (the first iteration of a launch). A wavefront takes
// up to 64 consecutive buckets, fewer in a small list; four buckets' loads are in flight
// at a time. Bound by memory: 4 B per entry, 0.15 ms for 8e7 entries, 7 us for a small list.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tiles(EngineArgs a, const SysDesc *__restrict__ desc) {
    const int lane = threadIdx.x & 63;
    const int64_t nbk = *a.nchunks * BPC, waves = (int64_t)gridDim.x * 4;
    const int64_t share = (nbk + waves - 1) / waves;
    const int per = (int)(share < 64 ? (share + 3) / 4 * 4 : 64);
    for (int64_t b0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per; b0 < nbk; b0 += waves * per) {
        unsigned long long x = 0;
        int sx = 0, nx = 0;
        uint32_t lx = 0;
        for (int k = 0; k < per && b0 + k < nbk; k += BPC) {   // one chunk: BPC buckets of a system
            const int sy = __builtin_amdgcn_readfirstlane(a.chunk_sys[(b0 + k) / BPC]);
            if (sy < 0) continue;
            const SysDesc &d = desc[sy];
            if (!participating(d, a.status[sy])) continue;
            const int64_t lb = (int64_t)a.chunk_local[(b0 + k) / BPC] * BPC;
            int n[BPC];
            int4 q[BPC];
#pragma unroll
            for (int u = 0; u < BPC; ++u) {
                n[u] = d.bcnt[lb + u];
                q[u] = gload_i4(d.pop + (lb + u) * BQ + 4 * lane);   // (past the entries: masked)
            }
#pragma unroll
            for (int u = 0; u < BPC; ++u) {
                const int e = 4 * lane;
                if (e >= n[u]) q[u].x = 0;
                if (e + 1 >= n[u]) q[u].y = 0;
                if (e + 2 >= n[u]) q[u].z = 0;
                if (e + 3 >= n[u]) q[u].w = 0;
                const unsigned long long w = wave_sum(abs_sum4(q[u]));
                if (lane == k + u) {
                    x = w;
                    sx = sy;
                    nx = n[u];
                    lx = (uint32_t)(lb + u);
                }
            }
        }
        emit_tiles(a, 2, (int)((b0 / per) & (NLIST - 1)), b0 + lane, sx, lx, x, nx);
    }
}

// ---------------------------------------------------------------------------
// K3: spawning. Every wavefront works on its own, with no workgroup barrier: it takes a
// tile (consecutive attempts of one bucket), stages the bucket's entries in LDS with the
// first attempt of each, and runs through the attempts 64 at a time. An attempt's entry is
// found by a maximum over the lanes below it of the entries that begin there. Attempts
// that are left over (fewer than 64) wait in registers for the next tile's, so that every
// step but a wavefront's last one is full.
//
// An attempt draws its excitation and is then tested against an upper bound of its
// acceptance probability, from a table of bounds on the matrix elements; only attempts
// that pass are queued (per wavefront, in LDS) and evaluated 64 at a time: matrix
// element, pgen, acceptance. A rejected attempt would have been rejected by the full
// test too (the bound holds for every rounding), so the walkers are the same; what is
// saved is the element's two gathers and the division for most attempts, and wavefronts
// that run them for a few lanes only. Single excitations are queued apart.
//
// Bound, in large launches, by vector-instruction issue (420 wavefront instructions per 64
// attempts, a Philox block and the choice of four orbitals most of them); in small ones by
// the chain of memory round trips from the lists to the records (some 17 us for one tile).
// Against a workgroup per tile of a 1024-entry chunk, which searched each attempt's entry
// and evaluated every element: 1.90 -> 1.50 ms (24 electrons, 1.4e8 walkers), 148 -> 85 us
// (3.5e6), 78 -> 36 us (ring of 14 sites, 8e5), 35 -> 20 us (ring of 8 sites, 1.8e4).
// ---------------------------------------------------------------------------

// A spawn record into its child's bucket's slots, at the place the bucket's counter
// gives it (past the slots that every bucket of the system has, in the bucket's extension,
// if it has one). A record past those is dropped (still counted) and the system
// marked: the iteration is then abandoned and re-run with more slots per bucket.
// Walkers spawned onto the reference go to a per-system sum instead (every
// iteration sends it many: the reference is the hot spot of Sec. 4.1).
__device__ __forceinline__ void put_record(const EngineArgs &a, const SysDesc &d, det_t D,
                                           int32_t v, bool init, uint32_t *status) {
    const uint32_t b = bucket_of(D, (uint64_t)d.nbuckets);
    const uint32_t k = __hip_atomic_fetch_add(&a.bhist[d.gchunk0 * BPC + b], 1u, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
    int64_t at = d.rec0 + (int64_t)b * d.rec_r + k;
    if (k >= (uint32_t)d.rec_r) {
        const uint64_t x = a.bext[d.gchunk0 * BPC + b];
        const uint32_t over = k - (uint32_t)d.rec_r;
        if (over >= (uint32_t)(x & ((1ull << EXT_BITS) - 1ull))) {
            atomicOr(status, ST_TABLE_FULL);
            return;
        }
        at = (int64_t)(x >> EXT_BITS) + over;
    }
    put_rec(recs_of(a) + at, D, v, init ? 1u : 0u);
}

// The acceptance uniform: the type word's uniform rescaled within the chosen
// type's interval [0, P_double) or [P_double, 1); given the type it is uniform
// on [0, 1) and independent of the orbital words.
__device__ __forceinline__ double accept_uniform(const SysDesc &d, uint32_t w0) {
    const double u = u01_32(w0);
    return u < d.p_double ? u * d.inv_p_double : (u - d.p_double) * d.inv_p_single;
}

// Walkers spawned (signed; 0: none) from a walker of a determinant with negative (neg) or
// positive population.
__device__ __forceinline__ int32_t accept(const SysDesc &d, double hel, double pgen, double ua,
                                          bool neg, uint32_t *status) {
    const double pr = (d.tau * fabs(hel)) / pgen;
    const double fl = floor(pr);
    if (fl > 1073741824.0) {
        atomicOr(status, ST_SPAWN_OVERFLOW);
        return 0;
    }
    const int32_t m = (int32_t)fl + (ua < pr - fl ? 1 : 0);
    return (!neg == (hel > 0.0)) ? -m : m;
}

constexpr int SPAWN_WAVES = 4;    // wavefronts of a k_spawn workgroup
// Queue items of a wavefront: double excitations from the bottom, singles from the top;
// at most 63 and SGL_DRAIN - 1 before a step adds up to 64.
constexpr int SGL_DRAIN = FQ_DET_WORDS == 1 ? 48 : 32;   // (two words: four workgroups in LDS)
constexpr int SPAWN_QUEUE = SGL_DRAIN + 128;
static_assert(63 + SGL_DRAIN - 1 + 64 <= SPAWN_QUEUE, "a step's attempts fit the queue");
constexpr uint32_t ENT_NEG = 1u << 31, ENT_INIT = 1u << 30, ENT_FIRST = 1u << 29;
constexpr uint32_t ENT_REL = (1u << 22) - 1u;
constexpr int TILE_MAX = 1 << TILE_MAX_SH(FQ_DET_WORDS);
constexpr int ORB_BITS = 7;       // orbital numbers in a queue item
constexpr uint32_t ORB_MASK = (1u << ORB_BITS) - 1u;

// Bound tables in LDS for one-word determinants (with two words they would take a
// workgroup per CU).
constexpr int BOUND_N = 32 * FQ_DET_WORDS;
constexpr int BOUND_LDS = FQ_DET_WORDS == 1 ? BOUND_N * BOUND_N : 2;

template <bool PLAIN>
struct SpawnWave {
    det_t key[BQ];                   // staged entries: determinant,
    uint32_t ent[BQ];                // its first attempt in the tile | sign | initiator | it
                                     // began before the tile (k0 attempts earlier)
    alignas(8) uint8_t head[TILE_MAX];   // entry that begins at an attempt (0: none, or entry 0)
    det_t qd[SPAWN_QUEUE];           // queued attempts: determinant,
    uint2 qm[SPAWN_QUEUE];           // type word (deferred single: ordinal), orbitals | flags
    det_t cm[PLAIN ? 1 : NCLASS];    // class masks of the system
    uint32_t k0;
};

__device__ __forceinline__ float half_to_float(uint16_t h) {
    _Float16 x;
    __builtin_memcpy(&x, &h, 2);
    return (float)x;
}
// x0 y0 + x1 y1 of half-precision numbers, in single precision (no subnormals among them).
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float half_dot2(uint16_t x0, uint16_t x1, uint16_t y0, uint16_t y1) {
    const uint32_t x = (uint32_t)x0 | ((uint32_t)x1 << 16), y = (uint32_t)y0 | ((uint32_t)y1 << 16);
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, x), __builtin_bit_cast(half2_t, y), 0.0f, false);
}

// One queued attempt of system s (item i of a wavefront's queue; kind 0: double, 1: single):
// matrix element, pgen, acceptance, record. Returns whether it spawned.
template <bool PLAIN, int KIND>
__device__ __forceinline__ bool evaluate(const EngineArgs &a, const SysDesc *__restrict__ desc, int s,
                                     const SpawnSys &hs, const uint8_t *s_sel8,
                                     const double *s_recip, const det_t *cm,
                                     const SpawnWave<PLAIN> &Q, int i) {
    const SysDesc &d = desc[s];
    uint32_t *const status = &a.status[s];
    const bool defer = hs.defer != 0, c1 = PLAIN || hs.c1 != 0, coupled = !PLAIN && hs.coupled != 0;
    const ClassView<true> cv1{hs.valid, nullptr};
    const ClassView<false> cvg{hs.valid, cm};
    const det_t D = Q.qd[i];
    const uint2 it = Q.qm[i];
    const bool neg = (it.y >> 28) & 1u;
    uint32_t w0 = it.x;
    Excit ex;
    bool ok = true;
    if (KIND == 0) {
        const int p = (int)(it.y & ORB_MASK), q = (int)((it.y >> ORB_BITS) & ORB_MASK);
        const int ia = (int)((it.y >> (2 * ORB_BITS)) & ORB_MASK);
        const int ib = (int)((it.y >> (3 * ORB_BITS)) & ORB_MASK);
        ex.det = D ^ DBIT(p) ^ DBIT(q) ^ DBIT(ia) ^ DBIT(ib);
        if (c1)
            ex.pgen = ((p ^ q) & 1) == 0 ? (p & 1 ? d.pgen_c1[1] : d.pgen_c1[0])
                                         : (ia & 1 ? d.pgen_c1[3] : d.pgen_c1[2]);
        else
            ex.pgen = pgen_target(d, cm, s_recip, D, ex.det);
        if (!coupled) ex.hel = hel_double(d, D, p, q, ia, ib);
    } else {
        if (defer) {
            // (the ordinal was queued: the same words again)
            const uint4 w = spawn_words(hs, D, it.x);
            w0 = w.x;
            ok = c1 ? excite_single(d, cv1, D, w.y, w.z, s_sel8, ex)
                    : excite_single(d, cvg, D, w.y, w.z, s_sel8, ex);
        } else {
            ex.p = (int)(it.y & ORB_MASK);
            ex.a = (int)((it.y >> ORB_BITS) & ORB_MASK);
            ex.det = D ^ DBIT(ex.p) ^ DBIT(ex.a);
            ex.pgen = c1 ? single_pgen(d, cv1, D, ex.p) : single_pgen(d, cvg, D, ex.p);
        }
        if (ok && !coupled) ex.hel = hel_single(d, D, ex.p, ex.a);
    }
    if (!PLAIN && ok && d.space && !in_space(d, ex.det)) ok = false;
    if (!PLAIN && ok && coupled) ok = to_function(d, cm, s_recip, D, ex);
    if (!ok || ex.hel == 0.0) return false;
    const int32_t v = accept(d, ex.hel, ex.pgen, accept_uniform(d, w0), neg, status);
    if (v == 0) return false;
    if (ex.det == ref_of(d))
        __hip_atomic_fetch_add(&a.d0acc[s], (long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        put_record(a, d, ex.det, v, ((it.y >> 29) & 1u) != 0u, status);
    return true;
}

// One-word determinants: at most 96 VGPRs, five wavefronts per SIMD (the LDS allows five
// workgroups per CU); four with two words.
// PLAIN: every system of the launch has no point group, no restricted space and plain
// determinants (EngineArgs::plain), so those branches are compiled out.
#define SPAWN_WPE(PLAIN) (FQ_DET_WORDS == 1 ? 5 : 4)
template <bool PLAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SPAWN_WPE(PLAIN), SPAWN_WPE(PLAIN))))
void k_spawn(EngineArgs a, const SysDesc *__restrict__ desc, int first) {
    __shared__ SpawnWave<PLAIN> L[SPAWN_WAVES];
    __shared__ uint8_t s_sel8[8 * 256];
    __shared__ double s_recip[PLAIN ? 1 : 65];
    __shared__ uint16_t s_bound[BOUND_LDS];
    __shared__ unsigned long long s_spawned;   // spawning events of system s_tsys,
    __shared__ int s_done;                     // wavefronts that have added theirs
    __shared__ unsigned int s_len[NLIST];      // listed tiles per list
    __shared__ int s_nd[SPAWN_WAVES], s_ns[SPAWN_WAVES];   // items left queued at the end
    // (everything but the lanes' own attempts is uniform, and has to be seen to be: the
    // descriptor's fields are then scalar loads)
    const int t = threadIdx.x, lane = t & 63, wid = __builtin_amdgcn_readfirstlane(t >> 6);
    SpawnWave<PLAIN> &W = L[wid];
    const int half = cur_half(a), h = first ? 2 : half;
    if (blockIdx.x == 0 && t < NLIST) {   // k_post's counters of this iteration
        a.work[CTR_POST(t)] = 0u;
        a.total[CTR_TILES(half ^ 1, t)] = 0ull;
        if (t == 0) a.total[CTR_UNLISTED(half ^ 1)] = 0ull;
    }
    // the lane's list's length, and over all lists
    unsigned int n_list = 0;
    if (lane < NLIST) {
        const unsigned long long n = a.total[CTR_TILES(h, lane)];
        n_list = (unsigned int)(n < (unsigned long long)a.list_cap ? n : (unsigned long long)a.list_cap);
    }
    const unsigned int n_tiles =
        (unsigned int)__builtin_amdgcn_readlane((int)wave_incl_sum32(n_list), 63);
    if (t < NLIST) s_len[t] = n_list;
    if (!PLAIN && t > 0 && t <= 64) s_recip[t] = 1.0 / (double)t;
    for (uint32_t k = 0; k < 8; ++k) s_sel8[(k << 8) | t] = sel8_entry(k, (uint32_t)t);
    if (t == 0) {
        if (!PLAIN) s_recip[0] = 0.0;
        s_spawned = 0ull;
        s_done = 0;
    }
    // Tiles per share: a wavefront's whole part in one when it is small (neighbouring tiles
    // are mostly of one system, and a change of system empties the queues), an eighth of it
    // when it is large (so that the faster wavefronts take more).
    const unsigned int n_waves = SPAWN_WAVES * gridDim.x;
    const unsigned int per_wave = (n_tiles + n_waves - 1u) / n_waves;
    Handout ho{a.work + CTR_SPAWN(0), s_len, SPAWN_WAVES,
               per_wave < 4u ? (per_wave > 0u ? per_wave : 1u)
                             : per_wave < 32u ? 4u : per_wave < 128u ? per_wave / 8u : 16u,
               (int)(blockIdx.x & (NLIST - 1)), true};
    // The system of the workgroup's first tile: its bound table serves from LDS (a tile of
    // another system reads its own from memory), and what is left queued of it at the end
    // is evaluated together.
    const int home = (int)(blockIdx.x & (NLIST - 1));
    const unsigned int first_tile = (blockIdx.x / NLIST) * SPAWN_WAVES * ho.share;
    const uint64_t any = __ballot(n_list > 0u);
    const bool own = first_tile < (unsigned int)__builtin_amdgcn_readlane((int)n_list, home);
    const int tlist = own ? home : any ? __builtin_ctzll(any) : -1;
    const int tsys = tlist >= 0 ? __builtin_amdgcn_readfirstlane(ld_uniform(
                                      a.tiles + 4 * ((int64_t)tlist * a.list_cap + (own ? first_tile : 0u))))
                                : -1;
    if (FQ_DET_WORDS == 1 && tsys >= 0)
        for (int i = t; i < BOUND_LDS / 2; i += 256)
            ((uint32_t *)s_bound)[i] = *gp((const uint32_t *)desc[tsys].bound + i);
    __syncthreads();

    const unsigned int rank = (blockIdx.x / NLIST) * SPAWN_WAVES + (unsigned int)wid;
    unsigned int g_at = 0, g_n = 0;    // the rest of the share at hand
    // Buckets whose tiles are not listed (a list was too small), from a counter of their own.
    int mode = 0;                      // 0: listed tiles, 1: unlisted buckets, 2: none left
    uint32_t f_lb = 0, f_j = 0, f_n = 0;
    int f_sys = 0, f_ne = 0;
    unsigned long long f_x = 0;

    // The tile at hand (uniform): system, bucket, number in the bucket, attempts, entries.
    int ts = -1, t_ne = 0;
    uint32_t t_lb = 0, t_j = 0;
    int t_n = 0;
    bool t_big = false;
    bool have = false, run = false, end = false;   // fetched, staged, nothing left to fetch
    int cur = -1;                      // system of the queued work and tallies
    int nd = 0, ns = 0;                // queued doubles and singles
    uint32_t spawned = 0;              // this lane's spawning events of system cur
    SpawnSys hs{};
    bool stopped = false;
    int xs = 0;                        // attempt of the tile that lane 0 takes next
    uint32_t sl0 = 0, k0 = 0;          // last entry of the step before; W.k0
    int np = 0;                        // attempts waiting in lanes 0 .. np - 1:
    det_t pD = det_t(0ull);            // determinant, ordinal, flags
    uint32_t pk = 0, pf = 0;

    for (;;) {
        if (!have && !run && !end) {
            // the next tile
            if (mode == 0) {
                if (g_n == 0u && !handout_next(ho, rank, g_at, g_n)) {
                    mode = a.total[CTR_UNLISTED(h)] > 0ull ? 1 : 2;
                } else {
                    const v4i32 e = ld_uniform((const v4i32 *)(
                        a.tiles + 4 * ((int64_t)ho.list * a.list_cap + (int64_t)g_at)));
                    ts = __builtin_amdgcn_readfirstlane(e.x);
                    t_lb = (uint32_t)__builtin_amdgcn_readfirstlane(e.y);
                    t_j = (uint32_t)__builtin_amdgcn_readfirstlane(e.z);
                    const uint32_t nn = (uint32_t)__builtin_amdgcn_readfirstlane(e.w);
                    t_n = (int)(nn & ((1u << TILE_ENT_SHIFT) - 1u));
                    t_ne = (int)((nn & ~TILE_BIG) >> TILE_ENT_SHIFT);
                    t_big = (nn & TILE_BIG) != 0u;
                    ++g_at;
                    --g_n;
                    have = true;
                }
            }
            if (mode == 1) {
                if (f_j >= f_n) {
                    unsigned int g = 0;
                    if (lane == 0) g = atomicAdd(&a.work[CTR_FALLBACK], 1u);
                    g = (unsigned int)__builtin_amdgcn_readfirstlane((int)g);
                    if ((unsigned long long)g >= a.total[CTR_UNLISTED(h)]) {
                        mode = 2;
                    } else {
                        const uint32_t gb = a.unlisted[g];
                        f_sys = __builtin_amdgcn_readfirstlane(a.chunk_sys[gb / BPC]);
                        f_lb = (uint32_t)a.chunk_local[gb / BPC] * BPC + gb % BPC;
                        f_ne = desc[f_sys].bcnt[f_lb];
                        f_x = bucket_walkers(desc[f_sys], f_lb, f_ne);
                        f_n = (uint32_t)((f_x + (1ull << a.wsh) - 1ull) >> a.wsh);
                        f_j = 0u;
                    }
                }
                if (mode == 1 && f_j < f_n) {
                    const unsigned long long rest = f_x - ((unsigned long long)f_j << a.wsh);
                    ts = __builtin_amdgcn_readfirstlane(f_sys);
                    t_lb = (uint32_t)__builtin_amdgcn_readfirstlane((int)f_lb);
                    t_j = (uint32_t)__builtin_amdgcn_readfirstlane((int)f_j);
                    t_n = __builtin_amdgcn_readfirstlane(
                        (int)(rest < (1ull << a.wsh) ? (uint32_t)rest : 1u << a.wsh));
                    t_ne = __builtin_amdgcn_readfirstlane(f_ne);
                    t_big = true;
                    ++f_j;
                    have = true;
                }
            }
            if (mode == 2) end = true;
        }
        // waiting and queued work belongs to the current system: finished before another
        // one's tile
        // (at the end, what is left of the table's system is evaluated by the workgroup)
        const bool flush = !run && (end || (have && ts != cur));
        const bool rest = end && cur == tsys;
        if (flush && np == 0 && (rest || (nd == 0 && ns == 0))) {
            if (rest) break;
            if (cur >= 0) {
                const unsigned long long w = wave_sum((unsigned long long)spawned);
                spawned = 0;
                if (lane == 0 && w) {
                    if (cur == tsys)
                        atomicAdd(&s_spawned, w);
                    else
                        atomicAdd(&a.spawns[cur * SPAWN_SLOTS + (blockIdx.x & (SPAWN_SLOTS - 1))], w);
                }
            }
            if (end) break;
            cur = ts;
            hs = spawn_sys(desc[uni((uint32_t)cur)]);
            // no attempts for a system that has stopped (paused after a spill). A plain load:
            // reading past the caches, once per tile, was one address for the whole chip
            // (60 to 100 us of an iteration of eight systems).
            stopped = uni(a.status[uni((uint32_t)cur)]) != 0u;
            if (!PLAIN && lane < NCLASS) W.cm[lane] = cmask_of(desc[cur], lane);
        }
        const int s = __builtin_amdgcn_readfirstlane(cur >= 0 ? cur : 0);
        const SysDesc &d = desc[s];
        if (have && ts == cur) {
            // Stage the bucket's entries (entry u 64 + lane; packed, so no compaction).
            have = false;
            run = true;
            if (stopped) t_n = 0;
            const int64_t base = (int64_t)t_lb * BQ + lane;
            const int R = (t_ne + 63) >> 6;
            int32_t pv[4] = {0, 0, 0, 0};
            det_t kv[4] = {det_t(0ull), det_t(0ull), det_t(0ull), det_t(0ull)};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u >= R) break;
                if ((u << 6) + lane < t_ne) {
                    pv[u] = *gp(d.pop + base + (u << 6));
                    kv[u] = ldk(keys_of(d) + base + (u << 6));
                }
            }
            static_assert(TILE_MAX <= 64 * 8, "one 8-byte store per lane clears the heads");
            if (8 * lane < TILE_MAX) ((uint64_t *)W.head)[lane] = 0ull;
            wave_sync();
            // the first attempt of each entry, relative to the tile's first (in 32 bits when
            // the bucket's walkers fit, which the tile says)
            const unsigned long long off = (unsigned long long)t_j << a.wsh;
            unsigned long long before = 0;
            bool k0_here = false;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u >= R) break;
                const uint32_t ab = (uint32_t)(pv[u] < 0 ? -pv[u] : pv[u]);
                int32_t st, en;
                if (!t_big) {
                    const uint32_t incl = wave_incl_sum32(ab);
                    en = (int32_t)((uint32_t)before - (uint32_t)off + incl);
                    st = en - (int32_t)ab;
                    before += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                } else {
                    const unsigned long long incl = wave_incl_scan((unsigned long long)ab);
                    const long long e64 = (long long)(before + incl) - (long long)off;
                    const long long s64 = e64 - (long long)ab;
                    const long long lim = 1ll << 30;
                    en = (int32_t)(e64 > lim ? lim : e64 < -lim ? -lim : e64);
                    st = (int32_t)(s64 > lim ? lim : s64 < -2 * lim ? -2 * lim : s64);
                    before += __shfl(incl, 63, 64);
                }
                const int e = (u << 6) + lane;
                if (e < t_ne) {
                    const bool init = (int64_t)ab > d.n_a || kv[u] == ref_of(d);
                    W.key[e] = kv[u];
                    W.ent[e] = (st < 0 ? ENT_FIRST : (uint32_t)st & ENT_REL) | (pv[u] < 0 ? ENT_NEG : 0u) |
                               (init ? ENT_INIT : 0u);
                    if (ab != 0u && en > 0 && st < t_n) W.head[st < 0 ? 0 : st] = (uint8_t)e;
                    if (st <= 0 && en > 0) {
                        W.k0 = (uint32_t)(-st);
                        k0_here = true;
                    }
                }
            }
            wave_sync();
            k0 = __ballot(k0_here) ? (uint32_t)__builtin_amdgcn_readfirstlane((int)W.k0) : 0u;
            xs = -np;
            sl0 = 0u;
        }
        const bool defer = hs.defer != 0;   // singles are rare: queued by ordinal, drawn again later
        const bool c1 = PLAIN || hs.c1 != 0;
        const bool coupled = !PLAIN && hs.coupled != 0;
        const ClassView<true> cv1{hs.valid, nullptr};
        const ClassView<false> cvg{hs.valid, W.cm};
        // 64 attempts when that many are at hand, or the waiting ones of a system that ends
        const int n_at = run ? t_n : 0;
        const bool go = run ? n_at - xs >= 64 : flush && np > 0;
        if (go || run) {
            const int x = run ? xs + lane : lane - np;
            const bool act = x < n_at;
            bool qdbl = false, qsgl = false;
            uint32_t meta = 0u, word = 0u;
            det_t D = pD;
            uint32_t k = pk, ent = pf;
            if (run) {
                // the entries of the attempts of this tile (x >= 0)
                const bool in = act && x >= 0;
                uint32_t hd = in ? (uint32_t)W.head[x] : 0u;
                hd = wave_incl_max32(hd);
                hd = hd > sl0 ? hd : sl0;
                sl0 = (uint32_t)__builtin_amdgcn_readlane((int)hd, 63);
                if (in) {
                    ent = W.ent[hd];
                    D = W.key[hd];
                    k = (uint32_t)x - (ent & ENT_REL) + (ent & ENT_FIRST ? k0 : 0u);
                }
            }
            if (!go) {
                // fewer than 64 are left: they wait
                pD = D;
                pk = k;
                pf = ent;
                np = n_at - xs;
                run = false;
                continue;
            }
            if (run) xs += 64;
            np = 0;
            if (act) {
                const uint4 w = spawn_words(hs, D, k);
                word = w.x;
                meta = (ent & ENT_NEG ? 1u << 28 : 0u) | (ent & ENT_INIT ? 1u << 29 : 0u);
                if (hs.has_double && w.x <= hs.dbl_thr) {
                    DoubleDraw x;
                    const bool ok = c1 ? draw_double_c1(hs, D, w, s_sel8, x)
                                       : draw_double(d, cvg, D, w, s_recip, s_sel8, x);
                    qdbl = ok;
                    if (defer) {
                        // |H| <= s_pa' s_qb' (+ s_pb' s_qa' for like spins), a' of p's spin
                        const bool sw = ((x.a ^ x.p) & 1) != 0, same = ((x.p ^ x.q) & 1) == 0;
                        const int ap = (sw ? x.b : x.a) >> 1, bp = (sw ? x.a : x.b) >> 1;
                        const int rp = (x.p >> 1) * BOUND_N, rq = (x.q >> 1) * BOUND_N;
                        uint16_t t0, t1, t2, t3;
                        if (FQ_DET_WORDS == 1 && cur == tsys) {
                            t0 = s_bound[rp + ap];
                            t1 = s_bound[rp + bp];
                            t2 = s_bound[rq + bp];
                            t3 = s_bound[rq + ap];
                        } else {
                            t0 = *gp(d.bound + rp + ap);
                            t1 = *gp(d.bound + rp + bp);
                            t2 = *gp(d.bound + rq + bp);
                            t3 = *gp(d.bound + rq + ap);
                        }
                        float b = half_dot2(t0, same ? t1 : (uint16_t)0, t2, t3);
                        if (coupled) {
                            // the partner's element counts too where it is within reach;
                            // otherwise sqrt2 covers a closed pair
                            const det_t T = D ^ DBIT(x.p) ^ DBIT(x.q) ^ DBIT(x.a) ^ DBIT(x.b);
                            b = dpopc(spin_flip(T) ^ D) <= 4 ? INFINITY : b * 1.41422f;
                        }
                        const float u = (float)w.x;
                        if (c1) {
                            const bool odd = (x.pc & 1) != 0;
                            const float f = pick_if((x.pc & 2) != 0, pick_if(odd, hs.f3, hs.f2),
                                                    pick_if(odd, hs.f1, hs.f0));
                            qdbl = ok && !(u > b * f);
                        } else {
                            qdbl = ok && !(u * (float)x.pgen > b * hs.ft);
                        }
                    }
                    meta |= (uint32_t)x.p | ((uint32_t)x.q << ORB_BITS) |
                            ((uint32_t)x.a << (2 * ORB_BITS)) | ((uint32_t)x.b << (3 * ORB_BITS));
                } else if (defer) {
                    qsgl = true;
                    word = k;
                } else {
                    Excit ex;
                    const bool ok = c1 ? excite_single(d, cv1, D, w.y, w.z, s_sel8, ex)
                                       : excite_single(d, cvg, D, w.y, w.z, s_sel8, ex);
                    if (ok) {
                        const int i = (ex.p >> 1) * BOUND_N + (ex.a >> 1);
                        float b = half_to_float(FQ_DET_WORDS == 1 && cur == tsys ? s_bound[i]
                                                                                 : *gp(d.bound + i));
                        if (coupled) b = dpopc(spin_flip(ex.det) ^ D) <= 4 ? INFINITY : b * 1.41422f;
                        qsgl = !((float)w.x * hs.sg_mul - hs.sg_sub > b * (hs.ft * (float)ex.nt));
                        meta |= (uint32_t)ex.p | ((uint32_t)ex.a << ORB_BITS);
                    }
                }
            }
            const uint64_t md = __ballot(qdbl), ms = __ballot(qsgl);
            const uint64_t below = (1ull << lane) - 1ull;
            if (qdbl) {
                const int i = nd + __popcll(md & below);
                W.qd[i] = D;
                W.qm[i] = make_uint2(word, meta);
            }
            if (qsgl) {
                const int i = SPAWN_QUEUE - 1 - ns - __popcll(ms & below);
                W.qd[i] = D;
                W.qm[i] = make_uint2(word, meta);
            }
            nd += __popcll(md);
            ns += __popcll(ms);
            wave_sync();
        }
        // Evaluate what is queued: 64 at a time, all of it before another system's tile.
        if (nd >= (flush && !rest && nd > 0 ? 1 : 64)) {
            const int n = nd < 64 ? nd : 64;
            nd -= n;
            if (lane < n) spawned += evaluate<PLAIN, 0>(a, desc, s, hs, s_sel8, s_recip, W.cm, W, nd + lane);
        }
        if (ns >= (flush && !rest && ns > 0 ? 1 : SGL_DRAIN)) {
            const int n = ns < 64 ? ns : 64;
            ns -= n;
            if (lane < n)
                spawned += evaluate<PLAIN, 1>(a, desc, s, hs, s_sel8, s_recip, W.cm, W, SPAWN_QUEUE - 1 - ns - lane);
        }
    }
    // What the wavefronts left queued of the table's system, shared out evenly: a launch of
    // few attempts per wavefront would evaluate mostly nearly empty batches.
    if (lane == 0) {
        s_nd[wid] = cur == tsys ? nd : 0;
        s_ns[wid] = cur == tsys ? ns : 0;
    }
    if (!PLAIN && tsys >= 0 && lane < NCLASS) W.cm[lane] = cmask_of(desc[tsys], lane);
    if (tsys >= 0) hs = spawn_sys(desc[uni((uint32_t)tsys)]);
    __syncthreads();
    if (tsys >= 0) {
        const int i0 = 64 * wid + lane;
        int i = i0, v = 0;
        while (v < SPAWN_WAVES - 1 && i >= s_nd[v]) i -= s_nd[v++];
        if (i < s_nd[v]) spawned += evaluate<PLAIN, 0>(a, desc, tsys, hs, s_sel8, s_recip, W.cm, L[v], i);
        i = i0;
        v = 0;
        while (v < SPAWN_WAVES - 1 && i >= s_ns[v]) i -= s_ns[v++];
        if (i < s_ns[v])
            spawned += evaluate<PLAIN, 1>(a, desc, tsys, hs, s_sel8, s_recip, W.cm, L[v], SPAWN_QUEUE - 1 - i);
    }
    {
        const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum32(spawned), 63);
        if (lane == 0 && w) atomicAdd(&s_spawned, (unsigned long long)w);
    }
    // the workgroup's spawning events of its table's system, by the last wavefront done
    if (lane == 0) {
        if (atomicAdd(&s_done, 1) == SPAWN_WAVES - 1) {
            const unsigned long long w = atomicAdd(&s_spawned, 0ull);
            if (w) atomicAdd(&a.spawns[tsys * SPAWN_SLOTS + (blockIdx.x & (SPAWN_SLOTS - 1))], w);
        }
    }
}

// ---------------------------------------------------------------------------
// K4: annihilation. A workgroup takes windows of consecutive chunks from lists of
// them and, in each chunk, every wavefront one bucket, with no workgroup barrier
// inside a bucket:
//   - the bucket's records are merged per child in the wavefront's LDS hash
//     (the sort and compress of Sec. 4.1, by hashing);
//   - every entry dies first (Eq. pdeath); then the walkers that arrived for it
//     are added if it is still occupied, and otherwise survive only if an
//     initiator sent some of them (Sec. 4.2);
//   - children outside the bucket with an initiator parent become new entries
//     (emptied positions first); the other children are discarded;
//   - the bucket is re-packed; the estimator partials are added up, and the next
//     iteration's tiles listed from the buckets' sums of |C|.
// A bucket with more than NREC records merges them in rounds of at most NREC distinct
// children, staging each merged child outside the bucket in the slot of the record that
// entered it into the hash.
//
// Bound by instruction issue and, per bucket, by a chain of loads, LDS and stores (8 us for
// a bucket alone) that four wavefronts per SIMD do not cover; small launches by the chain
// around the buckets as well (lists, metadata, tiles, diagonal elements: some 20 us). With
// the records in their buckets' slots, the queue of new determinants kept over windows,
// statistics in shares and the tiles listed here: 242 -> 100 us at 3.5e6 walkers (24
// electrons), 104 -> 80 us at 1.1e7 (10 electrons), 90 -> 52 us on a ring of 14 sites (8e5),
// 27 -> 20 us on one of 8 (1.8e4), and at 1.4e8 walkers 1.26 -> 1.19 ms with the sort of
// its records (0.13 ms) and a pass over statistics (0.03 ms) gone besides.
// ---------------------------------------------------------------------------
constexpr int NREC = 64;                // distinct children per round in a wavefront's hash
constexpr int WHASH = 128;              // hash slots per wavefront (load <= 0.5)
constexpr int POST_QUEUE = 1024;        // new determinants whose H_DD is still to be computed
constexpr int POST_FLUSH = 256;         // queued new determinants that are computed at once
constexpr int POST_MAX_SYS = 256;       // systems whose status k_post snapshots in LDS
constexpr int POST_WIN = 32;            // chunks per window of bucket metadata in LDS
// the window's POST_WIN BPC record counts are loaded by one thread each
static_assert(POST_WIN * BPC <= 256, "one k_post thread per record count of a window");
constexpr uint32_t F_INIT = 1u;         // from an initiator parent (records and hash slots)
constexpr uint32_t F_MATCHED = 2u;      // hash slot: the child is an entry of the bucket
constexpr uint32_t F_MAYBE = 2u;        // record: found the hash full in this round,
constexpr uint32_t F_DEFER = 4u;        // record: left for a later round
constexpr uint32_t F_STAGED = 8u;       // record: holds a merged child outside the bucket
constexpr int OWN_SHIFT = 2;            // hash slot: the record that entered the child
constexpr int DIAG_SPILL = BQ;          // (see place() in k_post)
constexpr int DIAG_SHIFT = 4;           // staged record: place()'s answer + 1

// Home slot: a multiplicative hash of the folded words (the determinants of one
// bucket agree in the bits of mix64 that chose the bucket, not in these).
static_assert(WHASH == 128, "wh_home takes the top 7 bits of the product");
__device__ __forceinline__ uint32_t wh_home(det_t D) {
    const uint64_t f = lo64(D) ^ hi64(D);
    return (((uint32_t)f ^ (uint32_t)(f >> 32)) * 0x9E3779B1u) >> 25;
}

// A wavefront's working set in k_post: its merge hash (children, walkers arrived,
// flags) and the positions emptied in its bucket. One-word children mark an empty
// slot by 0 and are claimed by a 64-bit compare-and-swap; two-word children have no
// such atomic, so a 32-bit owner word (0: empty, else the claiming lane + 1) is
// claimed and the owner then writes the child.
struct WaveLds {
    det_t key[WHASH];          // child (one word: 0 when empty)
    long long acc[WHASH];      // walkers arrived for it
    uint32_t flg[WHASH];       // F_INIT | F_MATCHED, slow path: record << OWN_SHIFT
#if FQ_DET_WORDS == 2
    uint32_t own[WHASH];       // 0: empty; else the lane that entered the child, + 1
#endif
    uint16_t free_[BQ];        // positions emptied this iteration, ascending
};

#if FQ_DET_WORDS == 1
// Slot of D in a wavefront's hash (-1: absent). Call when no lane inserts.
__device__ __forceinline__ int wh_find(uint64_t D, const uint64_t *hk) {
    uint32_t h = wh_home(D);
    for (int k = 0; k < WHASH; ++k) {
        const uint64_t x = hk[h];
        if (x == D) return (int)h;
        if (x == 0ull) return -1;
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
    return -1;
}

// Slot of D, claimed when absent. Lanes that race for an empty slot with the same D
// agree on it; with different D the losers probe on. For at most WHASH - 1
// distinct children (no limit needed). *own: this lane entered D (one lane per D).
__device__ __forceinline__ int wh_claim(uint64_t D, uint64_t *hk, bool *own) {
    uint32_t h = wh_home(D);
    *own = false;
    for (;;) {
        const uint64_t x = hk[h];
        if (x == D) return (int)h;
        if (x == 0ull) {
            const unsigned long long old =
                atomicCAS((unsigned long long *)&hk[h], 0ull, (unsigned long long)D);
            *own = old == 0ull;
            if (old == 0ull || old == D) return (int)h;
        }
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
}

// As wh_claim, with at most NREC claims per round: *ncl counts claims made and
// claims in flight. -1 when D is absent and no claim is left (D may have been
// entered meanwhile by another lane, which a lookup afterwards settles).
__device__ __forceinline__ int wh_claim_limited(uint64_t D, uint64_t *hk, int *ncl, bool *own) {
    uint32_t h = wh_home(D);
    *own = false;
    for (int k = 0; k < WHASH; ++k) {
        const uint64_t x = hk[h];
        if (x == D) return (int)h;
        if (x == 0ull) {
            if (atomicAdd(ncl, 1) >= NREC) {
                atomicSub(ncl, 1);
                return -1;
            }
            const unsigned long long old =
                atomicCAS((unsigned long long *)&hk[h], 0ull, (unsigned long long)D);
            *own = old == 0ull;
            if (old == 0ull) return (int)h;
            atomicSub(ncl, 1);   // the slot went to another lane's claim
            if (old == D) return (int)h;
        }
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
    return -1;
}

__device__ __forceinline__ int wl_find(det_t D, const WaveLds &W) { return wh_find(D, W.key); }
__device__ __forceinline__ int wl_claim(det_t D, WaveLds &W, bool *own, int) {
    return wh_claim(D, W.key, own);
}
__device__ __forceinline__ int wl_claim_limited(det_t D, WaveLds &W, int *ncl, bool *own, int) {
    return wh_claim_limited(D, W.key, ncl, own);
}
__device__ __forceinline__ bool wl_used(const WaveLds &W, int h) { return W.key[h] != 0ull; }
__device__ __forceinline__ void wl_clear(WaveLds &W, int h) { W.key[h] = 0ull; }
#else
__device__ __forceinline__ bool wl_used(const WaveLds &W, int h) { return W.own[h] != 0u; }
__device__ __forceinline__ void wl_clear(WaveLds &W, int h) { W.own[h] = 0u; }
__device__ __forceinline__ int wl_find(det_t D, const WaveLds &W) {
    uint32_t h = wh_home(D);
    for (int k = 0; k < WHASH; ++k) {
        if (W.own[h] == 0u) return -1;
        if (W.key[h] == D) return (int)h;
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
    return -1;
}
// Claim of a slot: lanes that find it empty race for its owner word; the winner
// writes the child, and after the wave-level ordering point every lane still
// probing compares the (now written) child with its own. A lane whose probe ends
// early leaves the loop masked off; the others stay in step.
__device__ __forceinline__ int wl_claim(det_t D, WaveLds &W, bool *own, int lane) {
    uint32_t h = wh_home(D);
    *own = false;
    for (;;) {
        bool won = false;
        if (W.own[h] == 0u) won = atomicCAS(&W.own[h], 0u, (uint32_t)lane + 1u) == 0u;
        if (won) W.key[h] = D;
        wave_sync();
        if (won) {
            *own = true;
            return (int)h;
        }
        if (W.key[h] == D) return (int)h;
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
}
__device__ __forceinline__ int wl_claim_limited(det_t D, WaveLds &W, int *ncl, bool *own,
                                                int lane) {
    uint32_t h = wh_home(D);
    *own = false;
    for (int k = 0; k < WHASH; ++k) {
        bool won = false, full = false;
        if (W.own[h] == 0u) {
            if (atomicAdd(ncl, 1) >= NREC) {
                atomicSub(ncl, 1);
                full = true;
            } else {
                won = atomicCAS(&W.own[h], 0u, (uint32_t)lane + 1u) == 0u;
                if (!won) atomicSub(ncl, 1);   // the slot went to another lane's claim
            }
        }
        if (won) W.key[h] = D;
        wave_sync();
        *own = won;
        if (won) return (int)h;
        if (full) return -1;
        if (W.key[h] == D) return (int)h;
        h = (h + 1u) & (uint32_t)(WHASH - 1);
    }
    return -1;
}
#endif

// The LDS copy of the pair table is its upper triangle, row after row: entry (p, q) at
// pair_row(p, n) + q (one entry before the first is readable, see hdiag_lds).
__device__ __forceinline__ int pair_row(int p, int n) { return p * (2 * n - p - 3) / 2 - 1; }
__device__ __forceinline__ int take_low(det_t &m) {
    const int q = dctz(m);
    m &= m - 1ull;
    return q;
}
#if FQ_DET_WORDS == 1
// H_DD = E_core + sum_p h_pp + sum_{p<q} [(pp|qq) - (pq|qp)], accumulated in ascending
// (p, q) order from the LDS copies of h_pp and of the pair table (nel: electrons, uniform).
// A chain of N (N - 1) / 2 dependent adds: bound by latency where a workgroup has few new
// determinants, by the instructions between the adds where it has many. So the occupied
// spin orbitals are taken out of the determinant once, a byte each, and the sum walks over
// words of four of them: while four entries are added, the next four are read. (Finding each
// partner's bit in the 64-bit word as it came up is eight instructions a pair.) A word's
// entries outside the sum (partners up to i, past the last) are read as well and left out:
// q <= p falls on an earlier row, at least on entry -1. A function of its own: inlined, its
// values spilled registers of the whole kernel. k_post with it, in us: 24 electrons 117 -> 103
// (3.5e6 walkers) and 1281 -> 1195 (1.4e8), 10 electrons 86 -> 78 (1.1e7).
typedef uint32_t v16u32 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) const double lds_double;
__device__ __attribute__((noinline)) double hdiag_lds(double e_core, det_t D, int nel, lds_double *hpp,
                                 lds_double *jk, int n) {
    nel = (int)uni((uint32_t)nel);
    n = (int)uni((uint32_t)n);
    const int words = (nel + 3) >> 2;
    v16u32 occ = 0u;
    double x = e_core;
    for (int w = 0; w < words; ++w) {
        uint32_t v = 0u;
        double h[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (4 * w + u >= nel) break;
            const int q = take_low(D);
            v |= (uint32_t)q << (8 * u);
            h[u] = hpp[q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (4 * w + u < nel) x = x + h[u];
        occ[w] = v;
    }
    if (nel < 2) return x;
    int i = 0, w = 0;   // electron i with the partners in word w
    lds_double *row = jk + pair_row((int)(occ[0] & 255u), n);
    double c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = row[(occ[0] >> (8 * u)) & 255u];
    for (;;) {
        int i2 = i, w2 = w + 1;
        if (w2 >= words) {
            i2 = i + 1;
            w2 = (i2 + 1) >> 2;
        }
        const bool more = i2 < nel - 1;
        double e[4] = {0.0, 0.0, 0.0, 0.0};
        if (more) {
            if (i2 != i) row = jk + pair_row((int)((occ[i2 >> 2] >> (8 * (i2 & 3))) & 255u), n);
            const uint32_t v = occ[w2];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = row[(v >> (8 * u)) & 255u];
        }
        const int lo = i + 1 - 4 * w, hi = nel - 4 * w;
        if (lo <= 0 && hi >= 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) x = x + c[u];
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u >= lo && u < hi) x = x + c[u];
        }
        if (!more) break;
        i = i2;
        w = w2;
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = e[u];
    }
    return x;
}
#endif

#if FQ_DET_WORDS == 2
// The same for two determinants of two words with the same number of electrons at once: two
// independent chains that hide each other's add latency. The table loads of four partners q
// are issued before their four dependent adds, so a sum waits once per four loads.
__device__ __forceinline__ void hdiag_lds2(double e_core, det_t da, det_t db, int nel,
                                           const double *hpp, const double *jk, int n,
                                           double &ra, double &rb) {
    double xa = e_core, xb = e_core;
    for (det_t ma = da, mb = db; ma; ma &= ma - 1ull, mb &= mb - 1ull) {
        xa = xa + hpp[dctz(ma)];
        xb = xb + hpp[dctz(mb)];
    }
    det_t m1a = da, m1b = db;
    for (int left = nel - 1; left > 0; --left) {
        const int ba = pair_row(take_low(m1a), n), bb = pair_row(take_low(m1b), n);
        det_t m2a = m1a, m2b = m1b;
        int r = left;
        for (; r >= 4; r -= 4) {
            double va[4], vb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                va[u] = jk[ba + take_low(m2a)];
                vb[u] = jk[bb + take_low(m2b)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                xa = xa + va[u];
                xb = xb + vb[u];
            }
        }
        for (; r > 0; --r) {
            xa = xa + jk[ba + take_low(m2a)];
            xb = xb + jk[bb + take_low(m2b)];
        }
    }
    ra = xa;
    rb = xb;
}

// As hdiag_lds2, with the pair table read from global memory ([n_so][NSO_MAX],
// entry (p, q) at p NSO_MAX + q): for more than 64 spin orbitals, whose upper
// triangle would take 65 KB of LDS.
__device__ __forceinline__ void hdiag_glb2(double e_core, det_t da, det_t db, const double *hpp,
                                           const double *jk, double &ra, double &rb) {
    double xa = e_core, xb = e_core;
    for (det_t ma = da, mb = db; ma; ma &= ma - 1ull, mb &= mb - 1ull) {
        xa = xa + hpp[dctz(ma)];
        xb = xb + hpp[dctz(mb)];
    }
    const gdouble *t = gptr(jk);
    for (det_t m1a = da, m1b = db; m1a; m1a &= m1a - 1ull, m1b &= m1b - 1ull) {
        const gdouble *ra_ = t + dctz(m1a) * NSO_MAX, *rb_ = t + dctz(m1b) * NSO_MAX;
        for (det_t m2a = m1a & (m1a - 1ull), m2b = m1b & (m1b - 1ull); m2a;
             m2a &= m2a - 1ull, m2b &= m2b - 1ull) {
            xa = xa + ra_[dctz(m2a)];
            xb = xb + rb_[dctz(m2b)];
        }
    }
    ra = xa;
    rb = xb;
}
#endif

// Diagonal elements of the queued new determinants (positions in the system's
// arrays, all of one system, so all with the same electron count). One word: a lane each,
// the pair table in LDS. Two words: two per thread at a time; the pair table from LDS (jk),
// or from global memory when jk is null (more than 64 spin orbitals).
#if FQ_DET_WORDS == 1
template <bool PLAIN>
__device__ __forceinline__ void flush_new_dets(const SysDesc &d, const uint32_t *queue, int n,
                                               const double *hpp, const double *jk) {
    for (int j = threadIdx.x; j < n; j += (int)blockDim.x) {
        const uint32_t i = queue[j];
        const det_t k = ldk(keys_of(d) + i);
        const double h = hdiag_lds(d.e_core, k, d.N, (lds_double *)hpp, (lds_double *)jk, d.n_so);
        *gp(d.hdiag + i) = diag_from<PLAIN>(d, k, h);
    }
}
#else
template <bool PLAIN>
__device__ __forceinline__ void flush_new_dets(const SysDesc &d, const uint32_t *queue, int n,
                                               const double *hpp, const double *jk) {
    const int step = 2 * (int)blockDim.x;
    for (int j = threadIdx.x; j < n; j += step) {
        const uint32_t i0 = queue[j];
        const bool two = j + (int)blockDim.x < n;
        const uint32_t i1 = two ? queue[j + blockDim.x] : i0;
        double h0, h1;
        const det_t k0 = ldk(keys_of(d) + i0), k1 = ldk(keys_of(d) + i1);
        if (jk)
            hdiag_lds2(d.e_core, k0, k1, d.N, hpp, jk, d.n_so, h0, h1);
        else
            hdiag_glb2(d.e_core, k0, k1, hpp, d.jk, h0, h1);
        *gp(d.hdiag + i0) = diag_from<PLAIN>(d, k0, h0);
        if (two) *gp(d.hdiag + i1) = diag_from<PLAIN>(d, k1, h1);
    }
}

// The same for a queue too short to fill the workgroup, where one lane per determinant is a
// chain of hundreds of dependent steps behind the staging of the tables: the whole workgroup
// gathers the terms
// of up to `cap` determinants from the tables in memory into LDS, then one lane per
// determinant adds them up in their order. A determinant takes `stride` bytes of LDS: itself,
// the numbers of its occupied spin orbitals, and its terms (h_pp of its N electrons, then
// the pairs in ascending (p, q) order), an odd number of places in all so that the adding
// lanes meet different banks. Whole workgroup; the queue is complete and `lds` free.
struct FewDets {
    int terms, stride, cap;   // per determinant: terms, bytes of LDS; determinants at once
    __device__ __forceinline__ FewDets(int nel, int bytes) {
        terms = nel * (nel + 1) / 2;
        // (in units of a determinant, an odd number of them)
        constexpr int U = (int)sizeof(det_t);
        stride = ((terms * 8 + NSO_MAX + 2 * U - 1) / U | 1) * U;
        cap = bytes / stride < 256 ? bytes / stride : 256;
    }
};
template <bool PLAIN>
__device__ __forceinline__ void flush_few(const SysDesc &d, const uint32_t *queue, int n,
                                          const FewDets &f, char *lds) {
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int N = d.N;
    const int per_it = 256 / f.terms, rest = 256 % f.terms;
    const auto key_at = [&](int j) { return (det_t *)(lds + j * f.stride); };
    const auto orb_at = [&](int j) { return (uint8_t *)(lds + j * f.stride + sizeof(det_t)); };
    const auto sum_at = [&](int j) { return (double *)(lds + j * f.stride + sizeof(det_t) + NSO_MAX); };
    for (int j0 = 0; j0 < n; j0 += f.cap) {
        const int m = n - j0 < f.cap ? n - j0 : f.cap;
        uint32_t at = 0u;
        if (t < m) {
            at = queue[j0 + t];
            *key_at(t) = ldk(keys_of(d) + at);
        }
        __syncthreads();
        for (int j = wid; j < m; j += 4) {
            const det_t D = *key_at(j);
            uint8_t *const o = orb_at(j);
            for (int p = lane; p < 64 * FQ_DET_WORDS; p += 64)
                if ((bool)(D & DBIT(p))) o[dpopc(D & (DBIT(p) - 1ull))] = (uint8_t)p;
        }
        __syncthreads();
        // term k of determinant j; the next one of this thread is 256 terms on
        int j = t / f.terms, k = t % f.terms;
        while (j < m) {
            double x[8];
            double *to[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                to[u] = nullptr;
                if (j < m) {
                    const uint8_t *const o = orb_at(j);
                    to[u] = sum_at(j) + k;
                    if (k < N) {
                        x[u] = h_so(d, o[k], o[k]);
                    } else {
                        // the pair: row i begins at term i (2 N - i - 1) / 2 of the pairs
                        const int v = k - N, b = 2 * N - 1;
                        int i = (int)(((float)b - sqrtf((float)(b * b - 8 * v))) * 0.5f);
                        i = i * (b - i) / 2 > v ? i - 1 : i;
                        i = (i + 1) * (b - i - 1) / 2 <= v ? i + 1 : i;
                        x[u] = gptr(d.jk)[o[i] * NSO_MAX + o[i + 1 + v - i * (b - i) / 2]];
                    }
                }
                j += per_it;
                k += rest;
                if (k >= f.terms) {
                    k -= f.terms;
                    ++j;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (to[u]) *to[u] = x[u];
        }
        __syncthreads();
        if (t < m) {
            const double *const v = sum_at(t);
            double x = d.e_core;
            int i = 0;
            for (; i + 8 <= f.terms; i += 8) {
                double y[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) y[u] = v[i + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) x = x + y[u];
            }
            for (; i < f.terms; ++i) x = x + v[i];
            *gp(d.hdiag + at) = diag_from<PLAIN>(d, *key_at(t), x);
        }
        __syncthreads();
    }
}
#endif

// Adding up statistics: by their owner, and (any order) into a system's share in memory.
__device__ __forceinline__ void add_stat(IterStat &x, const IterStat &y) {
    x.nw += y.nw;
    x.nd += y.nd;
    x.merged += y.merged;
    x.aborted += y.aborted;
    x.used += y.used;
    x.born += y.born;
    x.num = x.num + y.num;
}
__device__ __forceinline__ void add_stat_global(IterStat *x, const IterStat &y) {
    atomicAdd((unsigned long long *)&x->nw, (unsigned long long)y.nw);
    atomicAdd((unsigned long long *)&x->nd, (unsigned long long)y.nd);
    if (y.merged) atomicAdd((unsigned long long *)&x->merged, (unsigned long long)y.merged);
    if (y.aborted) atomicAdd((unsigned long long *)&x->aborted, (unsigned long long)y.aborted);
    atomicAdd((unsigned long long *)&x->used, (unsigned long long)y.used);
    if (y.born) atomicAdd((unsigned long long *)&x->born, (unsigned long long)y.born);
    if (y.num != 0.0) unsafeAtomicAdd(&x->num, y.num);
}

__device__ __forceinline__ uint64_t lanes_below(int lane) { return (1ull << lane) - 1ull; }

// Sum over the wavefront's lanes of a per-lane count v < 8, from ballots of its bits.
__device__ __forceinline__ int wave_total8(int v) {
    return __popcll(__ballot(v & 1)) + 2 * __popcll(__ballot(v & 2)) + 4 * __popcll(__ballot(v & 4));
}

// PLAIN: as for k_spawn.
template <bool PLAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_post(EngineArgs a, const SysDesc *__restrict__ desc) {
    // Each wavefront's working set, and (between chunks only) the pair table from
    // which the diagonal elements of new determinants are computed.
    struct PairTable {
        double before;            // (read as entry -1, never used)
        double jk[64 * 63 / 2];   // (up to 64 spin orbitals)
        double hpp[NSO_MAX];
    };
#if FQ_DET_WORDS == 1
    // side by side: the staged pair table stays valid while the wavefronts use theirs
    struct PostLds {
        WaveLds w[POST_WAVES];
        PairTable tab;
    };
#else
    union PostLds {   // (two words: no room for both at four workgroups per CU)
        WaveLds w[POST_WAVES];
        PairTable tab;
    };
#endif
    __shared__ PostLds L;
    __shared__ uint32_t s_queue[POST_QUEUE];
    __shared__ uint32_t s_stat[POST_MAX_SYS];   // the systems' status at the kernel's start
    // Metadata of a window of POST_WIN chunks, read once for all its buckets.
    __shared__ int s_csys[POST_WIN];                 // system of the chunk (-1: not taking part)
    __shared__ int s_cloc[POST_WIN];                 // chunk index inside its system's table
    __shared__ uint8_t s_cnext[POST_WIN];            // its walkers spawn next iteration
    __shared__ int16_t s_bn[POST_WIN * BPC];         // entries per bucket
    __shared__ uint32_t s_nr[POST_WIN * BPC];        // records per bucket
    __shared__ unsigned long long s_bnw[POST_WIN * BPC];   // walkers per bucket that spawn next
    __shared__ int s_qn, s_qsys;
#if FQ_DET_WORDS == 1
    __shared__ int s_tabsys;                         // system whose pair table is staged (-1: none)
#endif
    __shared__ int s_ncl[POST_WAVES];
    __shared__ int64_t s_win;                        // first chunk of the window taken
    __shared__ unsigned int s_len[NLIST];            // windows per list
    __shared__ int s_list;                           // list taken from
    __shared__ IterStat s_acc[POST_WAVES];           // statistics of system s_accsys
    __shared__ int s_accsys;
    const int64_t nch = *a.nchunks;
    // (The wavefront's number, a segment's system and a bucket's sizes are left to vector
    // registers: as scalars they were loaded again at each use, 1.44 instead of 1.23 ms at
    // 1.4e8 walkers. The kernel spills 143 scalar and 68 vector registers as it is.)
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    WaveLds &W = L.w[wid];
    if (blockIdx.x == 0 && t < NLIST) {   // k_spawn's counters, for the next iteration
        a.work[CTR_SPAWN(t)] = 0u;
        a.total[CTR_TILES(2, t)] = 0ull;
        if (t == 0) {
            a.work[CTR_FALLBACK] = 0u;
            a.total[CTR_UNLISTED(2)] = 0ull;
        }
    }
    // Which systems take part is decided from the status at the start: bits set while
    // this kernel runs (population overflow) are fatal to their system anyway.
    for (int i = t; i < a.max_sys && i < POST_MAX_SYS; i += 256) s_stat[i] = a.status[i];
    if (t == 0) {
        s_qn = 0;
        s_qsys = -1;
#if FQ_DET_WORDS == 1
        s_tabsys = -1;
#endif
        s_accsys = -1;
        for (int w = 0; w < POST_WAVES; ++w) s_acc[w] = IterStat{};
    }
    auto flush = [&]() {   // (uniform) H_DD of the queued new determinants
        const int sq = (int)uni((uint32_t)s_qsys);
        const int qn = (int)uni((uint32_t)s_qn), nq = qn < POST_QUEUE ? qn : POST_QUEUE;
        const SysDesc &dq = desc[sq];
#if FQ_DET_WORDS == 1
        if (s_tabsys != sq) {   // (uniform)
            const int n = dq.n_so, q = t & 63;
#pragma unroll
            for (int v = 0; v < 64; v += 32) {
                if (v >= n) break;
                double x[8];   // (eight loads under way at a time)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int p = v + 4 * u + wid;
                    x[u] = q > p && q < n ? gptr(dq.jk)[p * NSO_MAX + q] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int p = v + 4 * u + wid;
                    if (q > p && q < n) L.tab.jk[pair_row(p, n) + q] = x[u];
                }
            }
            if (t < n) L.tab.hpp[t] = h_so(dq, t, t);
            __syncthreads();
            if (t == 0) s_tabsys = sq;   // (read again only after the barrier below)
        }
        flush_new_dets<PLAIN>(dq, s_queue, nq, L.tab.hpp, L.tab.jk);
#else
        // Few of them, up to four of flush_few's batches (a batch takes 3 to 5 us; staging the
        // tables, which two words have no room to keep, 7, and a sum from them 10 to 20: k_post
        // with 10 electrons in 36 orbitals 73 -> 61 us at 2.2e6 walkers).
        const FewDets few(dq.N, (int)sizeof L);
        if (nq <= 4 * few.cap) {
            flush_few<PLAIN>(dq, s_queue, nq, few, (char *)&L);
            return;
        }
        const bool in_lds = dq.n_so <= 64;   // the pair table's upper triangle fits in LDS
        if (in_lds)
            for (int i = t; i < dq.n_so * 64; i += 256) {
                const int p = i >> 6, q = i & 63;
                if (q > p && q < dq.n_so)
                    L.tab.jk[pair_row(p, dq.n_so) + q] = gptr(dq.jk)[p * NSO_MAX + q];
            }
        for (int i = t; i < dq.n_so; i += 256) L.tab.hpp[i] = h_so(dq, i, i);
        __syncthreads();
        flush_new_dets<PLAIN>(dq, s_queue, nq, L.tab.hpp, in_lds ? L.tab.jk : nullptr);
#endif
        __syncthreads();
    };
    auto flush_stat = [&]() {   // (thread f < 7 hands over the f-th number)
        if (s_accsys < 0 || t > 6) return;
        IterStat *const to = a.acc + s_accsys * ACC_SLOTS + (blockIdx.x & (ACC_SLOTS - 1));
        if (t < 6) {
            unsigned long long x = 0;
            for (int w = 0; w < POST_WAVES; ++w) {
                unsigned long long *const f = (unsigned long long *)&s_acc[w] + t;
                x += *f;
                *f = 0ull;
            }
            if (x) atomicAdd((unsigned long long *)to + t, x);
        } else {
            double x = 0.0;
            for (int w = 0; w < POST_WAVES; ++w) {
                x = x + s_acc[w].num;
                s_acc[w].num = 0.0;
            }
            if (x != 0.0) unsafeAtomicAdd(&to->num, x);   // (the hardware's add: device memory)
        }
    };
    // The workgroups take windows of consecutive chunks from shared counters (so the
    // faster ones take more): POST_WIN chunks when every workgroup gets many, fewer for
    // small launches, down to one window each (a window costs a dozen us of its own: the
    // counter, the metadata's chain of loads, the barriers); inside a window the wavefronts run through the chunks
    // independently. When it is done, its buckets' tiles are appended to the next
    // iteration's list.
    const int64_t per_wg = (nch + gridDim.x - 1) / gridDim.x;
    const int gwin = per_wg <= 8 ? (int)per_wg : per_wg < 32 ? 8 : per_wg < 4 * POST_WIN ? (int)(per_wg / 4) : POST_WIN;
    // List l holds the windows of the l-th of NLIST equal ranges of windows; the last
    // wavefront does the taking.
    const auto win0 = [&](int l) { return (uint32_t)((nch + gwin - 1) / gwin) * (uint64_t)l / NLIST; };
    if (t < NLIST) s_len[t] = (unsigned int)(win0(t + 1) - win0(t));
    if (t == 0) {
        s_list = (int)(blockIdx.x & (NLIST - 1));
        s_win = -1;
    }
    // Each pass takes a segment: consecutive chunks of one system in the window at hand, at
    // most post_seg (or first the next window). Between segments the workgroup meets and
    // empties its queue of new determinants when it holds one per thread or belongs to
    // another system. What does not go through the queue (one system at a time, POST_QUEUE
    // places) is computed in place, a chain of gathers that stops a wavefront for 100 us;
    // hence a segment per system, shorter ones where lists grow fast. The queue is kept over
    // windows: small launches bring few new determinants per window, and emptying it is a
    // latency of its own.
    int64_t c0 = 0;
    int nwin = 0, ci = 0;      // the window's chunks, and the segment's first
    bool begin = true;
    for (;;) {
        __syncthreads();   // the previous segment is done
        const bool fresh = ci >= nwin;
        if (fresh) {
            if (wid == POST_WAVES - 1) {
                unsigned int at = 0, count = 0;
                Handout ho{a.work + CTR_POST(0), s_len, 1u, 1u, __builtin_amdgcn_readfirstlane(s_list), begin};
                const bool more = handout_next(ho, blockIdx.x / NLIST, at, count);
                if (lane == 0) {
                    s_win = more ? (int64_t)(win0(ho.list) + at) * gwin : nch;
                    s_list = ho.list;
                }
            }
            // list the tiles of the window just done
            if (t < (nwin * BPC + 63) / 64 * 64) {   // (whole wavefronts)
                const bool in = t < nwin * BPC;
                emit_tiles(a, cur_half(a) ^ 1, (int)((c0 / gwin) & (NLIST - 1)), c0 * BPC + t,
                           in ? s_csys[t / BPC] : 0, in ? (uint32_t)(s_cloc[t / BPC] * BPC + t % BPC) : 0u,
                           in ? s_bnw[t] : 0ull, in ? s_bn[t] : 0);
            }
            __syncthreads();
            c0 = (int64_t)uni((uint64_t)s_win);
            begin = false;
            ci = 0;
            nwin = (int)(nch - c0 < gwin ? nch - c0 : gwin);
        }
        const bool done = c0 >= nch;
        const int nsys = done ? -2 : fresh ? a.chunk_sys[c0] : s_csys[ci];
        if (s_qn >= POST_FLUSH || (s_qn > 0 && nsys != s_qsys)) {   // (uniform)
            flush();
            if (t == 0) s_qn = 0;
        }
        // the workgroup's statistics belong to one system: handed over at a change
        if (fresh && nsys != s_accsys) flush_stat();
        if (done) break;
        __syncthreads();
        if (t == 0) {
            if (s_qn == 0) s_qsys = -1;
            if (fresh) s_accsys = nsys;
        }
        if (fresh) {
            if (t < nwin) {
                const int sc = a.chunk_sys[c0 + t];
                bool live = false, next = false;
                if (sc >= 0) {
                    const SysDesc &dc = desc[sc];
                    live = participating(dc, sc < POST_MAX_SYS ? s_stat[sc] : a.status[sc]);
                    next = live && dc.iter + 1 < dc.stop_at;
                }
                s_csys[t] = live ? sc : -1;
                s_cloc[t] = a.chunk_local[c0 + t];
                s_cnext[t] = next ? 1 : 0;
            }
            uint32_t nrec = 0;
            if (t < nwin * BPC) {
                nrec = a.bhist[c0 * BPC + t];
                if (nrec) {
                    a.bhist[c0 * BPC + t] = 0u;   // counted afresh next iteration
                    a.bprev[c0 * BPC + t] = nrec;
                }
                s_nr[t] = nrec;
                // the fullest bucket, from which the host plans the slots (of an abandoned
                // iteration too: its dropped records were counted)
                const int sr = nrec ? a.chunk_sys[c0 + t / BPC] : -1;
                if (sr >= 0 && nrec > a.rec_max[sr]) atomicMax(&a.rec_max[sr], nrec);
            }
            __syncthreads();
            if (t < nwin * BPC) {
                const int sc = s_csys[t / BPC];
                s_bn[t] = sc >= 0 ? (int16_t)desc[sc].bcnt[(int64_t)s_cloc[t / BPC] * BPC + t % BPC] : 0;
            }
        }
        __syncthreads();
        // this wavefront's statistics over the segment's buckets (per lane)
        int64_t a_nw = 0, a_ab = 0, a_born = 0;
        uint64_t a_cnt = 0;
        double a_num = 0.0;
        const int s = s_csys[ci];
        const bool live = s >= 0;
        const uint64_t cut = __ballot(lane > ci && (lane >= nwin || s_csys[lane & (POST_WIN - 1)] != s ||
                                                    lane % a.post_seg == 0));
        const int seg_end = __builtin_ctzll(cut);   // (lane POST_WIN >= nwin is always set)
        for (; ci < seg_end; ++ci) {
            int64_t nw = 0, aborted = 0;
            uint64_t cnt = 0;                 // entries | merged targets << 21 | occupied << 42
            double num = 0.0;
            unsigned long long nwb = 0;       // sum |C| over the bucket's entries after the iteration
            int64_t born = 0;                 // new determinants (uniform)
            if (live) {
                const SysDesc &d = desc[s];
                uint32_t *status = &a.status[s];
                const int64_t lb = (int64_t)s_cloc[ci] * BPC + wid;
                const int64_t base = lb * BQ;
                const int n = s_bn[ci * BPC + wid];
                const uint32_t nr = s_nr[ci * BPC + wid];
                rec_t *const seg = recs_of(a) + d.rec0 + lb * d.rec_r;   // the bucket's records
                // fast path: one record per lane, all in the bucket's own slots
                const bool fast = nr <= (uint32_t)NREC && nr <= (uint32_t)d.rec_r;
                // slow path: record j (see put_record)
                auto rec_at = [&](uint32_t j) -> rec_t * {
                    if (j < (uint32_t)d.rec_r) return seg + j;
                    const uint64_t x = a.bext[(c0 + ci) * BPC + wid];
                    return recs_of(a) + ((int64_t)(x >> EXT_BITS) + (j - (uint32_t)d.rec_r));
                };
                // the H_DD queue serves one system at a time: the first to use it in a window
                if (lane == 0 && s_qsys < 0) atomicCAS(&s_qsys, -1, s);
                // entry u * 64 + lane is this lane's u-th; R rounds cover the n entries
                const int R = (n + 63) >> 6;
                det_t kin[4] = {det_t(0ull), det_t(0ull), det_t(0ull), det_t(0ull)};
                int32_t pin[4] = {0, 0, 0, 0};
                double hin[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (u >= R) break;
                    if ((u << 6) + lane < n) {
                        kin[u] = ldk(keys_of(d) + base + (u << 6) + lane);
                        pin[u] = *gp(d.pop + base + (u << 6) + lane);
                        hin[u] = *gp(d.hdiag + base + (u << 6) + lane);
                    }
                }
                det_t rd = det_t(0ull);   // this lane's record (fast path), its hash slot, and
                int32_t rw = 0;       // whether this lane entered the child there
                uint32_t rf = 0u;
                int rh = 0;
                bool rown = false;
                if ((uint32_t)lane < nr && fast) {
                    const rec_t r = get_rec(seg + lane);
                    rd = r.det;
                    rw = r.w;
                    rf = r.tag;
                }
                wl_clear(W, lane);
                wl_clear(W, lane + 64);
                W.acc[lane] = 0ll;
                W.acc[lane + 64] = 0ll;
                W.flg[lane] = 0u;
                W.flg[lane + 64] = 0u;
                // death of every entry (Eq. pdeath, one stochastic rounding for the whole
                // determinant); it depends on nothing that arrives
                // (branch-free over the lanes: p = 0 past the bucket's entries gives pd = 0)
                int32_t pdv[4] = {0, 0, 0, 0};
                bool ovf = false;   // a population left int32 (reported once for the bucket)
    #pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (u >= R) break;
                    const int32_t p = pin[u];
                    uint64_t xd, xu;
                    draw2(d.seed, kin[u], 0xFFFFFFFFu, d.iter, 0x80u, xd, xu);
                    const uint32_t absC = (uint32_t)(p < 0 ? -p : p);   // |p| <= 2^31 - 1
                    const double dv = ((hin[u] - d.e0) - d.shift) * d.tau * (double)absC;
                    const double ad = fabs(dv);
                    const double fl = floor(ad);
                    const bool big = fl > 1073741824.0;   // the entry is left as it is
                    // m <= 2^30 + 1; C - sign(C) sign(d) m
                    const int32_t m = (int32_t)(big ? 0.0 : fl) + (u01(xd) < ad - fl ? 1 : 0);
                    const int64_t pm = (int64_t)p + (((p > 0) == (dv > 0.0)) ? -(int64_t)m : (int64_t)m);
                    const bool range = pm > 2147483647ll || pm < -2147483647ll;
                    ovf |= p != 0 && (big || range);
                    pdv[u] = p == 0 ? 0 : big ? p : range ? 0 : (int32_t)pm;
                }
                wave_sync();
                long long spv[4] = {0ll, 0ll, 0ll, 0ll};   // walkers arrived per entry
                uint32_t flv = 0u;                         // bit u: an initiator sent some
                if (fast) {
                    // Fast path: at most NREC records, so at most NREC distinct children.
                    if ((uint32_t)lane < nr) {
                        rh = wl_claim(rd, W, &rown, lane);
                        atomicAdd((unsigned long long *)&W.acc[rh], (unsigned long long)(long long)rw);
                        if (rf & F_INIT) atomicOr(&W.flg[rh], F_INIT);
                    }
                    wave_sync();
                    if (nr > 0) {
    #pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (u >= R) break;
                            if ((u << 6) + lane >= n) continue;
                            const int h = wl_find(kin[u], W);
                            if (h < 0) continue;
                            spv[u] = W.acc[h];
                            flv |= (W.flg[h] & F_INIT) << u;
                            W.flg[h] |= F_MATCHED;   // a child matches at most one entry
                        }
                    }
                    wave_sync();
                } else {
                    // Slow path: rounds of at most NREC distinct children. A child whose
                    // records found the hash full is left whole for a later round; the
                    // children outside the bucket are staged, merged, in the slots of the
                    // records that entered them.
                    for (int round = 0;; ++round) {
                        if (round > 0) {
                            wl_clear(W, lane);
                            wl_clear(W, lane + 64);
                            W.acc[lane] = 0ll;
                            W.acc[lane + 64] = 0ll;
                            W.flg[lane] = 0u;
                            W.flg[lane + 64] = 0u;
                        }
                        if (lane == 0) s_ncl[wid] = 0;
                        wave_sync();
                        bool maybe = false;
                        for (uint32_t j = lane; j < nr; j += 64) {   // (a record stays with its lane)
                            const rec_t r = get_rec(rec_at(j));
                            if (round > 0 && !(r.tag & F_DEFER)) continue;
                            bool own;
                            const int h = wl_claim_limited(r.det, W, &s_ncl[wid], &own, lane);
                            if (h < 0) {
                                rec_at(j)->tag = (r.tag & F_INIT) | F_MAYBE;
                                maybe = true;
                                continue;
                            }
                            if (r.tag & F_DEFER) rec_at(j)->tag = r.tag & F_INIT;
                            atomicAdd((unsigned long long *)&W.acc[h], (unsigned long long)(long long)r.w);
                            const uint32_t f = (r.tag & F_INIT) | (own ? j << OWN_SHIFT : 0u);
                            if (f) atomicOr(&W.flg[h], f);
                        }
                        wave_sync();
                        bool defer = false;
                        if (__ballot(maybe)) {
                            for (uint32_t j = lane; j < nr; j += 64) {
                                const rec_t r = get_rec(rec_at(j));
                                if (!(r.tag & F_MAYBE)) continue;
                                const int h = wl_find(r.det, W);
                                if (h < 0) {
                                    rec_at(j)->tag = (r.tag & F_INIT) | F_DEFER;
                                    defer = true;
                                    continue;
                                }
                                rec_at(j)->tag = r.tag & F_INIT;
                                atomicAdd((unsigned long long *)&W.acc[h],
                                          (unsigned long long)(long long)r.w);
                                if (r.tag & F_INIT) atomicOr(&W.flg[h], F_INIT);
                            }
                            wave_sync();
                        }
    #pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (u >= R) break;
                            if ((u << 6) + lane >= n) continue;
                            const int h = wl_find(kin[u], W);
                            if (h < 0) continue;
                            spv[u] += W.acc[h];
                            flv |= (W.flg[h] & F_INIT) << u;
                            W.flg[h] |= F_MATCHED;
                        }
                        wave_sync();
                        // stage this round's children outside the bucket (one per slot)
                        for (int h = lane; h < WHASH; h += 64) {
                            const uint32_t f = W.flg[h];
                            if (!wl_used(W, h) || (f & F_MATCHED)) continue;
                            long long sp = W.acc[h];
                            if (sp > 2147483647ll || sp < -2147483647ll) {
                                atomicOr(status, ST_POP_OVERFLOW);
                                sp = 0;
                            }
                            put_rec(rec_at(f >> OWN_SHIFT), W.key[h], (int32_t)sp, (f & F_INIT) | F_STAGED);
                        }
                        wave_sync();
                        if (!__ballot(defer)) break;
                    }
                    __threadfence();   // the staged children, read back below by other lanes
                }
                // Annihilation (Sec. 4.2) of the bucket's own entries.
                int32_t npv[4] = {0, 0, 0, 0};
                uint32_t keepm = 0u;
                uint32_t nearm = 0u;   // bit u: entry u contributes to the projected energy
                int reborn = 0;        // entries emptied by death and re-entered by initiator
                                       // spawns (new determinants kept in place)
                // (branch-free over the lanes: past the bucket's entries D = 0, and nothing
                // arrives, so np = 0 and nothing is counted)
    #pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (u >= R) break;
                    const det_t D = kin[u];
                    const bool is_ref = D == ref_of(d);
                    const int64_t pd = pdv[u];
                    // (walkers spawned onto the reference arrive in their own sum)
                    long long sp = spv[u];
                    if (is_ref) sp += a.d0acc[s];
                    const bool alive = pd != 0 || is_ref;
                    const bool reb = !alive && sp != 0 && ((flv >> u) & 1u);
                    const long long asp = sp < 0 ? -sp : sp;
                    int64_t np = alive ? pd + sp : (reb ? sp : 0ll);
                    reborn += reb ? 1 : 0;
                    aborted += (!alive && !reb) ? asp : 0ll;
                    cnt += sp != 0 ? 1ull << CNT_SHIFT_MERGED : 0ull;
                    const bool range = np > 2147483647ll || np < -2147483647ll;
                    ovf |= range;
                    np = range ? 0ll : np;
                    npv[u] = (int32_t)np;
                    if (is_ref) {
                        a.c0[s] = np;
                        a.d0acc[s] = 0ll;   // consumed
                    }
                    const int64_t an = np < 0 ? -np : np;
                    nw += an;
                    nwb += (unsigned long long)an;
                    cnt += np != 0 ? 1ull << CNT_SHIFT_ND : 0ull;
                    nearm |= (np != 0 && !is_ref && near_ref<PLAIN>(d, D)) ? 1u << u : 0u;
                    keepm |= (np != 0 || is_ref) ? 1u << u : 0u;   // the reference keeps its entry at 0
                }
                if (ovf) atomicOr(status, ST_POP_OVERFLOW);
                // positions emptied this iteration, ascending (round by round, lanes in order)
                int H = 0;
    #pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (u >= R) break;
                    const bool hole = (u << 6) + lane < n && !((keepm >> u) & 1u);
                    const uint64_t m = __ballot(hole);
                    if (hole) W.free_[H + __popcll(m & lanes_below(lane))] = (uint16_t)((u << 6) + lane);
                    H += __popcll(m);
                }
                const int Lk = n - H;
                wave_sync();
                // New determinants: children outside the bucket with an initiator parent go
                // to the emptied positions first, then past the end; the others are discarded.
                int K = 0;
                // (all lanes; D = 0: none.) Returns where the determinant's diagonal element is
                // still to be computed: its position in the bucket, DIAG_SPILL + its place in
                // the spill list, or -1 (none, or queued).
                auto place = [&](det_t D, long long sp, bool init) -> int {
                    const bool real = D != det_t(0ull) && sp != 0;
                    if (real) cnt += 1ull << CNT_SHIFT_MERGED;
                    if (real && !init) aborted += sp < 0 ? -sp : sp;
                    const bool nd = real && init;
                    const uint64_t m = __ballot(nd);
                    const int k = K + __popcll(m & lanes_below(lane));
                    K += __popcll(m);
                    if (!nd) return -1;
                    const int64_t an = sp < 0 ? -sp : sp;
                    nw += an;
                    cnt += 1ull << CNT_SHIFT_ND;
                    const int pos = k < H ? (int)W.free_[k] : n + (k - H);
                    if (pos < BQ) {
                        nwb += (unsigned long long)an;
                        stk(keys_of(d) + base + pos, D);
                        *gp(d.pop + base + pos) = (int32_t)sp;
                        const int q = s_qsys == s ? atomicAdd(&s_qn, 1) : POST_QUEUE;
                        if (q >= POST_QUEUE) return pos;   // (many new determinants)
                        s_queue[q] = (uint32_t)(base + pos);
                    } else {
                        // the bucket is full: completed in the spill list, re-bucketed by the host
                        const unsigned long long j = atomicAdd(a.sp_count, 1ull);
                        if (j < (unsigned long long)a.sp_cap) {
                            spill_dets(a)[j] = D;
                            a.sp_pop[j] = (int32_t)sp;
                            a.sp_sys[j] = s;
                            a.spilled[s] = 1u;
                            return DIAG_SPILL + (int)j;
                        } else {
                            atomicOr(status, ST_SPILL_FULL);
                        }
                    }
                    return -1;
                };
                int diag = -1;         // fast path: place()'s answer for this lane's child
                long long rsp = 0ll;   // fast path: walkers that arrived for this lane's child
                if (fast) {
                    // one lane per distinct child: the lane that entered it into the hash
                    const uint32_t f = rown ? W.flg[rh] : F_MATCHED;
                    const bool cand = !(f & F_MATCHED);
                    rsp = cand ? W.acc[rh] : 0ll;
                    if (rsp > 2147483647ll || rsp < -2147483647ll) {
                        atomicOr(status, ST_POP_OVERFLOW);
                        rsp = 0ll;
                    }
                    rf = cand ? f & F_INIT : 0u;   // (set: a new determinant)
                    diag = place(cand && rsp != 0ll ? rd : det_t(0ull), rsp, (f & F_INIT) != 0u);
                } else {
                    for (uint32_t i0 = 0; i0 < nr; i0 += 64) {
                        const uint32_t i = i0 + lane;
                        const rec_t r = get_rec(rec_at(i < nr ? i : 0u));
                        const bool in = i < nr && (r.tag & F_STAGED);
                        const int at = place(in ? r.det : det_t(0ull), in ? (long long)r.w : 0ll,
                                             in && (r.tag & F_INIT));
                        if (at >= 0) rec_at(i)->tag = r.tag | (uint32_t)(at + 1) << DIAG_SHIFT;
                    }
                }
                // Re-pack: n' = (kept entries) + (new determinants); when fewer new
                // determinants than emptied positions arrived, the kept entries past n' move
                // into the emptied positions that remain below n'.
                const int np_ = Lk + K < BQ ? Lk + K : BQ;
                uint32_t movedm = 0u;
                if (K < H) {   // uniform
                    int r = K;
    #pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (u >= R) break;
                        const bool mv = ((keepm >> u) & 1u) && (u << 6) + lane >= np_;
                        const uint64_t m = __ballot(mv);
                        if (mv) {
                            const int64_t dst = base + W.free_[r + __popcll(m & lanes_below(lane))];
                            stk(keys_of(d) + dst, kin[u]);
                            *gp(d.pop + dst) = npv[u];
                            *gp(d.hdiag + dst) = hin[u];
                            movedm |= 1u << u;
                        }
                        r += __popcll(m);
                    }
                }
    #pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (((keepm & ~movedm) >> u) & 1u && npv[u] != pin[u])
                        *gp(d.pop + base + (u << 6) + lane) = npv[u];
                if (lane == 0) {
                    d.bcnt[lb] = np_;
                    s_bn[ci * BPC + wid] = (int16_t)np_;
                    cnt += (uint64_t)np_;
                }
                born = K + wave_total8(reborn);
                // Projected-energy numerator (Eq. ProjE), the occupied determinants within a
                // double excitation of the reference, and the diagonal elements still to be
                // computed, taken last, when few values are live: a lane's entries (bits 0-3
                // of todo) and its new determinant (bits 4 and 5; many of them on the slow
                // path).
                for (uint32_t i0 = 0; i0 == 0 || (!fast && i0 < nr); i0 += 64) {
                    bool fresh_det = fast && rown && rf != 0u && rsp != 0ll;
                    if (!fast) {
                        const uint32_t i = i0 + lane;
                        const rec_t r = get_rec(rec_at(i < nr ? i : 0u));
                        fresh_det = i < nr && (r.tag & F_STAGED) && (r.tag & F_INIT) && r.w != 0;
                        rd = r.det;
                        rsp = r.w;
                        diag = fresh_det ? (int)(r.tag >> DIAG_SHIFT) - 1 : -1;
                    }
                    uint32_t todo = (i0 == 0 ? nearm : 0u) |
                                    (fresh_det && near_ref<PLAIN>(d, rd) ? 1u << 4 : 0u) |
                                    (diag >= 0 ? 1u << 5 : 0u);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if ((todo >> u) & 1u) num = num + ref_hel<PLAIN>(d, kin[u]) * (double)npv[u];
                    if ((todo >> 4) & 1u) num = num + ref_hel<PLAIN>(d, rd) * (double)rsp;
                    if ((todo >> 5) & 1u) {
                        double *const to = diag >= DIAG_SPILL ? a.sp_hd + (diag - DIAG_SPILL)
                                                              : d.hdiag + base + diag;
                        *gp(to) = diag_from<PLAIN>(d, rd, hdiag_of(d, rd));
                    }
                }
            }
            a_nw += nw;
            a_ab += aborted;
            a_cnt += cnt;
            a_num = a_num + num;
            a_born += born;
            // the wavefront's statistics at the segment's end: into the workgroup's sums, or
            // (another system) the system's
            if (ci + 1 == seg_end && live) {
                IterStat st;
                st.nw = wave_sum((long long)a_nw);
                st.aborted = wave_sum((long long)a_ab);
                const uint64_t c3 = wave_sum((unsigned long long)a_cnt);
                st.used = (int64_t)(c3 & CNT_FIELD);
                st.merged = (int64_t)((c3 >> CNT_SHIFT_MERGED) & CNT_FIELD);
                st.nd = (int64_t)(c3 >> CNT_SHIFT_ND);
                st.born = a_born;
                st.num = wave_sum(a_num);
                if (lane == 0) {
                    if (s == s_accsys) add_stat(s_acc[wid], st);
                    else add_stat_global(a.acc + s * ACC_SLOTS + (blockIdx.x & (ACC_SLOTS - 1)), st);
                }
            }
            {   // the wavefront's total, by DPP (all lanes active here)
                const unsigned long long x = wave_incl_scan(nwb);
                nwb = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63) |
                      ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), 63) << 32);
            }
            if (lane == 0) {
                // walkers that spawn next iteration: none if the system stops after this one
                s_bnw[ci * BPC + wid] = s_cnext[ci] ? nwb : 0ull;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// K5: per system (one wavefront): sum of the ACC_SLOTS shares of its statistics, the shift
// update, the per-iteration record.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_finalize(EngineArgs a) {
    const int s = blockIdx.x;
    if (s == 0 && threadIdx.x == 0) *a.step += 1ull;   // every kernel of this iteration has read it
    SysDesc &d = a.desc[s];
    const int t = threadIdx.x;
    IterStat p{};
    if (t < ACC_SLOTS) {   // (emptied also for a system that has just stopped)
        p = a.acc[s * ACC_SLOTS + t];
        a.acc[s * ACC_SLOTS + t] = IterStat{};
    }
    if (!participating(d, a.status[s])) return;   // uniform across the wavefront
    const int64_t nw = wave_sum((long long)p.nw);
    const int64_t nd = wave_sum((long long)p.nd);
    const int64_t c0 = a.c0[s];
    const int64_t merged = wave_sum((long long)p.merged);
    const int64_t aborted = wave_sum((long long)p.aborted);
    const int64_t used = wave_sum((long long)p.used);
    const int64_t born = wave_sum((long long)p.born);
    const double num = wave_sum(p.num);
    unsigned long long spawned = t < SPAWN_SLOTS ? a.spawns[s * SPAWN_SLOTS + t] : 0ull;
    if (t < SPAWN_SLOTS) a.spawns[s * SPAWN_SLOTS + t] = 0ull;
    spawned = wave_sum(spawned);
    if (t == 0) {
        const int64_t done = d.iter + 1;
        {
            if (done % d.A == 0) {
                if (!d.varying) {
                    if (nw >= d.target) {
                        d.varying = 1;
                        d.n_prev = nw;
                        d.n_var = done;
                    }
                } else {
                    d.shift = d.shift - (d.zeta / ((double)d.A * d.tau)) *
                                            shift_log((double)nw / (double)d.n_prev);
                    d.n_prev = nw;
                }
            }
            if (nw == 0) a.status[s] |= ST_DIED;
        }
        IterRecord r;
        r.iter = done;
        r.nw = nw;
        r.nd = nd;
        r.c0 = c0;
        r.attempts = d.nw;   // one per walker at the iteration's start
        d.nw = nw;
        r.spawns = (int64_t)spawned;
        r.merged = merged;
        r.aborted = aborted;
        r.born = born;
        r.used = used;
        r.n_var = d.n_var;
        r.n_prev = d.n_prev;
        r.rec_max = (int64_t)a.rec_max[s];
        a.rec_max[s] = 0u;
        r.num = num;
        r.shift = d.shift;
        r.varying = d.varying;
        r.status = (int32_t)a.status[s];
        if (a.spilled[s]) {
            // new determinants wait in the spill list: pause until the host re-buckets
            a.status[s] |= ST_SPILLED;
            r.status = (int32_t)a.status[s];
            a.spilled[s] = 0u;
        }
        a.rec[(int64_t)s * REC_CAP + (done % REC_CAP)] = r;
        d.iter = done;
    }
}

static_assert(ACC_SLOTS <= 64 && SPAWN_SLOTS <= 64, "k_finalize sums one share per lane of a wavefront");
static_assert(POST_WAVES * 64 == 256, "one bucket of a chunk per wavefront of a k_post workgroup");

void launch_iteration(const EngineArgs &a, int post_grid, int spawn_grid, bool first,
                      hipStream_t s, hipEvent_t *ev) {
    if (ev) (void)hipEventRecord(ev[0], s);
    if (first)
        hipLaunchKernelGGL(k_tiles, dim3((unsigned)post_grid), dim3(256), 0, s, a,
                           (const SysDesc *)a.desc);
    if (ev) (void)hipEventRecord(ev[1], s);
    if (ev) (void)hipEventRecord(ev[2], s);
    if (a.plain)
        hipLaunchKernelGGL(k_spawn<true>, dim3((unsigned)spawn_grid), dim3(256), 0, s, a,
                           (const SysDesc *)a.desc, first ? 1 : 0);
    else
        hipLaunchKernelGGL(k_spawn<false>, dim3((unsigned)spawn_grid), dim3(256), 0, s, a,
                           (const SysDesc *)a.desc, first ? 1 : 0);
    if (ev) (void)hipEventRecord(ev[3], s);
    if (a.plain)
        hipLaunchKernelGGL(k_post<true>, dim3((unsigned)post_grid), dim3(256), 0, s, a,
                           (const SysDesc *)a.desc);
    else
        hipLaunchKernelGGL(k_post<false>, dim3((unsigned)post_grid), dim3(256), 0, s, a,
                           (const SysDesc *)a.desc);
    if (ev) (void)hipEventRecord(ev[4], s);
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)a.max_sys), dim3(64), 0, s, a);
    if (ev) (void)hipEventRecord(ev[5], s);
}

// ---------------------------------------------------------------------------
// Loading a walker list, re-bucketing into more (or fewer) buckets, exporting.
// ---------------------------------------------------------------------------
// Append determinant D (population p, diagonal element hd) to its bucket.
__device__ __forceinline__ bool bucket_put(const SysDesc &d, det_t D, int32_t p, double hd) {
    const uint32_t b = bucket_of(D, (uint64_t)d.nbuckets);
    const int pos = atomicAdd(&d.bcnt[b], 1);
    if (pos >= BQ) return false;
    const int64_t j = (int64_t)b * BQ + pos;
    keys_of(d)[j] = D;
    d.pop[j] = p;
    d.hdiag[j] = hd;
    return true;
}

// (add_ref: the reference is not among the entries and is put in without walkers)
__global__ void k_load(SysDesc *desc, int32_t sys, const det_t *det, const int32_t *pop,
                       int64_t n, int add_ref, uint32_t *err) {
    const SysDesc &d = desc[sys];
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n + add_ref;
         i += (int64_t)gridDim.x * blockDim.x) {
        const det_t D = i < n ? det[i] : ref_of(d);
        const int32_t p = i < n ? pop[i] : 0;
        if (p == 0 && i < n) continue;
        if (!bucket_put(d, D, p, fn_diag(d, D))) atomicOr(err, 1u);
    }
}

// What a walker list to be loaded into system sys holds: its sums, whether it ascends
// strictly without an empty entry, and the first entry that the system cannot hold (entry
// number * 8 + reason, LIST_*). Bound by the list's memory traffic.
__global__ __launch_bounds__(256) void k_check_list(const SysDesc *desc, int32_t sys,
                                                    const det_t *det, const int32_t *pop,
                                                    int64_t n, int na, int nb, ListCheck *out) {
    const SysDesc &d = desc[sys];
    const det_t ref = ref_of(d), valid = valid_of(d);
    unsigned long long bad = ~0ull;
    long long nw = 0;
    int nd = 0, unsorted = 0;
    uint32_t most = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = pop[i];
        if (p == 0) {
            unsorted = 1;
            continue;
        }
        const det_t D = det[i];
        if (i + 1 < n && !(D < det[i + 1])) unsorted = 1;
        int why = 0;
        if ((bool)(D & ~valid) || dpopc(D & even_bits()) != na || dpopc(D & odd_bits()) != nb)
            why = LIST_COUNTS;
        else if (p == INT32_MIN)
            why = LIST_RANGE;
        else if (!in_space(d, D))
            why = LIST_SPACE;
        else if (d.hphf) {
            const det_t f = spin_flip(D);
            if (f < D || (f == D && d.hphf < 0)) why = LIST_PAIR;
        }
        const unsigned long long at = (unsigned long long)i * 8ull + (unsigned long long)why;
        if (why && at < bad) bad = at;
        if (D == ref) {
            out->c0 = p;
            out->have_ref = 1;
        }
        const uint32_t q = p < 0 ? 0u - (uint32_t)p : (uint32_t)p;
        nw += q;
        nd++;
        most = q > most ? q : most;
    }
    nw = wave_sum(nw);
    const long long nds = wave_sum((long long)nd);
    for (int o = 32; o; o >>= 1) {
        const unsigned long long b = __shfl_xor(bad, o, 64);
        const uint32_t q = __shfl_xor(most, o, 64);
        bad = b < bad ? b : bad;
        most = q > most ? q : most;
    }
    const bool any = __ballot(unsorted) != 0;
    if ((threadIdx.x & 63) == 0) {
        if (nds) {
            atomicAdd(&out->nw, (unsigned long long)nw);
            atomicAdd(&out->nd, (unsigned long long)nds);
            atomicMax(&out->most, most);
        }
        if (bad != ~0ull) atomicMin(&out->bad, bad);
        if (any) atomicOr(&out->unsorted, 1);
    }
}

// Whether a sorted list holds two entries with walkers on one determinant (entries without
// walkers between them do not count).
__global__ __launch_bounds__(256) void k_twice(const det_t *det, const int32_t *pop, int64_t n,
                                               ListCheck *out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (pop[i] == 0) continue;
        for (int64_t j = i - 1; j >= 0 && det[j] == det[i]; --j)
            if (pop[j] != 0) {
                out->twice = 1;
                break;
            }
    }
}

__global__ void k_rebucket(SysDesc *desc, int32_t sys, const det_t *skey, const int32_t *spop,
                           const double *shd, const int32_t *scnt, int64_t snb,
                           const det_t *xdet, const int32_t *xpop, const double *xhd,
                           const int32_t *xsys, int64_t nx, uint32_t *err) {
    const SysDesc &d = desc[sys];
    const int64_t ns = snb * BQ;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns + nx;
         i += (int64_t)gridDim.x * blockDim.x) {
        det_t D;
        int32_t p;
        double hd;
        if (i < ns) {
            if ((int)(i % BQ) >= scnt[i / BQ]) continue;
            D = skey[i];
            p = spop[i];
            hd = shd[i];
        } else {
            const int64_t k = i - ns;
            if (xsys[k] != sys) continue;
            D = xdet[k];
            p = xpop[k];
            hd = xhd[k];
        }
        if (p == 0 && D != ref_of(d)) continue;
        if (!bucket_put(d, D, p, hd)) atomicOr(err, 1u);
    }
}

// Occupied entries (population != 0) of nb buckets, in any order, into odet/opop
// (at most `limit` written; *count gets the total, also with limit 0). A wavefront takes a
// whole chunk's 1024 slots, so that one counter atomic serves up to 1024 entries: all of them
// go to one address, which takes about 100 a microsecond (with one per 64 slots, the counter
// alone took 20 ms on a list of 8e7).
__global__ __launch_bounds__(256) void k_compact(const det_t *kv, const int32_t *pop,
                                                 const int32_t *cnt, int64_t nb, det_t *odet,
                                                 int32_t *opop, unsigned long long *count,
                                                 int64_t limit) {
    constexpr int R = CHUNK / 64;
    const int lane = threadIdx.x & 63;
    const int64_t nc = nb / BPC;   // (buckets come in whole chunks)
    for (int64_t c = blockIdx.x * 4ll + (threadIdx.x >> 6); c < nc; c += gridDim.x * 4ll) {
        const int64_t base = c * CHUNK;
        int32_t p[R];
        int total = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = base + r * 64 + lane;
            p[r] = (int)(i % BQ) < cnt[i / BQ] ? pop[i] : 0;
            total += __popcll(__ballot(p[r] != 0));
        }
        if (!total) continue;
        unsigned long long b = 0;
        if (lane == 0) b = atomicAdd(count, (unsigned long long)total);
        b = __shfl(b, 0, 64);
        if (b >= (unsigned long long)limit) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t m = __ballot(p[r] != 0);
            const unsigned long long j = b + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull));
            if (p[r] != 0 && j < (unsigned long long)limit) {
                odet[j] = kv[base + r * 64 + lane];
                opop[j] = p[r];
            }
            b += (unsigned long long)__popcll(m);
        }
    }
}

// ---------------------------------------------------------------------------
// Sorting a list by determinant: a least-significant-digit radix sort of (determinant,
// population) by 8-bit digits, three launches per digit. A wavefront owns SORT_RUN
// consecutive entries through all of them, so the passes need no workgroup barrier and are
// stable. Bound by memory: per digit every determinant is read twice and each entry
// written once, in runs as long as a digit's share of a wavefront's entries.
// Lanes of the same digit are found with eight ballots, not with LDS atomics: most
// determinants of a list agree in most digits (the electrons below the Fermi level), and
// 64 atomics on one counter are served one after another.
// ---------------------------------------------------------------------------
constexpr int SORT_RUN = 1024;

__device__ __forceinline__ uint32_t sort_digit(det_t D, int shift) {
    return (uint32_t)lo64(D >> shift) & 255u;
}
// Lanes of this wavefront with ok and the same digit.
__device__ __forceinline__ uint64_t same_digit(uint32_t g, bool ok) {
    uint64_t m = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t v = __ballot((g >> b) & 1u);
        m &= ((g >> b) & 1u) ? v : ~v;
    }
    return m;
}

// Occurrences of each digit in each run: hist[digit * nr + run].
__global__ __launch_bounds__(256) void k_sort_count(const det_t *key, int64_t n, int64_t nr,
                                                    int shift, uint32_t *hist) {
    __shared__ uint32_t s_n[4][256];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t run = blockIdx.x * 4ll + wid;
    if (run >= nr) return;   // (no barrier below: a wavefront uses its own counters only)
    for (int q = lane; q < 256; q += 64) s_n[wid][q] = 0u;
    wave_sync();
#pragma unroll 4
    for (int r = 0; r < SORT_RUN / 64; ++r) {
        const int64_t i = run * SORT_RUN + r * 64 + lane;
        const bool ok = i < n;
        const uint32_t g = ok ? sort_digit(key[i], shift) : 0u;
        const uint64_t m = same_digit(g, ok);
        if (ok && lane == __builtin_ctzll(m)) s_n[wid][g] += (uint32_t)__popcll(m);
        wave_sync();
    }
    for (int q = lane; q < 256; q += 64) hist[q * nr + run] = s_n[wid][q];
}

// One workgroup per digit: its counts become their running sum over the runs, its total
// goes to tot[digit].
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t *hist, int64_t nr, uint32_t *tot) {
    __shared__ uint32_t s_w[4];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    uint32_t *row = hist + (int64_t)blockIdx.x * nr;
    uint32_t carry = 0;
    for (int64_t b = 0; b < nr; b += 256) {
        const uint32_t v = b + t < nr ? row[b + t] : 0u;
        uint32_t x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) s_w[wid] = x;
        __syncthreads();
        uint32_t before = carry;
        for (int w = 0; w < wid; ++w) before += s_w[w];
        carry += s_w[0] + s_w[1] + s_w[2] + s_w[3];
        if (b + t < nr) row[b + t] = before + x - v;
        __syncthreads();
    }
    if (t == 0) tot[blockIdx.x] = carry;
}

// Every run's entries to their places.
__global__ __launch_bounds__(256) void k_sort_move(const det_t *key, const int32_t *val, int64_t n,
                                                   int64_t nr, int shift, const uint32_t *hist,
                                                   const uint32_t *tot, det_t *okey,
                                                   int32_t *oval) {
    __shared__ uint32_t s_at[4][256];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t run = blockIdx.x * 4ll + wid;
    if (run >= nr) return;
    uint32_t c[4], sum = 0;
    for (int q = 0; q < 4; ++q) sum += c[q] = tot[lane * 4 + q];
    uint32_t x = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    uint32_t at = x - sum;   // entries of smaller digits
    for (int q = 0; q < 4; ++q) {
        s_at[wid][lane * 4 + q] = at + hist[(lane * 4 + q) * nr + run];
        at += c[q];
    }
    wave_sync();
#pragma unroll 4
    for (int r = 0; r < SORT_RUN / 64; ++r) {
        const int64_t i = run * SORT_RUN + r * 64 + lane;
        const bool ok = i < n;
        const det_t D = ok ? key[i] : det_t(0ull);
        const int32_t p = ok ? val[i] : 0;
        const uint32_t g = sort_digit(D, shift);
        const uint64_t m = same_digit(g, ok);
        const uint32_t first = ok ? s_at[wid][g] : 0u;
        wave_sync();
        if (ok && lane == __builtin_ctzll(m)) s_at[wid][g] = first + (uint32_t)__popcll(m);
        wave_sync();
        const uint32_t j = first + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (ok) {
            okey[j] = D;
            oval[j] = p;
        }
    }
}

// Initiator flag of each of n entries: |pop| > n_a, or the reference.
__global__ void k_flags(const det_t *key, const int32_t *val, int64_t n, int32_t n_a, uint64_t d0,
                        uint64_t d0_hi, uint32_t *flags) {
    const det_t ref = make_det(d0, d0_hi);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = val[i] < 0 ? -(int64_t)val[i] : (int64_t)val[i];
        flags[i] = (a > (int64_t)n_a || key[i] == ref) ? 1u : 0u;
    }
}

hipError_t launch_flags(const uint64_t *key, const int32_t *val, int64_t n, int32_t n_a,
                        uint64_t d0, uint64_t d0_hi, uint32_t *flags, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_flags, dim3((unsigned)(g < 8192 ? g : 8192)), dim3(256), 0, s,
                       (const det_t *)key, val, n, n_a, d0, d0_hi, flags);
    return hipGetLastError();
}

hipError_t launch_sort(uint64_t *key, int32_t *val, uint64_t *key2, int32_t *val2, uint32_t *hist,
                       int64_t n, int passes, hipStream_t s) {
    if (n < 1 || n > SORT_MAX || passes < 1 || passes > 8 * FQ_DET_WORDS)
        return hipErrorInvalidValue;
    const int64_t nr = (n + SORT_RUN - 1) / SORT_RUN;
    uint32_t *tot = hist, *rows = hist + 256;
    det_t *a = (det_t *)key, *b = (det_t *)key2;
    const dim3 grid((unsigned)((nr + 3) / 4));
    for (int k = 0; k < passes; ++k) {
        hipLaunchKernelGGL(k_sort_count, grid, dim3(256), 0, s, (const det_t *)a, n, nr, 8 * k, rows);
        hipLaunchKernelGGL(k_sort_scan, dim3(256), dim3(256), 0, s, rows, nr, tot);
        hipLaunchKernelGGL(k_sort_move, grid, dim3(256), 0, s, (const det_t *)a,
                           (const int32_t *)val, n, nr, 8 * k, (const uint32_t *)rows,
                           (const uint32_t *)tot, b, val2);
        std::swap(a, b);
        std::swap(val, val2);
    }
    return hipGetLastError();
}

// Places for the records that crowded buckets get beyond their system's slots (once per
// launch, and only for systems that need it).
__global__ void k_extend(const uint32_t *bprev, uint64_t *bext, int64_t nb, uint32_t rec_r,
                         float factor, int64_t pool0, int64_t pool, unsigned long long *used) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nb;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float need = (float)bprev[i] * factor + 16.0f;
        uint64_t x = 0ull;
        if (need > (float)rec_r) {
            const float over = fminf(need - (float)rec_r, (float)((1 << EXT_BITS) - 64));
            const unsigned long long n = ((unsigned long long)over + 8ull) / 8ull * 8ull;
            const unsigned long long at = atomicAdd(used, n);
            if ((int64_t)(at + n) <= pool) x = (uint64_t)(pool0 + (int64_t)at) << EXT_BITS | n;
        }
        bext[i] = x;
    }
}

hipError_t launch_extend(const uint32_t *bprev, uint64_t *bext, int64_t nb, uint32_t rec_r,
                         float factor, int64_t pool0, int64_t pool, unsigned long long *used,
                         hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    const int64_t g = (nb + 255) / 256;
    hipLaunchKernelGGL(k_extend, dim3((unsigned)(g < 4096 ? g : 4096)), dim3(256), 0, s, bprev, bext,
                       nb, rec_r, factor, pool0, pool, used);
    return hipGetLastError();
}

hipError_t launch_load(SysDesc *d_desc, int32_t sys, const uint64_t *det, const int32_t *pop,
                       int64_t n, int add_ref, uint32_t *d_err, hipStream_t s) {
    if (n + add_ref <= 0) return hipSuccess;
    const int64_t g = (n + add_ref + 255) / 256;
    hipLaunchKernelGGL(k_load, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(256), 0, s, d_desc,
                       sys, (const det_t *)det, pop, n, add_ref, d_err);
    return hipGetLastError();
}

hipError_t launch_check_list(const SysDesc *desc, int32_t sys, const uint64_t *det,
                             const int32_t *pop, int64_t n, int na, int nb, ListCheck *out,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_check_list, dim3((unsigned)(g < 2048 ? g : 2048)), dim3(256), 0, s, desc,
                       sys, (const det_t *)det, pop, n, na, nb, out);
    return hipGetLastError();
}

hipError_t launch_twice(const uint64_t *det, const int32_t *pop, int64_t n, ListCheck *out,
                        hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_twice, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(256), 0, s,
                       (const det_t *)det, pop, n, out);
    return hipGetLastError();
}

hipError_t launch_rebucket(SysDesc *d_desc, int32_t sys, const uint64_t *src_key,
                           const int32_t *src_pop, const double *src_hd, const int32_t *src_cnt,
                           int64_t src_nb, const uint64_t *sp_det, const int32_t *sp_pop,
                           const double *sp_hd, const int32_t *sp_sys, int64_t n_sp,
                           uint32_t *d_err, hipStream_t s) {
    const int64_t g = (src_nb * BQ + n_sp + 255) / 256;
    if (g == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rebucket, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(256), 0, s,
                       d_desc, sys, (const det_t *)src_key, src_pop, src_hd, src_cnt, src_nb,
                       (const det_t *)sp_det, sp_pop, sp_hd, sp_sys, n_sp, d_err);
    return hipGetLastError();
}

hipError_t launch_compact(const uint64_t *key, const int32_t *pop, const int32_t *cnt, int64_t nb,
                          uint64_t *out_det, int32_t *out_pop, unsigned long long *count,
                          int64_t limit, hipStream_t s) {
    const int64_t g = (nb / BPC + 3) / 4;
    if (g == 0) return hipSuccess;
    hipLaunchKernelGGL(k_compact, dim3((unsigned)(g < 8192 ? g : 8192)), dim3(256), 0, s,
                       (const det_t *)key, pop, cnt, nb, (det_t *)out_det, out_pop, count, limit);
    return hipGetLastError();
}

#if FQ_DET_WORDS == 1
// ---------------------------------------------------------------------------
// Export through a fixed staging area (no allocation): the counter is cleared by
// a kernel (no memset node), the occupied slots are compacted with one counter
// atomic per wavefront, and the keys are sorted by a bitonic network over the
// next power of two (padding keys ~0 sort last).
// ---------------------------------------------------------------------------
__global__ void k_stage_clear(unsigned long long *count) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *count = 0ull;
}

__global__ void k_stage_pad(uint64_t *key, int64_t n, int64_t P) {
    for (int64_t i = n + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P;
         i += (int64_t)gridDim.x * blockDim.x)
        key[i] = ~0ull;
}

__global__ void k_stage_bitonic(uint64_t *key, int32_t *val, int64_t P, int64_t j, int64_t k) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t l = i ^ j;
        if (l <= i) continue;
        const bool up = (i & k) == 0;
        const uint64_t a = key[i], b = key[l];
        if ((a > b) == up) {
            key[i] = b;
            key[l] = a;
            const int32_t t = val[i];
            val[i] = val[l];
            val[l] = t;
        }
    }
}

hipError_t launch_stage_flags(void *stage, int64_t n, int32_t n_a, uint64_t d0, hipStream_t s) {
    char *p = (char *)stage;
    return launch_flags((const uint64_t *)(p + NOALLOC_KEYS_OFF),
                        (const int32_t *)(p + NOALLOC_VALS_OFF), n, n_a, d0, 0,
                        (uint32_t *)(p + NOALLOC_FLAGS_OFF), s);
}

hipError_t launch_stage_compact(const uint64_t *key, const int32_t *pop, const int32_t *cnt,
                                int64_t nb, void *stage, hipStream_t s) {
    char *p = (char *)stage;
    unsigned long long *count = (unsigned long long *)p;
    hipLaunchKernelGGL(k_stage_clear, dim3(1), dim3(64), 0, s, count);
    return launch_compact(key, pop, cnt, nb, (uint64_t *)(p + NOALLOC_KEYS_OFF),
                          (int32_t *)(p + NOALLOC_VALS_OFF), count, (int64_t)NOALLOC_MAX_DETS, s);
}

hipError_t launch_stage_sort(void *stage, int64_t n, hipStream_t s) {
    if (n > NOALLOC_MAX_DETS) return hipErrorInvalidValue;
    char *p = (char *)stage;
    uint64_t *key = (uint64_t *)(p + NOALLOC_KEYS_OFF);
    int32_t *val = (int32_t *)(p + NOALLOC_VALS_OFF);
    int64_t P = 1;
    while (P < n) P <<= 1;
    if (P < 2) return hipSuccess;
    const int64_t g = (P + 255) / 256;
    const unsigned grid = (unsigned)(g < 8192 ? g : 8192);
    hipLaunchKernelGGL(k_stage_pad, dim3(grid), dim3(256), 0, s, key, n, P);
    for (int64_t k = 2; k <= P; k <<= 1)
        for (int64_t j = k >> 1; j > 0; j >>= 1)
            hipLaunchKernelGGL(k_stage_bitonic, dim3(grid), dim3(256), 0, s, key, val, P, j, k);
    return hipGetLastError();
}

#endif   // the staging export (one-word determinants only)

__global__ void k_e0(const SysDesc *desc, int32_t sys, uint64_t lo, uint64_t hi, double *out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *out = fn_diag(desc[sys], make_det(lo, hi));
}

hipError_t launch_e0(const SysDesc *desc, int32_t sys, uint64_t lo, uint64_t hi, double *out,
                     hipStream_t s) {
    hipLaunchKernelGGL(k_e0, dim3(1), dim3(64), 0, s, desc, sys, lo, hi, out);
    return hipGetLastError();
}

#if FQ_DET_WORDS == 1

static int cu_count() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            cus = prop.multiProcessorCount;
    }
    return cus;
}
int post_grid_size() { return cu_count() * 4; }    // four workgroups per CU
// the spawning kernel's resident workgroups (five per CU; four with two words)
int spawn_grid_size(int W) { return cu_count() * (W == 1 ? 5 : 4); }
#endif

#if FQ_DET_WORDS == 2
}  // namespace w2
#endif
}  // namespace fq
