// bwfm: GPU side of the FM-index short-read alignment path and its C ABI.
//
// Method: Genetically Improved BarraCUDA, section 2 (backward search with an
// upper and a lower pointer per read, backtracking over alternatives for
// inexact reads, the whole index resident in GPU memory), with the search
// rules of the BWA short-read backtracking method that BarraCUDA derives
// from; locate and pairing as in "sampe" (sections 2 and 3.7).  The exact
// definitions are stated in include/bwfm.h.
//
// Layout.  Each direction of the index is an array of rank lines (64 or
// 128 bytes): four uint32 counts of A, C, G, T before the line ($ counted as
// A), then the line's BWT rows as bit planes -- per 32 rows a word of the
// codes' high bits and a word of their low bits -- so one rank query is one
// line fetch plus three popcounts per 32 rows.  Beside them, made at upload:
// the intervals of all strings of up to K bases, and the whole suffix array
// and its inverse; with the packed reference they let a search take the
// shallow part of its tree from one table entry a state, and the part below a
// string that occurs once from the text (build_search_tables).  Row-sampled
// suffix array values serve locate where these do not fit.
//
// Search.  One lane per read, both strands in turn, each strand 5' end
// first (strand +: reverse(read) on the index of reverse(T); strand -:
// revcomp(read) on the index of T).  Per strand the D-array lower bound is
// built on the other index, then a depth-first search runs
// whose current state lives in registers; the first surviving child becomes
// the next current state and its siblings go to a lane-private stack in
// device memory, so the common one-child step touches no stack; a shallow
// state's siblings are one entry there, and a run of exact matches is one
// step.  Children are
// taken in a fixed order (match, mismatches by base, insertion, deletions by
// base), and in BEST mode a state is dropped when its score plus the least
// cost of its remaining D[i] differences exceeds best + s_mm.  Distinct hits
// collect in a lane-private buffer.  Reads whose stack or hit buffer fills up
// are searched again in a second pass with buffers of the worst-case size.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "bwfm_internal.h"

using namespace bwfm;

namespace {

// 16- and 8-byte words as native vectors: a search state then lives in
// registers (HIP's vector classes kept the current state of the batched
// kernel in scratch memory, a store and a load every iteration: with these
// and as_global below 2M reads of 100 bases went from 99 to 77 ms).
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u4 mk4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return u4{x, y, z, w}; }
__device__ __forceinline__ u2 mk2(uint32_t x, uint32_t y) { return u2{x, y}; }

// ------------------------------------------------------------------ constants

constexpr int GAP_INS = 1, GAP_DEL = 2;  // gap state of a search state (0: not in a gap)
constexpr uint32_t ST_RESEARCH = 8;  // status bit: needed the second pass
constexpr int PH_FAST = 0, PH_BEST = 1, PH_COLLECT = 2;
constexpr int INF_SCORE = 0x7fffffff;
constexpr uint32_t PLAIN_STACK = 320;  // stack entries per lane, plain form first pass
// Tuning constants a variant build may override with -D (results do not
// depend on them; paper_1505_07855_amd/variants.py searches over them).
// First-pass hit slots per lane: 128 keeps reads with up to that many
// candidate hits, common on repeat-rich references, out of the second pass,
// at no cost on reads with few hits.
#ifndef BWFM_FAST_CAND
#define BWFM_FAST_CAND 128
#endif
#ifndef BWFM_POPS_PER_STEP
#define BWFM_POPS_PER_STEP 1
#endif
#ifndef BWFM_SLOW_LANES
#define BWFM_SLOW_LANES 16384
#endif
// Alternative implementations of single code sites ("genes"), chosen at
// compile time; every alternative computes the same results, only its cost
// differs.  0 is the shipped one.  paper_1505_07855_amd/variants.py
// searches over them.
//   ROWMASK:  row masks of a 32-row group by compare and select (0) or by
//             one 64-bit shift (1).
//   SUBHDR:   with SUBLOAD 0, a 128-byte sub-counted query reads the
//             boundary words only for rows past 128 (0) or always (1).
#ifndef BWFM_GENE_ROWMASK
#define BWFM_GENE_ROWMASK 0
#endif
#ifndef BWFM_GENE_SUBHDR
#define BWFM_GENE_SUBHDR 0
#endif
// Reads of this many bases and more are long: a batch of them has its few
// largest trees split early (DRAIN_EIGHTHS).
constexpr uint32_t LONG_READ = 200;
// Lanes of a wave that must wait for a strand or read change before the wave
// makes them (BWFM_TURN_MIN may override it).
#ifndef BWFM_TURN_MIN
#define BWFM_TURN_MIN 8
#endif
//   SUBLOAD:  a 128-byte sub-counted query loads the line's first 16 bytes
//             and, past row 128, its next 16 (0), or 12 bytes of counts and
//             the one boundary word its row needs (1, shipped: fewer
//             registers hold line data, 1.5% faster on the benchmark batch).
#ifndef BWFM_GENE_SUBLOAD
#define BWFM_GENE_SUBLOAD 1
#endif
constexpr uint32_t FAST_CAND = BWFM_FAST_CAND;  // hit slots per lane, first pass
constexpr int BLOCK = 256;
constexpr int POPS_PER_STEP = BWFM_POPS_PER_STEP;  // stack pops per lane per persistent iteration (more costs the
                                  // whole wave a pass of the pop code; measured best at 1)

struct Params {
    int max_diff, max_gapo, max_gape, seed_len, seed_diff, ies, s_mm, s_gapo, s_gape, mode, max_best;
    uint32_t max_hits;
    int minc, s1;
};

struct ReadsView {
    const uint8_t *bases;
    const uint64_t *off;
    const uint32_t *len;  // per-read lengths, or NULL: read r ends where read r + 1 starts
    const uint8_t *maxd;
    uint32_t n, max_len;
    const uint64_t *n_dev;  // or NULL; else the batch holds min(*n_dev, n) reads (set on the device)
};

// number of reads in the batch
__device__ __forceinline__ uint32_t reads_n(const ReadsView &rd) {
    return rd.n_dev ? (uint32_t)min(*rd.n_dev, (uint64_t)rd.n) : rd.n;
}

// a count known on the host (n) or, when n_dev is set, on the device (at most n)
__device__ __forceinline__ uint64_t count_of(uint64_t n, const uint64_t *n_dev) {
    return n_dev ? min(*n_dev, n) : n;
}

// A pointer known to be in device memory.  Pointers that a kernel loads from
// memory (its argument block) have no address space the compiler can see, so
// accesses through them become flat ones: these count as LDS accesses too,
// and every wait for an LDS read then waits for all of them.
// (The empty asm keeps the two casts from folding away.)
template <class T> __device__ __forceinline__ T *as_global(T *p) {
    auto g = (__attribute__((address_space(1))) T *)p;
    asm("" : "+v"(g));
    return (T *)g;
}

// start and length of read r
__device__ __forceinline__ void read_span(const ReadsView &rd, uint32_t r, uint64_t &o0, uint64_t &len, bool &bad) {
    const uint64_t *off = as_global(rd.off);
    o0 = off[r];
    if (rd.len) {
        len = as_global(rd.len)[r];
        bad = false;
    } else {
        const uint64_t o1 = off[r + 1];
        bad = o1 < o0;
        len = bad ? 0 : o1 - o0;
    }
}

// Lane-private buffers in device memory.  Element e of lane t sits at
// base[t * lane_step + e * stride]: interleaved (lane_step 1, stride = lanes)
// when a wave's lanes move in step, contiguous (lane_step = cap, stride 1)
// when they do not.  Each lane's strand pattern and D-array live in LDS,
// lds_stride bytes per lane.
struct LaneBufs {
    u4 *stack;
    u4 *cand;
    uint32_t stack_lane_step, stack_stride, stack_cap;
    uint32_t cand_lane_step, cand_stride, cand_cap;
    uint32_t lds_stride;
};

// ------------------------------------------------------------------ rank queries

// element b of a four-element register array without dynamic indexing
__device__ __forceinline__ uint32_t sel4(const uint32_t (&v)[4], int b) {
    return b == 0 ? v[0] : (b == 1 ? v[1] : (b == 2 ? v[2] : v[3]));
}

// direction 0 or 1 of the index without dynamic indexing into the argument
__device__ __forceinline__ DevDir pick_dir(const DevIndex &ix, int which) {
    DevDir d;
    d.lines = which ? ix.dir[1].lines : ix.dir[0].lines;
    d.sa = which ? ix.dir[1].sa : ix.dir[0].sa;
#pragma unroll
    for (int a = 0; a < 4; a++) d.C[a] = which ? ix.dir[1].C[a] : ix.dir[0].C[a];
    d.primary = which ? ix.dir[1].primary : ix.dir[0].primary;
    d.pad = 0;
    d.kt = which ? ix.dir[1].kt : ix.dir[0].kt;
    d.full = which ? ix.dir[1].full : ix.dir[0].full;
    return d;
}

__device__ __forceinline__ uint32_t line_of(const DevIndex &ix, uint32_t i) {
    return (uint32_t)__umul64hi((uint64_t)i, ix.magic);
}

// Rank-line format as a template tag: 8, 16 or 32 = lines of that many
// uint32 words with counts then bit planes; LW_SUB = 64-byte sub-counted
// lines of 160 rows (counts of C, G, T, then per base the counts at the
// first four 32-row boundaries as bytes, then the bit planes).
constexpr int LW_SUB = 17;
// LW_SUB128 = 128-byte sub-counted lines of 384 rows: counts of C, G, T
// before the line (words 0-2); the counts within the line before rows 64,
// 128, 192, 256 and 320, each as C | G << 9 | T << 18 (words 3-7); the bit
// planes (words 8-31), per 32 rows a word of high bits then one of low bits,
// so the four plane words of a 64-row group are one aligned 16-byte load.
// A rank query reads the line's first 16 bytes, its boundary word and one
// group: an L2 fill brings 128 bytes the query can use.
constexpr int LW_SUB128 = 33;
template <int LW> constexpr int line_words() { return LW == LW_SUB ? 16 : (LW == LW_SUB128 ? 32 : LW); }
constexpr uint32_t SUB128_ROWS = 384;

// The one-base extensions of a string, as the search takes them: per base a
// the interval (x, y) = (k, l), or (text position, SINGLE) for a string that
// occurs once and is followed in the text; bit a of mask: it occurs.
struct Kids {
    uint32_t x[4], y[4], mask;
};
// y of such a string: SINGLE0 and more, above every l (texts have the tables
// only below SINGLE0 bases): SINGLE0 + the code of the next NEXT bases to be
// prepended, the first in the lowest digit, or SINGLE where they are not known
constexpr uint32_t SINGLE = 0xffffffffu, SINGLE0 = 0xfffff800u;
constexpr int NEXT = 5;

// from the interval table's two 16-byte words (p: A and C, q: G and T); a
// string that does not occur has y = 0 (one that does has l >= 1, since row 0
// is the empty suffix's)
__device__ __forceinline__ void kt_pick(u4 p, u4 q, Kids &k) {
    k.x[0] = p.x;
    k.y[0] = p.y;
    k.x[1] = p.z;
    k.y[1] = p.w;
    k.x[2] = q.x;
    k.y[2] = q.y;
    k.x[3] = q.z;
    k.y[3] = q.w;
    k.mask = (p.y ? 1u : 0u) | (p.w ? 2u : 0u) | (q.y ? 4u : 0u) | (q.w ? 8u : 0u);
}
// first entry of level d <= 15, which fits 32 bits
__device__ __forceinline__ uint32_t kt_start32(int d) { return d == 0 ? 0u : ((1u << (2 * d)) + 8u) / 3u; }
// entry of the first child of the string of d < 15 bases with code c:
// level d + 1 starts at (4^(d+1) + 8) / 3, and every entry below level 16
// has an index under 2^32
__device__ __forceinline__ uint32_t kt_children(int d, uint32_t c) {
    return ((1u << (2 * d + 2)) + 8u) / 3u + 4u * c;
}

// Occ of all four bases at row i of a sub-counted line: the counts before
// the line, the count at the boundary of row i's 32-row group, and a count
// of bits in that one group.  A is what the rows leave ($ excluded).
__device__ __forceinline__ void occ4_sub(const DevIndex &ix, const DevDir &d, uint32_t i, uint32_t o[4]) {
    const uint32_t line = line_of(ix, i);
    const uint32_t r = i - line * 160u, g = r >> 5;
    const uint32_t *L = d.lines + (size_t)line * 16;
    const u4 h = *reinterpret_cast<const u4 *>(L);       // C, G, T before the line; C boundaries
    const u2 b = *reinterpret_cast<const u2 *>(L + 4);   // G, T boundaries
    const u2 w = *reinterpret_cast<const u2 *>(L + 6 + 2 * g);
    const uint32_t m = (1u << (r & 31)) - 1u;
    uint32_t cC = __popc(~w.x & w.y & m), cG = __popc(w.x & ~w.y & m), cT = __popc(w.x & w.y & m);
    if (g) {
        const uint32_t sh = 8 * (g - 1);
        cC += (h.w >> sh) & 255u;
        cG += (b.x >> sh) & 255u;
        cT += (b.y >> sh) & 255u;
    }
    o[1] = h.x + cC;
    o[2] = h.y + cG;
    o[3] = h.z + cT;
    o[0] = i - o[1] - o[2] - o[3] - (i > d.primary ? 1u : 0u);
}

// Occ of all four bases at row i from the pieces of its 128-byte
// sub-counted line: h = words 0-3 (C, G, T before the line, boundary word
// of row 64), b = words 4-7 (boundary words of rows 128 .. 320; read only
// when the row's group needs one of them), p = the four plane words of the
// row's 64-row group; r = i's row within the line.
__device__ __forceinline__ void sub128_count(u4 h, u4 b, u4 p, uint32_t r, uint32_t i, uint32_t primary,
                                             uint32_t o[4]) {
    const uint32_t g = r >> 6, t = r & 63;
    const uint32_t m0 = t >= 32 ? 0xffffffffu : (1u << t) - 1u;
    const uint32_t m1 = t > 32 ? (1u << (t - 32)) - 1u : 0u;
    // high plane set: G or T; low plane set: C or T; both: T
    const uint32_t cT = __popc(p.x & p.y & m0) + __popc(p.z & p.w & m1);
    const uint32_t cH = __popc(p.x & m0) + __popc(p.z & m1);
    const uint32_t cL = __popc(p.y & m0) + __popc(p.w & m1);
    const uint32_t bw = g == 0 ? 0u : (g == 1 ? h.w : (g == 2 ? b.x : (g == 3 ? b.y : (g == 4 ? b.z : b.w))));
    o[1] = h.x + (bw & 511u) + cL - cT;
    o[2] = h.y + ((bw >> 9) & 511u) + cH - cT;
    o[3] = h.z + (bw >> 18) + cT;
    o[0] = i - o[1] - o[2] - o[3] - (i > primary ? 1u : 0u);
}

// The same count from the counts before the line (C, G, T), the row's
// boundary word (0 for the first 64 rows) and its group's plane words.
__device__ __forceinline__ void sub128_count3(uint3 h, uint32_t bw, u4 p, uint32_t r, uint32_t i,
                                              uint32_t primary, uint32_t o[4]) {
    const uint32_t t = r & 63;
    const uint32_t m0 = t >= 32 ? 0xffffffffu : (1u << t) - 1u;
    const uint32_t m1 = t > 32 ? (1u << (t - 32)) - 1u : 0u;
    const uint32_t cT = __popc(p.x & p.y & m0) + __popc(p.z & p.w & m1);
    const uint32_t cH = __popc(p.x & m0) + __popc(p.z & m1);
    const uint32_t cL = __popc(p.y & m0) + __popc(p.w & m1);
    o[1] = h.x + (bw & 511u) + cL - cT;
    o[2] = h.y + ((bw >> 9) & 511u) + cH - cT;
    o[3] = h.z + (bw >> 18) + cT;
    o[0] = i - o[1] - o[2] - o[3] - (i > primary ? 1u : 0u);
}

// One row's pieces of its line: counts, boundary word, group planes.
__device__ __forceinline__ void sub128_load(const uint32_t *L, uint32_t r, uint3 &h, uint32_t &bw, u4 &p) {
    h = *reinterpret_cast<const uint3 *>(L);
    const uint32_t g = r >> 6;
    bw = 0;
    if (g) bw = L[2 + g];
    p = reinterpret_cast<const u4 *>(L)[2 + g];
}

__device__ __forceinline__ void occ4_sub128(const DevIndex &ix, const DevDir &d, uint32_t i, uint32_t o[4]) {
#if BWFM_GENE_SUBLOAD == 1
    {
        const uint32_t line = line_of(ix, i);
        const uint32_t r = i - line * SUB128_ROWS;
        uint3 h;
        uint32_t bw;
        u4 p;
        sub128_load(d.lines + (size_t)line * 32, r, h, bw, p);
        sub128_count3(h, bw, p, r, i, d.primary, o);
        return;
    }
#endif
    const uint32_t line = line_of(ix, i);
    const uint32_t r = i - line * SUB128_ROWS;
    const u4 *L = reinterpret_cast<const u4 *>(d.lines) + (size_t)line * 8;
    const u4 h = L[0];
    u4 b = mk4(0, 0, 0, 0);
    if (BWFM_GENE_SUBHDR == 1 || r >= 128) b = L[1];
    const u4 p = L[2 + (r >> 6)];
    sub128_count(h, b, p, r, i, d.primary, o);
}

// Occ at rows i1 and i2 (k and l + 1 of an interval) on 128-byte
// sub-counted lines: the shared parts of one line are read once.
__device__ __forceinline__ void occ4_sub128_pair(const DevIndex &ix, const DevDir &d, uint32_t i1, uint32_t i2,
                                                 uint32_t o1[4], uint32_t o2[4]) {
#if BWFM_GENE_SUBLOAD == 1
    {
        const uint32_t l1 = line_of(ix, i1), l2 = line_of(ix, i2);
        const uint32_t r1 = i1 - l1 * SUB128_ROWS, r2 = i2 - l2 * SUB128_ROWS;
        uint3 h1, h2;
        uint32_t b1, b2;
        u4 p1, p2;
        sub128_load(d.lines + (size_t)l1 * 32, r1, h1, b1, p1);
        if (l1 != l2 || (r1 >> 6) != (r2 >> 6)) {
            sub128_load(d.lines + (size_t)l2 * 32, r2, h2, b2, p2);
        } else {
            h2 = h1;
            b2 = b1;
            p2 = p1;
        }
        sub128_count3(h1, b1, p1, r1, i1, d.primary, o1);
        sub128_count3(h2, b2, p2, r2, i2, d.primary, o2);
        return;
    }
#endif
    const uint32_t l1 = line_of(ix, i1), l2 = line_of(ix, i2);
    const uint32_t r1 = i1 - l1 * SUB128_ROWS, r2 = i2 - l2 * SUB128_ROWS;
    const u4 *L1 = reinterpret_cast<const u4 *>(d.lines) + (size_t)l1 * 8;
    const u4 *L2 = reinterpret_cast<const u4 *>(d.lines) + (size_t)l2 * 8;
    const bool same = l1 == l2;
    const u4 h1 = L1[0];
    u4 b1 = mk4(0, 0, 0, 0), h2 = h1, b2 = b1;
    if (BWFM_GENE_SUBHDR == 1 || r1 >= 128 || (same && r2 >= 128)) b1 = L1[1];
    const u4 p1 = L1[2 + (r1 >> 6)];
    if (!same) {
        h2 = L2[0];
        if (BWFM_GENE_SUBHDR == 1 || r2 >= 128) b2 = L2[1];
    } else {
        b2 = b1;
    }
    u4 p2 = p1;
    if (!same || (r1 >> 6) != (r2 >> 6)) p2 = L2[2 + (r2 >> 6)];
    sub128_count(h1, b1, p1, r1, i1, d.primary, o1);
    sub128_count(h2, b2, p2, r2, i2, d.primary, o2);
}

// mask of the first t rows of a 32-row group (t may be <= 0 or >= 32)
__device__ __forceinline__ uint32_t rows_mask(int t) {
#if BWFM_GENE_ROWMASK == 1
    // the low t bits of a 64-bit all-ones word shifted right by 64 - t,
    // clamped to [0, 32] rows
    const int c = t < 0 ? 0 : (t > 32 ? 32 : t);
    return (uint32_t)(c == 0 ? 0ull : (~0ull >> (64 - c)));
#else
    return t >= 32 ? 0xffffffffu : (t <= 0 ? 0u : ((1u << t) - 1u));
#endif
}

// Occ(a, i) for all four bases (i <= n + 1).  Per 32-row group: one word of
// high bits (h) and one of low bits (l); T = h & l, G = h & ~l, C = ~h & l.
template <int LW>
__device__ __forceinline__ void occ4(const DevIndex &ix, const DevDir &d, uint32_t i, uint32_t o[4]) {
    if constexpr (LW == LW_SUB) {
        occ4_sub(ix, d, i, o);
        return;
    }
    if constexpr (LW == LW_SUB128) {
        occ4_sub128(ix, d, i, o);
        return;
    }
    uint32_t line = line_of(ix, i);
    int r = (int)(i - line * ix.bpl);
    const u4 *L = reinterpret_cast<const u4 *>(d.lines) + (size_t)line * (LW / 4);
    u4 h = L[0];
    uint32_t cC = 0, cG = 0, cT = 0;
#pragma unroll
    for (int q = 0; q < LW / 4 - 1; q++) {
        u4 v = L[1 + q];
        uint32_t m0 = rows_mask(r - q * 64), m1 = rows_mask(r - q * 64 - 32);
        cT += __popc(v.x & v.y & m0) + __popc(v.z & v.w & m1);
        cG += __popc(v.x & ~v.y & m0) + __popc(v.z & ~v.w & m1);
        cC += __popc(~v.x & v.y & m0) + __popc(~v.z & v.w & m1);
    }
    uint32_t cA = (uint32_t)r - cC - cG - cT;
    o[0] = h.x + cA - (i > d.primary ? 1u : 0u);
    o[1] = h.y + cC;
    o[2] = h.z + cG;
    o[3] = h.w + cT;
}

// A string's four extensions from the rank counts at its k (i1) and l + 1
// (i2).  On 128-byte sub-counted lines the two rows share what one line gives
// both; on the others they are counted one after the other, since holding two
// whole lines made the 4-wave build of the batched kernel spill (up to 81
// registers; rank queries are the rarer step now that short strings come from
// the table and unique ones from the text).
template <int LW>
__device__ __forceinline__ void rank_children(const DevIndex &ix, const DevDir &d, uint32_t i1, uint32_t i2, Kids &k) {
    uint32_t lo[4], hi[4];
    if constexpr (LW == LW_SUB128) {
        occ4_sub128_pair(ix, d, i1, i2, lo, hi);
    } else {
        occ4<LW>(ix, d, i1, lo);
        occ4<LW>(ix, d, i2, hi);
    }
    k.mask = 0;
#pragma unroll
    for (int a = 0; a < 4; a++) {
        k.x[a] = lo[a] + d.C[a];
        k.y[a] = hi[a] + d.C[a] - 1;
        k.mask |= lo[a] < hi[a] ? 1u << a : 0u;
    }
}

// Occ(a, i) for one base a.
template <int LW>
__device__ __forceinline__ uint32_t occ1(const DevIndex &ix, const DevDir &d, int a, uint32_t i) {
    if constexpr (LW == LW_SUB || LW == LW_SUB128) {
        uint32_t o[4];
        occ4<LW>(ix, d, i, o);
        return sel4(o, a);
    }
    uint32_t line = line_of(ix, i);
    int r = (int)(i - line * ix.bpl);
    const u4 *L = reinterpret_cast<const u4 *>(d.lines) + (size_t)line * (LW / 4);
    u4 h = L[0];
    // rows of base a have high bit (a >> 1) and low bit (a & 1)
    const uint32_t fh = (a & 2) ? 0u : 0xffffffffu, fl = (a & 1) ? 0u : 0xffffffffu;
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < LW / 4 - 1; q++) {
        u4 v = L[1 + q];
        c += __popc((v.x ^ fh) & (v.y ^ fl) & rows_mask(r - q * 64));
        c += __popc((v.z ^ fh) & (v.w ^ fl) & rows_mask(r - q * 64 - 32));
    }
    uint32_t base = a == 0 ? h.x : (a == 1 ? h.y : (a == 2 ? h.z : h.w));
    return base + c - ((a == 0 && i > d.primary) ? 1u : 0u);
}

// BWT symbol at row j (j != primary) and Occ(that symbol, j): one line.
template <int LW>
__device__ __forceinline__ uint32_t lf_step(const DevIndex &ix, const DevDir &d, uint32_t j) {
    if constexpr (LW == LW_SUB128) {
        const uint32_t line = line_of(ix, j);
        const uint32_t r = j - line * SUB128_ROWS;
        const u4 *L = reinterpret_cast<const u4 *>(d.lines) + (size_t)line * 8;
        const u4 h = L[0];
        u4 b = mk4(0, 0, 0, 0);
        if (r >= 128) b = L[1];
        const u4 p = L[2 + (r >> 6)];
        const uint32_t hi = (r & 32) ? p.z : p.x, lo = (r & 32) ? p.w : p.y, s = r & 31;
        const int a = (int)((((hi >> s) & 1u) << 1) | ((lo >> s) & 1u));
        uint32_t o[4];
        sub128_count(h, b, p, r, j, d.primary, o);
        return sel4(d.C, a) + sel4(o, a);
    }
    uint32_t line = line_of(ix, j);
    uint32_t r = j - line * ix.bpl;
    const uint32_t *L = d.lines + (size_t)line * line_words<LW>();
    constexpr int po = LW == LW_SUB ? 6 : 4;  // first word of the bit planes
    int a = (int)((((L[po + 2 * (r >> 5)] >> (r & 31)) & 1) << 1) | ((L[po + 1 + 2 * (r >> 5)] >> (r & 31)) & 1));
    return sel4(d.C, a) + occ1<LW>(ix, d, a, j);
}

// ------------------------------------------------------------------ search state

// Search states are packed in 16 bytes: x = k (or, while |X| is below the
// index's short-string levels, the code of X: see state_k), y = l,
// z = (i + 1) | gap state << 10 | n_mm << 12 | n_gapo << 16 | n_gape << 20 | seed diffs << 24 | family << 28,
// w = score | |X| << 10 | lb << 20, where lb = score + minc * D[i] is the
// state's lower bound on its final score, fixed once the D-array is built.
// Every field fits: diffs <= 15, score <= 15 * 63, |X| <= 512 + 15.
__device__ __forceinline__ int entry_lb(u4 v) { return (int)(v.w >> 20); }

// hit record, same bytes as bwfm_hit
__device__ __forceinline__ u4 make_hit(int strand, uint32_t k, uint32_t l, int len, int score, int nmm, int ngo,
                                          int nge) {
    return mk4(k, l, (uint32_t)len | ((uint32_t)score << 16),
                      (uint32_t)strand | ((uint32_t)nmm << 8) | ((uint32_t)ngo << 16) | ((uint32_t)nge << 24));
}
__device__ __forceinline__ int h_strand(u4 h) { return h.w & 255; }
__device__ __forceinline__ int h_score(u4 h) { return h.z >> 16; }
__device__ __forceinline__ int h_len(u4 h) { return h.z & 0xffff; }
__device__ __forceinline__ int h_nmm(u4 h) { return (h.w >> 8) & 255; }
__device__ __forceinline__ int h_ngo(u4 h) { return (h.w >> 16) & 255; }
__device__ __forceinline__ int h_nge(u4 h) { return (h.w >> 24) & 255; }
__device__ __forceinline__ int h_diffs(u4 h) { return h_nmm(h) + h_ngo(h) + h_nge(h); }

// (score, diffs, n_gapo, n_mm) of a is smaller than b's
__device__ __forceinline__ bool better(u4 a, u4 b) {
    if (h_score(a) != h_score(b)) return h_score(a) < h_score(b);
    if (h_diffs(a) != h_diffs(b)) return h_diffs(a) < h_diffs(b);
    if (h_ngo(a) != h_ngo(b)) return h_ngo(a) < h_ngo(b);
    return h_nmm(a) < h_nmm(b);
}

// report order (score, strand, k, len)
__device__ __forceinline__ bool before(u4 a, u4 b) {
    if (h_score(a) != h_score(b)) return h_score(a) < h_score(b);
    if (h_strand(a) != h_strand(b)) return h_strand(a) < h_strand(b);
    if (a.x != b.x) return a.x < b.x;
    return h_len(a) < h_len(b);
}

struct LaneCtx {
    u4 *stack, *cand;
    uint8_t *pd;  // LDS, per pattern position i: base code | D[i] << 3
    uint32_t sstride, cstride, stack_cap, cand_cap;
    uint32_t sp, sbase;  // stack entries [sbase, sp) are this lane's pending states
    uint32_t ncand;
    int best;
    uint32_t expand;
};

extern __shared__ __align__(16) uint8_t lds_bytes[];

__device__ __forceinline__ void init_ctx(LaneCtx &c, const LaneBufs &B, uint32_t lane) {
    c.stack = as_global(B.stack + (size_t)lane * B.stack_lane_step);
    c.cand = as_global(B.cand + (size_t)lane * B.cand_lane_step);
    c.pd = lds_bytes + (size_t)threadIdx.x * B.lds_stride;
    c.sstride = B.stack_stride;
    c.cstride = B.cand_stride;
    c.stack_cap = B.stack_cap;
    c.cand_cap = B.cand_cap;
    c.sp = 0;
    c.sbase = 0;
    c.ncand = 0;
    c.best = INF_SCORE;
    c.expand = 0;
}

__device__ __forceinline__ int pd_base(const LaneCtx &c, int i) { return c.pd[i] & 7; }
__device__ __forceinline__ int pd_d(const LaneCtx &c, int i) { return i >= 0 ? (c.pd[i] >> 3) : 0; }

enum { R_OK = 0, R_STACK = 1, R_CAND = 2 };

// Insert a hit: merge with an equal (strand, k, len), else append.  In the
// first pass a full buffer is first cleared of hits above best + s_mm.
__device__ int record(LaneCtx &c, const Params &P, u4 h, int phase) {
    if (phase == PH_BEST) return R_OK;
    for (uint32_t j = 0; j < c.ncand; j++) {
        u4 o = c.cand[(size_t)j * c.cstride];
        if (h_strand(o) == h_strand(h) && o.x == h.x && h_len(o) == h_len(h)) {
            if (better(h, o)) c.cand[(size_t)j * c.cstride] = h;
            return R_OK;
        }
    }
    if (c.ncand == c.cand_cap && phase == PH_FAST && P.mode == BWFM_MODE_BEST) {
        uint32_t w = 0;
        for (uint32_t j = 0; j < c.ncand; j++) {
            u4 o = c.cand[(size_t)j * c.cstride];
            if (h_score(o) <= c.best + P.s_mm) c.cand[(size_t)(w++) * c.cstride] = o;
        }
        c.ncand = w;
    }
    if (c.ncand == c.cand_cap) return R_CAND;
    c.cand[(size_t)(c.ncand++) * c.cstride] = h;
    return R_OK;
}

// Copy read W (m bases) into an LDS row reversed, row[i] = W[m - 1 - i]:
// the strand + pattern, whose D-array scan then rewrites each byte in place
// as base | D << 3 (strand -: the complement of the same low bits).  Whole
// aligned dwords are loaded 8 at a time, so a read costs a few memory round
// trips instead of one per D-array step; only dwords holding read bases are
// touched.  Returns whether the read holds an N.
__device__ __forceinline__ bool stage_read(uint8_t *row, const uint8_t *W, int m) {
    const uint32_t *A = as_global(reinterpret_cast<const uint32_t *>(reinterpret_cast<uintptr_t>(W) & ~uintptr_t(3)));
    const int off = (int)(reinterpret_cast<uintptr_t>(W) & 3);
    const int ndw = (off + m + 3) >> 2;
    uint32_t n_any = 0;
    for (int k0 = 0; k0 < ndw; k0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = k0 + j < ndw ? A[k0 + j] : 0u;
#pragma unroll
        for (int j = 0; j < 8; j++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int i = 4 * (k0 + j) + q - off;
                if (i >= 0 && i < m) {
                    row[m - 1 - i] = (uint8_t)(v[j] >> (8 * q));
                    n_any |= (v[j] >> (8 * q)) & 4u;
                }
            }
    }
    return n_any != 0;
}

// seed window of the strand pattern: the read's 5' end, consumed first
struct Seed {
    int sl, lo, hi;
};
__device__ __forceinline__ Seed seed_of(const Params &P, int m) {
    Seed s;
    s.sl = P.seed_len > 0 ? (P.seed_len < m ? P.seed_len : m) : 0;
    s.lo = m - s.sl;
    s.hi = s.sl ? m : 0;
    return s;
}

// fields of a packed state (see pack)
__device__ __forceinline__ int s_i(u4 s) { return (int)(s.z & 1023) - 1; }
__device__ __forceinline__ int s_gs(u4 s) { return (s.z >> 10) & 3; }
__device__ __forceinline__ int s_nmm(u4 s) { return (s.z >> 12) & 15; }
__device__ __forceinline__ int s_ngo(u4 s) { return (s.z >> 16) & 15; }
__device__ __forceinline__ int s_nge(u4 s) { return (s.z >> 20) & 15; }
__device__ __forceinline__ int s_sd(u4 s) { return (s.z >> 24) & 15; }
__device__ __forceinline__ int s_score(u4 s) { return s.w & 1023; }
__device__ __forceinline__ int s_len(u4 s) { return (s.w >> 10) & 1023; }

// Interval of a completed state: (x, y) itself; while X is shorter than the
// interval table's levels (x holds the code of X), X's table entry on the
// strand's search index; for a string that occurs once (x its position in
// that direction's text), the row of the suffix there.
__device__ __forceinline__ u2 state_kl(const DevIndex &ix, int strand, u4 s) {
    const int len = s_len(s);
    if (len < (int)ix.kt_levels) {
        const u2 *kt = reinterpret_cast<const u2 *>(strand == 0 ? ix.dir[1].kt : ix.dir[0].kt);
        return kt[kt_start32(len) + s.x];
    }
    if (ix.kt_levels && s.y >= SINGLE0) {
        const uint32_t *isa = (strand == 0 ? ix.dir[1].full : ix.dir[0].full) + (size_t)ix.n + 1;
        const uint32_t k = isa[s.x];
        return mk2(k, k);
    }
    return mk2(s.x, s.y);
}

// ---- runs of exact matches through the interval table
//
// Most states of a search may take no further difference: the next one
// would pass the budget, the bound or the seed's.  Such a state only follows
// the pattern until its string stops occurring, which for strings shorter
// than the table's levels one table entry decides: the entry of the whole
// run at the deepest level holds its interval, or how many of its bases
// occur.  On the benchmark batch three quarters of the expansions are steps
// of such runs, 4 of them to a run.

// Two bits per base of row[at, at + q), q <= 20, base j in bits 2 j: the row
// is read as whole dwords (it starts dword-aligned; at most 3 bytes past its
// last base are touched, inside the row's last dword).
template <int ND = 5>  // dwords read: 5 for q <= 17, 6 for q <= 20
__device__ __forceinline__ uint64_t row_code(const uint8_t *row, int at, int q) {
    const uint32_t *A = reinterpret_cast<const uint32_t *>(row) + (at >> 2);
    const int sh = at & 3, nd = (sh + q + 3) >> 2;
    uint32_t v[ND];
#pragma unroll
    for (int t = 0; t < ND; t++) v[t] = t < nd ? A[t] : 0u;
    uint64_t w = 0;
#pragma unroll
    for (int t = 0; t < ND; t++) {
        uint32_t u = v[t] & 0x03030303u;
        u |= u >> 6;
        w |= (uint64_t)((u & 0x0fu) | ((u >> 12) & 0xf0u)) << (8 * t);
    }
    return (w >> (2 * sh)) & ((1ull << (2 * q)) - 1ull);
}
// sixteen two-bit digits in the opposite order
__device__ __forceinline__ uint32_t rev16(uint32_t c) {
    const uint32_t r = __brev(c);
    return ((r >> 1) & 0x55555555u) | ((r & 0x55555555u) << 1);
}
// the q <= 15 two-bit digits of c in the opposite order
__device__ __forceinline__ uint32_t rev_digits(uint32_t c, int q) { return q ? rev16(c) >> (32 - 2 * q) : 0u; }

// The children of a state shorter than the table's levels that are not taken
// at once are one stack entry, its family: the state itself with the family
// field set, in y the children left (bits 0-3 mismatch by base, bit 4 the
// insertion, bits 8-11 deletion by base), lb their lowest.
constexpr uint32_t FAMILY = 1u << 28;
constexpr uint32_t FAM_MM = 15u, FAM_INS = 16u, FAM_DEL = 15u << 8;

// Steps of the exact run from state cur (i >= 0, |X| at most the table's
// levels) to the deepest level, or 0 when a difference may still be taken on
// the way: D falls towards the pattern's start, so no difference fits
// anywhere in the run when none fits with the D of its end.
__device__ __forceinline__ int run_steps(const DevIndex &ix, u4 cur, const uint8_t *pd, int maxd, int bound,
                                         bool has_n, const Seed &S, const Params &P) {
    const int q = (int)ix.kt_levels - s_len(cur);
    const int e = s_i(cur) - q;
    if (e < -1) return 0;
    const int De = e >= 0 ? pd[e] >> 3 : 0;
    const int diffs = s_nmm(cur) + s_ngo(cur) + s_nge(cur);
    const bool none = diffs + 1 + De > maxd || s_score(cur) + P.minc + P.minc * De > bound ||
                      (S.sl != 0 && !has_n && s_sd(cur) >= P.seed_diff && e + 1 >= S.lo);
    return none ? q : 0;
}

// cur, t matches on: x and y are the caller's
__device__ __forceinline__ void step_matches(u4 &cur, int t, const uint8_t *pd, const Params &P) {
    const int e = s_i(cur) - t;
    const int De = e >= 0 ? pd[e] >> 3 : 0;
    if (t) cur.z &= ~(3u << 10);
    cur.z -= (uint32_t)t;
    cur.w = (cur.w & 0xfffffu) + ((uint32_t)t << 10);
    cur.w |= (uint32_t)(s_score(cur) + P.minc * De) << 20;
}

// ---- strings that occur once
//
// The deepest level's entry of a string that occurs once holds its position
// p in the direction's text (y = SINGLE).  Its extensions are then read from
// the packed reference: sixteen bases in one load, the same line for the
// whole read, where the rank lines took a random line fill per base.  The
// row of a completed hit comes from the inverse suffix array.

// two words at any word boundary
typedef uint32_t u2w __attribute__((ext_vector_type(2), aligned(4)));
// first of the two words of the packed reference holding the 16 bases next to
// be prepended at position p > 0 of direction dir's text: T[p - 16, p), or,
// for reverse(T), T[n - p, n - p + 16) (the copy has a word of padding)
__device__ __forceinline__ uint32_t text_word(const DevIndex &ix, int dir, uint32_t p) {
    return dir == 0 ? (p >= 16 ? (p - 16) >> 4 : 0u) : (ix.n - p) >> 4;
}
// those bases from the two words: T[p - 1], T[p - 2], ... from the highest
// digit down (dir 0), or T[n - p], T[n - p + 1], ... from the lowest up (dir
// 1); digits past the text's end are arbitrary
__device__ __forceinline__ uint32_t text_bases(const DevIndex &ix, int dir, uint32_t p, uint32_t w0, uint32_t w1) {
    if (dir == 0) {
        const bool head = p < 16;
        return __builtin_amdgcn_alignbit(head ? w0 : w1, head ? 0u : w0, 2 * (p & 15));
    }
    return __builtin_amdgcn_alignbit(w1, w0, 2 * ((ix.n - p) & 15));
}

// One step of a state whose string occurs once at p, win its next bases from
// the highest digit down, pc the r <= 16 pattern bases it meets (r = 0: one
// base at a time).  A run of matches is taken at once: its
// positions have no mismatch children, and their gaps, where one may still
// open, go on the stack as one run entry (gap state GAP_RUN, y = the run's
// length, x, i and the rest as at its start, lb that of its cheapest gap),
// which is dropped whole once the bound passes it.  Returns true when the run
// was taken; else k receives the one child.
constexpr int GAP_RUN = 3;
__device__ __forceinline__ bool text_step(u4 &cur, uint32_t win, uint32_t pc, int r, int maxd, int bound,
                                          const Params &P, LaneCtx &c, Kids &k) {
    const int i = s_i(cur);
    const uint32_t p = cur.x;
    if (r) {
        const uint32_t df = win ^ (pc << (32 - 2 * r));
        int t = df ? __clz(df) >> 1 : 16;
        t = min(t, r);
        t = (int)min((uint32_t)t, p);
        if (t) {
            const int e = i - t;
            const int De = e >= 0 ? c.pd[e] >> 3 : 0;
            const int ngo = s_ngo(cur), lbg = s_score(cur) + P.s_gapo + P.minc * De;
            const bool gap = ngo < P.max_gapo && s_nmm(cur) + ngo + s_nge(cur) + 1 + De <= maxd && lbg <= bound;
            if (!gap || c.sp + 8 <= c.stack_cap) {
                if (gap) {
                    c.stack[(size_t)c.sp * c.sstride] = mk4(p, (uint32_t)t, cur.z | ((uint32_t)GAP_RUN << 10),
                                                            (cur.w & 0xfffffu) | ((uint32_t)lbg << 20));
                    c.sp++;
                }
                step_matches(cur, t, c.pd, P);
                cur.x = p - (uint32_t)t;
                c.expand += (uint32_t)t;
                return true;
            }
        }
    }
    const uint32_t a = win >> 30;
    k.mask = p ? 1u << a : 0u;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        k.x[q] = p - 1;
        k.y[q] = SINGLE;
    }
    c.expand++;
    return false;
}

// A run entry taken from the stack: its deepest position's gaps come next (k
// holds the deletion's child, cur the state there; the caller takes gaps
// only), the rest of the run goes back on the stack.
__device__ __forceinline__ void unroll_run(u4 &cur, const Params &P, LaneCtx &c, Kids &k) {
    const int t = (int)cur.y, i = s_i(cur);
    const int lb0 = s_score(cur) + P.s_gapo;
    const int j = i - t + 1;  // the position taken now
    if (t > 1) {
        const int De = c.pd[j] >> 3;  // the rest ends one position before j
        c.stack[(size_t)c.sp * c.sstride] =
            mk4(cur.x, (uint32_t)(t - 1), cur.z, (cur.w & 0xfffffu) | ((uint32_t)(lb0 + P.minc * De) << 20));
        c.sp++;
    }
    cur.x -= (uint32_t)(t - 1);
    cur.y = SINGLE;
    cur.z = (cur.z & ~(3u << 10)) - (uint32_t)(t - 1);
    cur.w = (cur.w & 0xfffffu) + ((uint32_t)(t - 1) << 10);
    k.mask = 1u << (c.pd[j] & 3);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        k.x[q] = cur.x - 1;
        k.y[q] = SINGLE;
    }
}

// Whether a state with one row left (k = l, |X| = len) is better followed in
// the text: past the table's depth by a few bases it is mostly the read's own
// place, while most states that get there by chance are gone.
__device__ __forceinline__ bool to_text(const DevIndex &ix, u4 cur) {
    return cur.x == cur.y && ix.kt_levels && s_len(cur) >= (int)ix.kt_levels + 3;
}

// the empty string's interval, nothing consumed, lower bound minc * D[m - 1]
__device__ __forceinline__ u4 root_state(const DevIndex &ix, int m, int lb) {
    return mk4(0u, ix.n, (uint32_t)m, (uint32_t)lb << 20);
}

// Advance the search until the current state needs expanding: pop, drop
// states whose stored lower bound exceeds the BEST bound, record completed
// hits.  At most max_pops entries are popped.  Returns 1 when cur must be
// expanded, 0 when the lane's part of the strand's search is over, 2 when
// the pop limit was reached first, 3 when cur is a completed hit left for
// the caller to record (only with defer), or -R_CAND when the hit buffer
// overflowed.
__device__ int resolve(u4 &cur, bool &valid, int strand, const Params &P, LaneCtx &c, int phase, int max_pops,
                       const DevIndex &ix, bool defer = false) {
    for (int pops = 0;;) {
        const int bound = (P.mode == BWFM_MODE_BEST && c.best != INF_SCORE) ? c.best + P.s_mm : INF_SCORE;
        if (!valid) {
            if (c.sp == c.sbase) return 0;
            if (pops == max_pops) return 2;
            pops++;
            c.sp--;
            cur = c.stack[(size_t)c.sp * c.sstride];
            valid = true;
        }
        if (entry_lb(cur) > bound) {
            valid = false;
            continue;
        }
        if (s_i(cur) < 0) {
            if (defer) return 3;
            const int score = s_score(cur);
            if (score < c.best) c.best = score;
            const u2 kl = state_kl(ix, strand, cur);
            int rc = record(c, P, make_hit(strand, kl.x, kl.y, s_len(cur), score, s_nmm(cur), s_ngo(cur), s_nge(cur)),
                            phase);
            if (rc) return -rc;
            valid = false;
            continue;
        }
        return 1;
    }
}

// Children of an expanded state, from its string's four extensions, built
// directly in packed form: each differs from the parent by a few field
// increments.  gaps_only: a run's position, whose match was taken before.
// They are taken in reverse of the fixed order (match, mismatches by base,
// insertion, deletions by base); the first surviving one becomes cur, the
// others are pushed with their lower bounds.  Returns R_OK or R_STACK.
__device__ int expand_children(u4 &cur, bool &valid, const Kids &k, bool gaps_only, int b, int m, int maxd, int Di,
                               int Dn, const Seed &S, const Params &P, LaneCtx &c, uint32_t K) {
    const int i = s_i(cur), gs = s_gs(cur), ngo = s_ngo(cur), nge = s_nge(cur), sd = s_sd(cur);
    const int score = s_score(cur), len = s_len(cur);
    const bool coded = (uint32_t)len < K;  // the children not taken are then one entry
    const int diffs = s_nmm(cur) + ngo + nge;
    const int bound = (P.mode == BWFM_MODE_BEST && c.best != INF_SCORE) ? c.best + P.s_mm : INF_SCORE;
    const uint32_t z0 = cur.z & ~(3u << 10);  // gap state cleared
    const uint32_t len1 = (uint32_t)(len + 1) << 10;
    // room for the at most 8 states pushed below: checked once per
    // expansion.  Entries below sbase were handed to other lanes; sliding
    // the pending ones down makes room when the top of the stack is reached.
    if (c.sp + 8 > c.stack_cap && c.sbase > 0) {
        for (uint32_t j = c.sbase; j < c.sp; j++)
            c.stack[(size_t)(j - c.sbase) * c.sstride] = c.stack[(size_t)j * c.sstride];
        c.sp -= c.sbase;
        c.sbase = 0;
    }
    if (c.sp + 8 > c.stack_cap) {
        valid = false;
        return R_STACK;
    }
    const uint32_t sp0 = c.sp;
    u4 last = cur;
    auto push = [&](u4 v) {
        c.stack[(size_t)c.sp * c.sstride] = v;
        c.sp++;
        last = v;
    };
    uint32_t fam = 0;
    int fam_lb = INF_SCORE;
    auto push_set = [&](uint32_t set, uint32_t z, uint32_t w) {
        while (set) {  // highest base first, so that the lowest is taken first
            const int a = 31 - __clz((int)set);
            set &= ~(1u << a);
            push(mk4(sel4(k.x, a), sel4(k.y, a), z, w));
        }
    };
    // deletions: reference base a between read bases i and i + 1 (same i)
    {
        const int bd = i + 1;
        const bool ext = gs == GAP_DEL;
        const int nd = diffs + 1, ngo2 = ngo + (ext ? 0 : 1), nge2 = nge + (ext ? 1 : 0);
        const int in = (bd > S.lo && bd < S.hi) ? 1 : 0;
        const int nsc = score + (ext ? P.s_gape : P.s_gapo);
        const int lb = nsc + P.minc * Di;
        if (bd >= P.s1 && bd <= m - P.s1 && nd <= maxd && ngo2 <= P.max_gapo &&
            (P.max_gape < 0 || nge2 <= P.max_gape) && (S.sl == 0 || sd + in <= P.seed_diff) && nd + Di <= maxd &&
            lb <= bound) {
            if (coded) {
                fam |= k.mask << 8;
                if (k.mask) fam_lb = lb;
            } else {
                push_set(k.mask,
                         (z0 | ((uint32_t)GAP_DEL << 10)) + (ext ? (1u << 20) : (1u << 16)) + ((uint32_t)in << 24),
                         (uint32_t)nsc | len1 | ((uint32_t)lb << 20));
            }
        }
    }
    const int in_i = (i >= S.lo && i < S.hi) ? 1 : 0;
    // insertion: read base w[i] without a reference base (same interval)
    if (i >= P.ies && i < m - P.ies) {
        const bool ext = gs == GAP_INS;
        const int nd = diffs + 1, ngo2 = ngo + (ext ? 0 : 1), nge2 = nge + (ext ? 1 : 0);
        const int nsc = score + (ext ? P.s_gape : P.s_gapo);
        const int lb = nsc + P.minc * Dn;
        if (nd <= maxd && ngo2 <= P.max_gapo && (P.max_gape < 0 || nge2 <= P.max_gape) &&
            (S.sl == 0 || sd + in_i <= P.seed_diff) && nd + Dn <= maxd && lb <= bound) {
            if (coded) {
                fam |= FAM_INS;
                fam_lb = min(fam_lb, lb);
            } else {
                push(mk4(cur.x, cur.y,
                         (z0 | ((uint32_t)GAP_INS << 10)) - 1u + (ext ? (1u << 20) : (1u << 16)) +
                             ((uint32_t)in_i << 24),
                         (uint32_t)nsc | ((uint32_t)len << 10) | ((uint32_t)lb << 20)));
            }
        }
    }
    // mismatches, then the match, which becomes current
    bool match = false;
    if (!gaps_only) {
        const int nsc = score + P.s_mm;
        const int lb = nsc + P.minc * Dn;
        if (diffs + 1 <= maxd && (S.sl == 0 || sd + in_i <= P.seed_diff) && diffs + 1 + Dn <= maxd && lb <= bound) {
            const uint32_t set = k.mask & ~(b < 4 ? 1u << b : 0u);
            if (coded) {
                fam |= set;
                if (set) fam_lb = min(fam_lb, lb);
            } else {
                push_set(set, z0 - 1u + (1u << 12) + ((uint32_t)in_i << 24),
                         (uint32_t)nsc | len1 | ((uint32_t)lb << 20));
            }
        }
        if (fam) push(mk4(cur.x, fam, cur.z | FAMILY, (cur.w & 0xfffffu) | ((uint32_t)fam_lb << 20)));
        const int lbm = score + P.minc * Dn;
        match = b < 4 && ((k.mask >> b) & 1u) && diffs + Dn <= maxd && lbm <= bound;
        if (match) {
            const bool code = (uint32_t)(len + 1) < K;
            cur = mk4(code ? (cur.x << 2) | (uint32_t)b : sel4(k.x, b), sel4(k.y, b), z0 - 1u,
                      (uint32_t)score | len1 | ((uint32_t)lbm << 20));
        }
    }
    valid = match || c.sp > sp0;
    if (!match && c.sp > sp0) {
        c.sp--;
        cur = last;
    }
    return R_OK;
}

// One step of the search from cur, for the lanes that go: the next of a
// family, a run of matches or the children through the interval table, the
// text, or the rank lines of the search index qd (direction qdir).  Loads of
// all kinds are issued before any is used, so lanes that take different ways
// share one round trip.  Returns R_OK or R_STACK.
template <int LW>
__device__ __forceinline__ int search_step(const DevIndex &ix, const DevDir &qd, int qdir, bool go, u4 &cur,
                                           bool &valid, int m, int maxd, bool has_n, const Seed &S, const Params &P,
                                           LaneCtx &c) {
    const int K = (int)ix.kt_levels;
    const int bound = (P.mode == BWFM_MODE_BEST && c.best != INF_SCORE) ? c.best + P.s_mm : INF_SCORE;
    const bool unroll = go && s_gs(cur) == GAP_RUN;
    const bool fam = go && (cur.z & FAMILY) != 0;
    bool shallow = go && !unroll && s_len(cur) < K;
    const bool deep = go && !unroll && !shallow;
    // a family: the children that the bound leaves, of them one kind now --
    // cur becomes its children's common state (x still the parent's code),
    // sib their bases (0: the insertion, whose code is the parent's)
    const uint32_t pz = cur.z, pw = cur.w;
    uint32_t sib = 0, left = 0;  // left: the family's other kinds
    if (fam) {
        const int i = s_i(cur), gs = s_gs(cur), score = s_score(cur), len = s_len(cur);
        const int Di = c.pd[i] >> 3, Dn = i > 0 ? c.pd[i - 1] >> 3 : 0;
        const bool xi = gs == GAP_INS, xd = gs == GAP_DEL;
        const int sm = score + P.s_mm, si = score + (xi ? P.s_gape : P.s_gapo), sd = score + (xd ? P.s_gape : P.s_gapo);
        const int lbm = sm + P.minc * Dn, lbi = si + P.minc * Dn, lbd = sd + P.minc * Di;
        left = (lbm <= bound ? cur.y & FAM_MM : 0u) | (lbi <= bound ? cur.y & FAM_INS : 0u) |
               (lbd <= bound ? cur.y & FAM_DEL : 0u);
        const uint32_t z0 = cur.z & ~(FAMILY | (3u << 10));
        const uint32_t in_i = (i >= S.lo && i < S.hi) ? 1u << 24 : 0u;
        if (left & FAM_MM) {
            sib = left & FAM_MM;
            left &= ~FAM_MM;
            cur.z = z0 - 1u + (1u << 12) + in_i;
            cur.w = (uint32_t)sm | ((uint32_t)(len + 1) << 10) | ((uint32_t)lbm << 20);
        } else if (left & FAM_INS) {
            left &= ~FAM_INS;
            cur.z = (z0 | ((uint32_t)GAP_INS << 10)) - 1u + (xi ? 1u << 20 : 1u << 16) + in_i;
            cur.w = (uint32_t)si | ((uint32_t)len << 10) | ((uint32_t)lbi << 20);
        } else if (left) {
            sib = left >> 8;
            left = 0;
            cur.z = (z0 | ((uint32_t)GAP_DEL << 10)) + (xd ? 1u << 20 : 1u << 16) +
                    ((i + 1 > S.lo && i + 1 < S.hi) ? 1u << 24 : 0u);
            cur.w = (uint32_t)sd | ((uint32_t)(len + 1) << 10) | ((uint32_t)lbd << 20);
        } else {
            shallow = false;  // nothing the bound leaves
            valid = false;
        }
    }
    // the family entry of what is left with `rest` of the kind taken (lb stays
    // the lowest of the whole family's)
    auto family = [&](uint32_t rest) {
        return mk4(cur.x, left | (s_gs(cur) == GAP_DEL ? rest << 8 : rest), pz, pw);
    };
    const int len = s_len(cur), i = s_i(cur);
    const bool text = deep && K && cur.y >= SINGLE0;
    const bool conv = deep && !text && to_text(ix, cur);
    const bool rank = deep && !text && !conv;
    int q = 0;
    bool run = false, sure = false;  // sure: no difference fits in the NEXT bases after the run either
    if (shallow) {
        q = run_steps(ix, cur, c.pd, maxd, bound, has_n, S, P);
        run = q > 0 || len == K;
        if (q > 0) {
            const int e = i - q - NEXT;
            const int De = e >= 0 ? c.pd[e] >> 3 : 0;
            sure = s_nmm(cur) + s_ngo(cur) + s_nge(cur) + 1 + De > maxd ||
                   s_score(cur) + P.minc + P.minc * De > bound;
        }
    }
    // the pattern bases of a run and the next ones, or of a text step
    const int nx = run ? min(NEXT, i + 1 - q) : 0;
    const int w = run ? q : (text && !has_n && s_gs(cur) == 0 && cur.x ? min(16, i + 1) : 0);
    uint32_t code = 0, next = 0;
    if (w + nx) {
        const uint64_t cw = row_code<6>(c.pd, i + 1 - w - nx, w + nx);
        next = (uint32_t)cw & ((1u << (2 * nx)) - 1u);
        code = (uint32_t)(cw >> (2 * nx));
    }
    const uint32_t sib1 = sib & (sib - 1), sib2 = sib1 & (sib1 - 1);
    u4 ta = mk4(0, 0, 0, 0), tb = ta;
    const bool kids = shallow && !run && i >= 0;
    if (run) {
        // up to three siblings' runs at once
        const u2 *e = reinterpret_cast<const u2 *>(qd.kt) + kt_start32(K) + code;
        const uint32_t x0 = sib ? (cur.x << 2) | (uint32_t)(__ffs((int)sib) - 1) : cur.x;
        const u2 v = e[x0 << (2 * q)];
        ta.x = v.x;
        ta.y = v.y;
        if (sib1) {
            const u2 v1 = e[((cur.x << 2) | (uint32_t)(__ffs((int)sib1) - 1)) << (2 * q)];
            ta.z = v1.x;
            ta.w = v1.y;
        }
        if (sib2) {
            const u2 v2 = e[((cur.x << 2) | (uint32_t)(__ffs((int)sib2) - 1)) << (2 * q)];
            tb.x = v2.x;
            tb.y = v2.y;
        }
    } else if (shallow) {
        // the first child on its own, the rest of the family back on the stack
        if (left | sib1) {
            c.stack[(size_t)c.sp * c.sstride] = family(sib1);
            c.sp++;
        }
        if (sib) cur.x = (cur.x << 2) | (uint32_t)(__ffs((int)sib) - 1);
        if (kids) {
            const u4 *e = reinterpret_cast<const u4 *>(qd.kt) + (kt_children(len, cur.x) >> 1);
            ta = e[0];
            tb = e[1];
        }
    }
    if (text && cur.x) {
        const u2w v = *reinterpret_cast<const u2w *>(ix.pac + text_word(ix, qdir, cur.x));
        ta.x = v.x;
        ta.y = v.y;
    }
    if (conv) ta.x = qd.full[cur.x];
    Kids k;
    k.mask = 0;
#pragma unroll
    for (int a = 0; a < 4; a++) k.x[a] = k.y[a] = 0;
    if (rank) rank_children<LW>(ix, qd, cur.x, cur.y + 1, k);

    bool grow = rank || unroll || kids;
    if (run) {
        uint32_t n = 0;  // states expanded by the runs that end
        // whether the run of entry kl ends: its string is absent (kl.x - 1
        // of its bases occur), or occurs once and is not followed by the
        // pattern's next bases
        next = rev_digits(next, nx);  // the first to come in the lowest digit
        auto ends = [&](u2 kl) {
            if (kl.y == 0) {
                n += kl.x - (uint32_t)len;
                return true;
            }
            if (!sure || kl.y < SINGLE0 || kl.y == SINGLE) return false;
            const uint32_t df = (kl.y ^ next) & ((1u << (2 * nx)) - 1u);
            if (!df) return false;
            n += (uint32_t)q + ((uint32_t)(__ffs((int)df) - 1) >> 1) + 1u;
            return true;
        };
        u2 kl = mk2(ta.x, ta.y);
        uint32_t rest = sib1;
        bool over = ends(kl);
        if (over && sib1) {
            kl = mk2(ta.z, ta.w);
            rest = sib2;
            over = ends(kl);
            if (over && sib2) {
                kl = mk2(tb.x, tb.y);
                rest = sib2 & (sib2 - 1);
                over = ends(kl);
            }
        }
        const bool more = (left | rest) != 0;
        const u4 f = family(rest);
        if (over) {
            cur = f;
            valid = more;
        } else {
            if (more) {
                c.stack[(size_t)c.sp * c.sstride] = f;
                c.sp++;
            }
            step_matches(cur, q, c.pd, P);
            cur.x = kl.x;
            cur.y = kl.y;
            n += (uint32_t)q;
        }
        c.expand += n;
    } else if (kids) {
        kt_pick(ta, tb, k);
    }
    if (conv) {
        cur.x = ta.x;
        cur.y = SINGLE;
    }
    if (text) {
        uint32_t win = text_bases(ix, qdir, cur.x, ta.x, ta.y);
        if (qdir) win = rev16(win);
        grow = !text_step(cur, win, code, w, maxd, bound, P, c, k);
    }
    if (unroll) unroll_run(cur, P, c, k);
    int rc = R_OK;
    if (grow) {
        if (!unroll && !text) c.expand++;
        const int j = s_i(cur);
        rc = expand_children(cur, valid, k, unroll, pd_base(c, j), m, maxd, pd_d(c, j), pd_d(c, j - 1), S, P, c,
                             (uint32_t)K);
    }
    return rc;
}

// Rewrite cnt bytes of the row from `at` on as base | z << 3, for strand -
// complementing the staged strand + bases (none of them N): whole dwords,
// loaded before any is stored.
__device__ __forceinline__ void row_fill(uint8_t *row, int at, int cnt, int z, int flip) {
    uint32_t *A = reinterpret_cast<uint32_t *>(row) + (at >> 2);
    const int sh = at & 3, nd = (sh + cnt + 3) >> 2;  // cnt <= 16: at most 5 dwords
    uint32_t v[5];
#pragma unroll
    for (int t = 0; t < 5; t++) v[t] = t < nd ? A[t] : 0u;
#pragma unroll
    for (int t = 0; t < 5; t++) {
        const int b0 = max(sh - 4 * t, 0), b1 = min(sh + cnt - 4 * t, 4);  // bytes [b0, b1) of this dword
        if (t < nd && b0 < b1) {
            const uint32_t mk = (b1 >= 4 ? 0xffffffffu : (1u << (8 * b1)) - 1u) & ~((1u << (8 * b0)) - 1u);
            const uint32_t nv = ((v[t] ^ (flip ? 0x03030303u : 0u)) & 0x07070707u) | (0x08080808u * (uint32_t)z);
            A[t] = (v[t] & ~mk) | (nv & mk);
        }
    }
}

// Matches of row[di, di + q) with the text bases next to be prepended at
// position p > 0 (words w0, w1) in the D-array scan's direction (0 for strand
// +, 1 for strand -), where the pattern is taken from its start.
__device__ __forceinline__ int dtext_matches(const DevIndex &ix, int strand, uint32_t p, uint32_t w0, uint32_t w1,
                                             const uint8_t *row, int di, int q) {
    uint32_t win = text_bases(ix, strand, p, w0, w1);
    if (strand == 0) win = rev16(win);
    uint32_t pc = (uint32_t)row_code(row, di, q);
    if (strand) pc = ~pc;
    const uint32_t df = win ^ pc;
    const int t = df ? (__ffs((int)df) - 1) >> 1 : 16;
    return (int)min((uint32_t)min(t, q), p);
}

// D-array of one strand on the other index, in place over the staged
// pattern (strand 0: row holds reverse(read), strand 1: its complement is
// taken here).  Returns false when the bound already exceeds the budget at
// the root (the strand cannot match).
template <int LW>
__device__ bool build_d(const DevIndex &ix, const DevDir &od, int m, int strand, int maxd, bool has_n, LaneCtx &c) {
    uint32_t k = 0, l = ix.n;
    bool fresh = true;  // at the start of a segment
    int z = 0;
    // bases from position i on, at most r, before an N
    auto to_n = [&](int i, int r) {
        int q = 0;
        while (q < r && !(c.pd[i + q] & 4)) q++;
        return q;
    };
    for (int i = 0; i < m;) {
        int d = 0;           // bases that occur from i on
        bool empty = true;   // and the next one ends the segment
        if (fresh && ix.kt_levels) {
            // the segment's first bases in one table entry
            int r = min((int)ix.kt_levels, m - i);
            if (has_n) r = to_n(i, r);
            if (r) {
                uint32_t code = rev_digits((uint32_t)row_code(c.pd, i, r), r);
                if (strand) code ^= (1u << (2 * r)) - 1u;
                const u2 kl = reinterpret_cast<const u2 *>(od.kt)[kt_start32(r) + code];
                empty = kl.y == 0;
                d = empty ? (int)kl.x - 1 : r;
                k = kl.x;
                l = kl.y;
            }
        } else if (ix.kt_levels && l >= SINGLE0) {
            // followed in the text to the first base that differs
            int r = min(16, m - i);
            if (has_n) r = to_n(i, r);
            if (k && r) {
                const u2w w = *reinterpret_cast<const u2w *>(ix.pac + text_word(ix, strand, k));
                d = dtext_matches(ix, strand, k, w.x, w.y, c.pd, i, r);
                k -= (uint32_t)d;
            }
            empty = d < r || r == 0;
        } else {
            const int b = c.pd[i] & 7;
            const int a = (strand == 0 || b > 3) ? b : 3 - b;
            if (a < 4) {
                const uint32_t ok = occ1<LW>(ix, od, a, k), ol = occ1<LW>(ix, od, a, l + 1);
                empty = ok >= ol;
                d = empty ? 0 : 1;
                k = sel4(od.C, a) + ok;
                l = sel4(od.C, a) + ol - 1;
                if (k == l && !empty && ix.kt_levels) {
                    k = od.full[k];
                    l = SINGLE;
                }
            }
        }
        row_fill(c.pd, i, d, z, strand);
        i += d;
        fresh = empty;
        if (empty) {
            if (++z > maxd) return false;
            // (an N keeps its code on both strands)
            row_fill(c.pd, i, 1, z, strand && !(c.pd[i] & 4));
            i++;
            k = 0;
            l = ix.n;
        }
    }
    return true;
}

// Depth-first search of one strand, one lane, start to end.
template <int LW>
__device__ int search_strand(const DevIndex &ix, const DevDir &sd_, int m, int strand, int maxd, bool has_n,
                             const Params &P, LaneCtx &c, int phase) {
    const Seed S = seed_of(P, m);
    u4 cur = root_state(ix, m, P.minc * pd_d(c, m - 1));
    bool valid = true;
    c.sp = 0;
    for (;;) {
        int rr = resolve(cur, valid, strand, P, c, phase, 0x7fffffff, ix);
        if (rr == 0) return R_OK;
        if (rr < 0) return -rr;
        const int rc = search_step<LW>(ix, sd_, strand == 0 ? 1 : 0, true, cur, valid, m, maxd, has_n, S, P, c);
        if (rc) return rc;
    }
}

// Canonicalise the lane's hit buffer: tiers, c1/c2, the max_hits rule, the
// report order.  Returns the number of reported hits (at the front of the
// buffer); sets status, c1, c2.
__device__ uint32_t finish(LaneCtx &c, const Params &P, uint8_t &status, uint32_t &c1o, uint32_t &c2o) {
    status = 0;
    c1o = c2o = 0;
    if (c.ncand == 0) return 0;
    const int S = c.best;
    uint32_t n = 0;
    uint64_t c1 = 0, c2 = 0;
    for (uint32_t j = 0; j < c.ncand; j++) {
        u4 h = c.cand[(size_t)j * c.cstride];
        int sc = h_score(h);
        if (P.mode == BWFM_MODE_ALL || sc <= S + P.s_mm) c.cand[(size_t)(n++) * c.cstride] = h;
        uint64_t w = (uint64_t)h.y - h.x + 1;
        if (sc == S) c1 += w;
        else if (sc <= S + P.s_mm) c2 += w;
    }
    if (n > P.max_hits) {
        status = BWFM_ST_OVERFLOW;
        c1o = c2o = 0xffffffffu;
        return 0;
    }
    c1o = c1 > 0xffffffffULL ? 0xffffffffu : (uint32_t)c1;
    c2o = c2 > 0xffffffffULL ? 0xffffffffu : (uint32_t)c2;
    const bool keep2 = c1 <= (uint64_t)P.max_best;
    uint32_t r = 0;
    for (uint32_t j = 0; j < n; j++) {
        u4 h = c.cand[(size_t)j * c.cstride];
        if (P.mode == BWFM_MODE_ALL || h_score(h) == S || keep2) c.cand[(size_t)(r++) * c.cstride] = h;
    }
    for (uint32_t j = 1; j < r; j++) {  // insertion sort by (score, strand, k, len)
        u4 v = c.cand[(size_t)j * c.cstride];
        uint32_t q = j;
        while (q > 0) {
            u4 u = c.cand[(size_t)(q - 1) * c.cstride];
            if (!before(v, u)) break;
            c.cand[(size_t)q * c.cstride] = u;
            q--;
        }
        c.cand[(size_t)q * c.cstride] = v;
    }
    status = r ? BWFM_ST_HIT : 0;
    return r;
}

// Both strands of one read, one lane: the read is staged in the lane's row
// once per strand (its D-array scan rewrites the row in place).
template <int LW>
__device__ int align_read(const DevIndex &ix, const uint8_t *W, int m, int maxd, const Params &P, LaneCtx &c,
                          int phase) {
    c.ncand = 0;
    const bool has_n = stage_read(c.pd, W, m);
    for (int strand = 0; strand < 2; strand++) {
        const DevDir sdir = pick_dir(ix, strand == 0 ? 1 : 0);
        const DevDir odir = pick_dir(ix, strand == 0 ? 0 : 1);
        if (!build_d<LW>(ix, odir, m, strand, maxd, has_n, c)) continue;
        int rc = search_strand<LW>(ix, sdir, m, strand, maxd, has_n, P, c, phase);
        if (rc) return rc;
    }
    return R_OK;
}

// Per-read outputs shared by the kernels.
struct ReadOut {
    uint32_t *n_rep, *c1, *c2;
    uint8_t *status;
    uint32_t *slow_list, *n_slow;
    u4 *stage;                    // reported hits, a block per read
    unsigned long long *stage_used;  // staging slots taken
    uint64_t stage_cap;
    uint64_t *stage_off;             // per read: first staging slot
    uint32_t *expand;                // per read work counter, or NULL
    unsigned long long *work;        // or NULL: [0] wave iterations, [1] lane iterations with a read,
                                     // [2] lane iterations that issued a rank query
};

__device__ __forceinline__ void send_to_second_pass(const ReadOut &O, uint32_t r) {
    as_global(O.status)[r] = ST_RESEARCH;
    as_global(O.n_rep)[r] = 0;
    as_global(O.slow_list)[atomicAdd(as_global(O.n_slow), 1u)] = r;
}

// Move a read's nr reported hits (the front of its hit buffer) to the
// staging arena.  The arena holds as many hits as the caller's output, so
// running out of it means the output is too small: the count is kept (the
// offsets scan then reports what is needed) and nothing is copied.
__device__ void stage_hits(const LaneCtx &c, const ReadOut &O, uint32_t r, uint32_t nr) {
    if (!nr) return;
    const unsigned long long off = atomicAdd(as_global(O.stage_used), (unsigned long long)nr);
    if (off + nr > O.stage_cap) return;
    u4 *stage = as_global(O.stage);
    for (uint32_t j = 0; j < nr; j++) stage[off + j] = c.cand[(size_t)j * c.cstride];
    as_global(O.stage_off)[r] = off;
}

// Canonicalise a finished read and move its reported hits to the staging
// arena.
__device__ void publish(LaneCtx &c, const Params &P, const ReadOut &O, uint32_t r, uint8_t extra = 0) {
    uint8_t st;
    uint32_t a, b;
    uint32_t nr = finish(c, P, st, a, b);
    if (O.expand) as_global(O.expand)[r] = c.expand;
    stage_hits(c, O, r, nr);
    as_global(O.n_rep)[r] = nr;
    as_global(O.status)[r] = st | extra;
    as_global(O.c1)[r] = a;
    as_global(O.c2)[r] = b;
}

// validity of read r: 0 = search it, 1 = done (empty or invalid, outputs written)
__device__ __forceinline__ int check_read(const ReadsView &rd, const Params &P, const ReadOut &O, uint32_t r, int &m,
                                          int &maxd, uint64_t &o0) {
    uint64_t len;
    bool bad;
    read_span(rd, r, o0, len, bad);
    m = (int)len;
    maxd = rd.maxd ? as_global(rd.maxd)[r] : P.max_diff;
    // (a read that is searched gets its outputs when it is published)
    const bool invalid = bad || len > rd.max_len || len > BWFM_MAX_READ || maxd > BWFM_MAX_DIFF;
    if (invalid || m == 0) {
        as_global(O.n_rep)[r] = 0;
        as_global(O.c1)[r] = 0;
        as_global(O.c2)[r] = 0;
        if (O.expand) as_global(O.expand)[r] = 0;
        as_global(O.status)[r] = invalid ? BWFM_ST_INVALID : 0;
        return 1;
    }
    return 0;
}

// Copy n dwords, the loads of eight issued before their stores: through
// generic pointers the compiler must assume a store may alias the next
// load, so a plain loop waits one memory round trip per dword.
__device__ __forceinline__ void copy_dwords(uint32_t *dst, const uint32_t *src, int n) {
    for (int k0 = 0; k0 < n; k0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = k0 + j < n ? src[k0 + j] : 0u;
#pragma unroll
        for (int j = 0; j < 8; j++)
            if (k0 + j < n) dst[k0 + j] = v[j];
    }
}

// ------------------------------------------------------------------ split searches

// Batched form: a read whose search outgrows a budget of expansions is
// split.  Its pending states become tasks that any lane of the grid may
// take, in rounds of one launch each, so that the largest trees of a batch
// are searched by the whole device rather than by one lane or one wave.
// The read's slot holds what a task needs (the strand's pattern and D-array
// row, the read's length and budget, the best score found so far) and
// collects the hits of every part; after the rounds each slot's read is
// canonicalised like any other, duplicates merged first.  The reported hits
// do not depend on how the tree was cut: each part prunes with a bound that
// is never below the final one, so every hit within the final bound is
// found by the part that holds it.
constexpr int SPLIT_ROUNDS = 8;               // task rounds; the last one runs every task to its end
constexpr uint32_t TASK_EMPTY = 0xffffffffu;  // a reserved task entry left unused
// hits a slot collects: those of the read's first-pass lane (at most
// FAST_CAND), then at most as many again from its tasks
constexpr uint32_t SLOT_HITS = 2 * FAST_CAND;
// control words: [0] slots taken; [1 + g] task entries reserved in
// generation g (0: by the first pass, k: by round k); [2 + SPLIT_ROUNDS + g]
// entries of generation g taken by round g + 1
// [SPLIT_DONE] waves of the first pass that have ended, plus DRAIN_HEAVY once
// DRAIN_SLOTS reads have been split; [SPLIT_LONG] long reads in every
// sixteenth wave of the D-array pass
constexpr uint32_t SPLIT_DONE = 2 * (SPLIT_ROUNDS + 1) + 2;
constexpr uint32_t SPLIT_LONG = SPLIT_DONE + 1;
constexpr uint32_t SPLIT_CTL = SPLIT_LONG + 1;
// Early splits: once DRAIN_EIGHTHS of the first pass's waves have ended, the
// parts still running are split after DRAIN_BUDGET expansions already, in a
// batch with an eighth of long reads or more (as the D-array pass sees them,
// not as the caller declares them): the few reads with the largest trees would
// otherwise hold single waves until each part has reached the full budget
// (150 k reads of 250 bases: 184 ms without, 47 with; 45 at 2 eighths, 58 at
// 6).  Batches of shorter reads mostly end sooner without (30 k reads of 150
// bases, 4 differences: 4.5 ms, with it 6.2), unless their trees prove as
// large: they wait for DRAIN_SLOTS reads that outgrew the full budget (50 k
// reads of 150 bases, 6 differences: 400 ms without, 110 with).  And where the
// declared length leaves the first pass a wave a SIMD or less, splitting is
// the shorter way for any reads (60 k of 100 bases, declared 512: 9.4, 8.2).
constexpr uint32_t DRAIN_EIGHTHS = 4, DRAIN_BUDGET = 256, DRAIN_SLOTS = 64, DRAIN_HEAVY = 1u << 24;

struct SplitBufs {
    uint32_t *slot_read;    // the slot's read
    uint32_t *slot_meta;    // m | budget << 10 | the read holds an N << 14
    int *slot_best;         // best score found by any part
    uint32_t *slot_nhit;    // hits delivered (above SLOT_HITS: the slot failed)
    uint32_t *slot_fail;    // nonzero: the read goes to the second pass
    uint32_t *slot_exp;     // states expanded by the read's parts
    uint32_t *slot_owner;   // the first-pass lane that owns the read (its hit buffer)
    uint32_t *slot_own;     // hits in that buffer when the first pass finished the read
    int *slot_obest;        // and its best score then
    uint8_t *slot_rows;     // per slot and strand: the pattern and D-array row, dstride bytes
    u4 *slot_hits;       // per slot: SLOT_HITS hits
    u4 *tasks[2];        // task states, by generation parity
    uint32_t *task_ref[2];  // slot | strand << 31, or TASK_EMPTY
    uint32_t *ctl;          // SPLIT_CTL control words
    u4 *lane_cand;       // the first pass's hit buffers, FAST_CAND per lane
    uint32_t slot_cap, task_cap, dstride;
    uint32_t budget;  // expansions of a lane's part of a read before it is split (endgame); 0: off
    uint32_t count;   // nonzero: the parts' expansions are summed (per-read work counters)
    uint32_t drain;   // ctl[SPLIT_DONE] from which the parts are split early (DRAIN_EIGHTHS)
};

__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p) {
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Reserve cnt task entries of generation g at off.  False when they do not
// all fit; reserved entries inside the array are then marked unused.
__device__ bool take_tasks(const SplitBufs &X, uint32_t g, uint32_t cnt, uint32_t &off) {
    // a full generation is not reserved from again, which also keeps the
    // counter far from wrapping
    if (ld_agent(&X.ctl[1 + g]) >= X.task_cap) return false;
    off = atomicAdd(&X.ctl[1 + g], cnt);
    if (off + cnt <= X.task_cap) return true;
    for (uint32_t j = off; j < X.task_cap; j++) X.task_ref[g & 1][j] = TASK_EMPTY;
    return false;
}

// Task entries a pending state takes: one, or a family's children one each.
__device__ __forceinline__ uint32_t task_count(u4 v) { return (v.z & FAMILY) ? (uint32_t)__popc(v.y) : 1u; }
__device__ uint32_t task_count(const LaneCtx &c, u4 cur, bool has_cur) {
    uint32_t n = has_cur ? task_count(cur) : 0u;
    for (uint32_t j = c.sbase; j < c.sp; j++) n += task_count(c.stack[(size_t)j * c.sstride]);
    return n;
}

// Write cur when has_cur, then the lane's pending stack entries, to the
// entries reserved at off in generation g; the lane's stack is left empty.
__device__ void put_tasks(const SplitBufs &X, uint32_t g, uint32_t off, uint32_t ref, LaneCtx &c, u4 cur,
                          bool has_cur) {
    u4 *T = as_global(X.tasks[g & 1]);
    uint32_t *R = as_global(X.task_ref[g & 1]);
    auto put = [&](u4 v) {
        uint32_t set = (v.z & FAMILY) ? v.y : 1u;
        for (; set; set &= set - 1, off++) {
            if (v.z & FAMILY) v.y = set & (0u - set);
            T[off] = v;
            R[off] = ref;
        }
    };
    if (has_cur) put(cur);
    for (uint32_t j = c.sbase; j < c.sp; j++) put(c.stack[(size_t)j * c.sstride]);
    c.sp = c.sbase = 0;
}

// Copy an m-byte pattern and D-array row from the lane's LDS row to the
// slot: whole dwords, within both rows.
// (A plain loop on purpose: this runs once per split read, in the endgame of
// the batched kernel, and a batched copy there changed the code of that
// kernel's whole loop and cost it about 3% on 100-base reads.)
__device__ __forceinline__ void save_row(const SplitBufs &X, uint32_t s, int strand, const uint8_t *pd, int m) {
    const uint32_t *src = reinterpret_cast<const uint32_t *>(pd);
    uint32_t *dst = reinterpret_cast<uint32_t *>(X.slot_rows + ((size_t)s * 2 + (size_t)strand) * X.dstride);
    for (int k = 0; k < (m + 3) / 4; k++) dst[k] = src[k];
}
// Deliver the lane's hits to slot s -- those within the bound of the best
// score known -- with its expansions; the lane's hit buffer is emptied.
__device__ void flush_slot(const SplitBufs &X, const Params &P, uint32_t s, LaneCtx &c) {
    if (X.count && c.expand) atomicAdd(&X.slot_exp[s], c.expand);
    c.expand = 0;
    // a lane's best score changes only with a hit it holds: without hits
    // there is nothing to deliver
    if (c.ncand == 0) return;
    const int old = atomicMin(&X.slot_best[s], c.best);
    const int best = old < c.best ? old : c.best;
    const int bound = (P.mode == BWFM_MODE_BEST && best != INF_SCORE) ? best + P.s_mm : INF_SCORE;
    uint32_t keep = 0;
    for (uint32_t j = 0; j < c.ncand; j++) keep += h_score(c.cand[(size_t)j * c.cstride]) <= bound ? 1u : 0u;
    if (keep) {
        uint32_t off = atomicAdd(&X.slot_nhit[s], keep);
        if (off + keep > SLOT_HITS) {  // the collection left room for FAST_CAND of them
            atomicOr(&X.slot_fail[s], 1u);
        } else {
            u4 *dst = X.slot_hits + (size_t)s * SLOT_HITS;
            for (uint32_t j = 0; j < c.ncand; j++) {
                const u4 h = c.cand[(size_t)j * c.cstride];
                if (h_score(h) <= bound) dst[off++] = h;
            }
        }
    }
    c.ncand = 0;
}

// Flag word of a read in its wave's sharing block: SH_FAIL, SH_HELPED, the
// strands whose rows the read's slot holds, SH_NOSPLIT once a split found
// no room, and the slot plus one above SH_SLOT_SHIFT (0: none yet).
enum { SH_FAIL = 1, SH_HELPED = 2, SH_ROW0 = 4, SH_NOSPLIT = 16 };
constexpr int SH_SLOT_SHIFT = 5;

// Endgame of the first pass: hand this lane's part of read r on `strand`
// -- cur when valid, then the pending stack entries -- to the tasks of
// generation 0, taking the read's slot at its first split (fl is the
// read's flag word; best its best score so far; owner the global index of
// the lane that owns the read).  The caller runs one lane of a wave at a
// time.  False, with the lane's search unchanged, when no slot or task room
// is left.
__device__ bool split_part(const SplitBufs &X, uint32_t r, uint32_t owner, int strand, int m, int maxd, bool has_n,
                           int best, LaneCtx &c, u4 cur, bool valid, int &fl) {
    const uint32_t cnt = task_count(c, cur, valid);
    const bool had = (fl >> SH_SLOT_SHIFT) != 0;
    if (!had && ld_agent(&X.ctl[0]) >= X.slot_cap) return false;
    uint32_t off = 0;
    if (!take_tasks(X, 0, cnt, off)) return false;
    uint32_t s;
    if (had) {
        s = (uint32_t)(fl >> SH_SLOT_SHIFT) - 1;
    } else {
        s = atomicAdd(&X.ctl[0], 1u);
        if (s >= X.slot_cap) {
            for (uint32_t j = 0; j < cnt; j++) X.task_ref[0][off + j] = TASK_EMPTY;
            return false;
        }
        X.slot_read[s] = r;
        X.slot_meta[s] = (uint32_t)m | ((uint32_t)maxd << 10) | ((uint32_t)has_n << 14);
        X.slot_best[s] = best;
        X.slot_nhit[s] = 0;
        X.slot_fail[s] = 0;
        X.slot_exp[s] = 0;
        X.slot_owner[s] = owner;
        X.slot_own[s] = 0;
        X.slot_obest[s] = INF_SCORE;
        if (s + 1 == DRAIN_SLOTS && X.drain >= DRAIN_HEAVY) atomicAdd(&X.ctl[SPLIT_DONE], DRAIN_HEAVY);
        fl |= (int)((s + 1) << SH_SLOT_SHIFT);
    }
    if (!(fl & (SH_ROW0 << strand))) {
        save_row(X, s, strand, c.pd, m);
        fl |= SH_ROW0 << strand;
    }
    put_tasks(X, 0, off, s | ((uint32_t)strand << 31), c, cur, valid);
    return true;
}

// The first pass's end of a split read (fl: its flag word, with the slot):
// the owner's hits stay in its hit buffer -- a lane whose wave has reached
// the endgame takes no further read -- and the slot records their number
// and the best score, for the collection before the rounds.  A failed read
// goes to the second pass through its slot.
__device__ __forceinline__ void end_split_read(const SplitBufs &X, const LaneCtx &c, int fl) {
    const uint32_t s = (uint32_t)(fl >> SH_SLOT_SHIFT) - 1;
    if (fl & SH_FAIL) {
        X.slot_fail[s] = 1;
        return;
    }
    X.slot_own[s] = c.ncand;
    X.slot_obest[s] = c.best;
    if (X.count) X.slot_exp[s] += c.expand;
}

// Before the rounds: each split read's first-pass hits join its slot's
// list, and the slot's best score takes theirs.  One thread per slot.
__global__ void k_split_collect(SplitBufs X) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= min(X.ctl[0], X.slot_cap) || X.slot_fail[s]) return;
    const uint32_t n = X.slot_own[s];
    const u4 *src = X.lane_cand + (size_t)X.slot_owner[s] * FAST_CAND;
    u4 *dst = X.slot_hits + (size_t)s * SLOT_HITS;
    for (uint32_t j = 0; j < n; j++) dst[j] = src[j];
    X.slot_nhit[s] = n;
    if (X.slot_obest[s] < X.slot_best[s]) X.slot_best[s] = X.slot_obest[s];
}

// After the rounds: each split read's hits, duplicates merged as a lane's
// buffer merges them, are canonicalised and published; a failed slot's
// read goes to the second pass.
__global__ void k_split_publish(Params P, SplitBufs X, ReadOut O) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t ns = min(X.ctl[0], X.slot_cap);
    if (s >= ns) return;
    const uint32_t r = X.slot_read[s];
    const uint32_t nh = X.slot_nhit[s];
    if (X.slot_fail[s] || nh > SLOT_HITS) {
        if (O.expand) O.expand[r] = X.slot_exp[s];
        send_to_second_pass(O, r);
        return;
    }
    LaneCtx c;
    c.cand = X.slot_hits + (size_t)s * SLOT_HITS;
    c.cstride = 1;
    uint32_t w = 0;
    for (uint32_t j = 0; j < nh; j++) {
        const u4 h = c.cand[j];
        uint32_t q = 0;
        while (q < w && !(h_strand(c.cand[q]) == h_strand(h) && c.cand[q].x == h.x && h_len(c.cand[q]) == h_len(h)))
            q++;
        if (q == w)
            c.cand[w++] = h;
        else if (better(h, c.cand[q]))
            c.cand[q] = h;
    }
    c.ncand = w;
    c.best = X.slot_best[s];
    c.expand = X.slot_exp[s];
    publish(c, P, O, r, (uint8_t)BWFM_ST_SPLIT);
}

// ------------------------------------------------------------------ kernels

// Plain form: one lane per read, one launch per batch.
template <int LW>
__global__ __launch_bounds__(BLOCK) void k_align_plain(DevIndex ix, ReadsView rd, Params P, LaneBufs B, ReadOut O) {
    uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= reads_n(rd)) return;
    int m, maxd;
    uint64_t o0;
    if (check_read(rd, P, O, r, m, maxd, o0)) return;
    LaneCtx c;
    init_ctx(c, B, r);
    int rc = align_read<LW>(ix, rd.bases + o0, m, maxd, P, c, PH_FAST);
    if (rc) {
        if (O.expand) O.expand[r] = c.expand;
        send_to_second_pass(O, r);
        return;
    }
    publish(c, P, O, r);
}

enum { PZ_IDLE = 0, PZ_TURN = 1, PZ_SEARCH = 2, PZ_HELP = 3, PZ_WAIT = 4 };

// Per-wave block in LDS through which the lanes of a wave share one read's
// search once the batch's reads are all taken: an idle lane receives the
// oldest pending state of a busy lane's stack (the root of the largest
// untouched subtree) and searches it on the owner's pattern, D-array, bound
// and hit buffer.  Arrays are indexed by the owner lane, the lane that took
// the read; box and meta pass the donated states, by donor rank.
struct WaveShare {
    int best[64];       // best score found so far for the owner's read
    int ncand[64];      // hits in the owner's hit buffer
    int pending[64];    // helper lanes still searching donated subtrees
    int flags[64];      // SH_FAIL: the hit buffer overflowed; SH_HELPED; the read's slot
    int hexp[64];       // states expanded by helpers
    u4 box[64];      // donated states
    uint32_t meta[64];  // owner lane | strand << 6 | budget << 7 | m << 11 | the read holds an N << 21
};

__device__ __forceinline__ int sh_ld(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void sh_st(int *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// order this wave's earlier LDS and global accesses before its later ones,
// as seen by the other lanes of the wave
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Batched form: a persistent grid whose lanes pull reads from a shared
// counter.  Each loop iteration performs one search expansion per busy lane,
// so lanes at different stages of different reads still share its memory
// round trips.  Lanes whose strand or read has ended wait until BWFM_TURN_MIN
// of the wave do; they then publish, take the next reads (one atomic per
// wave) and copy their rows together, sharing those round trips too.
// When the counter runs past the batch, idle lanes help the busy lanes of
// their wave through WaveShare instead of waiting for the slowest one.
// Arguments of the batched kernel that are used only at read boundaries:
// kept in device memory and loaded where used, so that they do not occupy
// scalar registers across the loop (the spills of a full argument list
// cost more vector instructions than the loop's own work).
struct PersistentArgs {
    ReadsView rd;
    LaneBufs B;
    ReadOut O;
    uint32_t *next_read;
    // the D-array pre-pass's output: per read, one row per strand of
    // dstride bytes (base | D << 3 per pattern position) and a byte whose
    // bit s is set when strand s is pruned at the root, bit 2 when the read
    // holds an N
    const uint8_t *drows;
    const uint8_t *dflag;
    uint32_t dstride;
    // split searches (X.budget 0: off), and per lane the read it owns
    // (helpers of a read find its index there)
    SplitBufs X;
    uint32_t *lane_read;
};

// Row of read r, strand s, in the pre-pass's output.
__device__ __forceinline__ const uint8_t *drow_of(const uint8_t *drows, uint32_t dstride, uint32_t r, int s) {
    return drows + ((size_t)r * 2 + (size_t)s) * dstride;
}

// D-array pre-pass of the batched form: one lane per read, both strands in
// turn on the other index, each strand's row staged in LDS and then copied
// out whole.  (In the search loop the same scan cost every wave its
// instructions in every iteration, though 4% of the lanes were at it: 2M
// reads of 100 bases searched in 72.7 ms with the scan in the loop, in 59.2
// with this pass's 3.3 ms before it and the grouped read changes.)
template <int LW>
__global__ __launch_bounds__(BLOCK) void k_dscan(DevIndex ix, ReadsView rd, Params P, uint8_t *drows, uint8_t *dflag,
                                                 uint32_t dstride, uint32_t lstride, uint32_t *n_long) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= reads_n(rd)) return;
    uint64_t o0, len;
    bool bad;
    read_span(rd, r, o0, len, bad);
    const int maxd = rd.maxd ? rd.maxd[r] : P.max_diff;
    // reads the search will not take (invalid or empty) get no rows
    if (bad || len == 0 || len > rd.max_len || len > BWFM_MAX_READ || maxd > BWFM_MAX_DIFF) return;
    const int m = (int)len;
    if (n_long && ((r >> 6) & 15) == 0) {
        const unsigned long long lm = __ballot(len >= LONG_READ);
        if (lm && (r & 63) == (uint32_t)__ffsll((long long)lm) - 1) atomicAdd(n_long, (uint32_t)__popcll(lm));
    }
    LaneCtx c;
    c.pd = lds_bytes + (size_t)threadIdx.x * lstride;
    const bool has_n = stage_read(c.pd, rd.bases + o0, m);
    uint8_t fl = has_n ? 4 : 0;
    for (int strand = 0; strand < 2; strand++) {
        const DevDir odir = pick_dir(ix, strand == 0 ? 0 : 1);
        if (!build_d<LW>(ix, odir, m, strand, maxd, has_n, c)) {
            fl |= (uint8_t)(1 << strand);
            continue;
        }
        copy_dwords(reinterpret_cast<uint32_t *>(drows + ((size_t)r * 2 + (size_t)strand) * dstride),
                    reinterpret_cast<const uint32_t *>(c.pd), (m + 3) / 4);
    }
    dflag[r] = fl;
}

// Copy a pre-pass row (m bytes) into the lane's LDS row.  The rows start
// 16-byte aligned and their stride is a multiple of 16, so whole 16-byte
// blocks are read, four of them before any store: a row costs a few memory
// round trips (one per dword when each load waits for the store before it,
// which the compiler must assume may alias it).
__device__ __forceinline__ void load_drow(uint8_t *pd, const uint8_t *row, int m) {
    const u4 *src = as_global(reinterpret_cast<const u4 *>(row));
    uint32_t *dst = reinterpret_cast<uint32_t *>(pd);
    const int ndw = (m + 3) >> 2;
    for (int q0 = 0; 4 * q0 < ndw; q0 += 4) {
        u4 v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = 4 * (q0 + j) < ndw ? src[q0 + j] : mk4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 4 * (q0 + j);
            if (k < ndw) dst[k] = v[j].x;
            if (k + 1 < ndw) dst[k + 1] = v[j].y;
            if (k + 2 < ndw) dst[k + 2] = v[j].z;
            if (k + 3 < ndw) dst[k + 3] = v[j].w;
        }
    }
}

// The batched kernel's argument block.  a.X.drain comes as the waves that must
// have ended before parts are split early; unless that is to be at once or the
// D-array pass has seen enough long reads, DRAIN_SLOTS reads must have been
// split too (which adds DRAIN_HEAVY to the count).
__global__ void k_set_args(PersistentArgs *dst, PersistentArgs a, uint32_t at_once) {
    if (threadIdx.x) return;
    if (a.X.budget && !at_once && (uint64_t)a.X.ctl[SPLIT_LONG] * 16 * 8 < reads_n(a.rd)) a.X.drain += DRAIN_HEAVY;
    *dst = a;
}

template <int LW>
__device__ __forceinline__ void persistent_body(const DevIndex &ix, const Params &P, const PersistentArgs *Aarg) {
    // the argument block, through an address space the compiler sees
    using GlobalArgs = const __attribute__((address_space(1))) PersistentArgs;
    GlobalArgs *Ag = (GlobalArgs *)Aarg;
    const PersistentArgs *A = (const PersistentArgs *)Ag;
    const uint32_t gl = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const uint32_t wave0 = threadIdx.x & ~63u;  // the wave's first thread in the block
    const uint32_t n_reads = reads_n(A->rd);
    const uint32_t lds_stride = A->B.lds_stride;
    WaveShare &ws = reinterpret_cast<WaveShare *>(lds_bytes + (size_t)blockDim.x * lds_stride)[threadIdx.x >> 6];
    LaneCtx c;
    init_ctx(c, A->B, gl);
    c.sstride = 1;  // persistent lanes own contiguous runs
    c.cstride = 1;
    u4 *const own_cand = c.cand;
    uint8_t *const own_pd = c.pd;

    // A batch of fewer reads than the grid has lanes is spread evenly: each
    // wave takes `cap` reads at once, at its first refill, and its other lanes
    // help from the start (the endgame's sharing), so that every wave of the
    // device works on it.  With 64 reads to a wave, 60 k reads ran on 940 of
    // 4096 waves, each 1.7 k iterations long.  (25 k reads of 36 bases, every
    // placement within 2 mismatches: 9.6 -> 2.3 ms; 30 k pairs of 100 bases,
    // aligned, paired and rescued: 16.0 -> 8.4 ms; batches of more reads than
    // lanes take 64 at a time as before and keep their time.)  2000
    // reads of 250 bases: 16.9 -> 9.4 ms.
    const uint32_t n_waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t cap = min((n_reads + n_waves - 1) / n_waves, 64u);
    int phase = PZ_IDLE;
    bool exhausted = (uint32_t)lane >= cap;
    bool endgame = false;  // wave-uniform: the batch's reads are all taken
    bool drain = false;    // wave-uniform: most of the grid has ended
    uint32_t eg_iter = 0;
    int ow = lane;         // owner lane of the read this lane works on
    uint32_t r = 0;
    int m = 0, maxd = 0, strand = 0;
    bool has_n = false;   // the read holds an N
    bool two = false;     // strand - is searched too
    // search state
    u4 cur = mk4(0, 0, 0, 0);
    bool valid = false;
    Seed S{0, 0, 0};
    // work statistics (measurement only)
    uint32_t w_iters = 0, w_busy = 0, w_query = 0;  // per lane: far below 2^32 per launch

    for (;;) {
        // an opaque step on the pointer keeps the argument loads inside the
        // loop, next to their uses
        asm volatile("" : "+s"(Ag));
        A = (const PersistentArgs *)Ag;
        const ReadsView &rd = A->rd;
        const ReadOut &O = A->O;
        uint32_t *const next_read = A->next_read;
        // lanes whose strand or read has ended, and idle ones while reads are
        // left, once enough of them wait (in the endgame, at once)
        const bool turn = phase == PZ_TURN || (phase == PZ_IDLE && !exhausted);
        const unsigned long long tm = __ballot(turn);
        if (tm && (endgame || __popcll(tm) >= BWFM_TURN_MIN || __ballot(phase >= PZ_SEARCH) == 0)) {
            bool load = false;
            if (phase == PZ_TURN) {
                const int fl = sh_ld(&ws.flags[lane]);
                if (fl & SH_FAIL) {
                    if (fl >> SH_SLOT_SHIFT)
                        end_split_read(A->X, c, fl);
                    else
                        send_to_second_pass(O, r);
                    if (O.expand) O.expand[r] = c.expand + (uint32_t)sh_ld(&ws.hexp[lane]);
                    phase = PZ_IDLE;
                } else if (strand == 0 && two) {
                    strand = 1;
                    load = true;
                } else {
                    c.ncand = (uint32_t)sh_ld(&ws.ncand[lane]);
                    const int sb = sh_ld(&ws.best[lane]);
                    if (sb < c.best) c.best = sb;
                    c.cand = own_cand;
                    c.expand += (uint32_t)sh_ld(&ws.hexp[lane]);
                    if (fl >> SH_SLOT_SHIFT)
                        end_split_read(A->X, c, fl);
                    else
                        publish(c, P, O, r, (fl & SH_HELPED) ? (uint8_t)BWFM_ST_SHARED : (uint8_t)0);
                    phase = PZ_IDLE;
                }
            }
            const bool want = phase == PZ_IDLE && !exhausted;
            const unsigned long long wm = __ballot(want);
            if (wm) {
                const int leader = __ffsll(wm) - 1;
                uint32_t base = 0;
                if (lane == leader) base = atomicAdd(as_global(next_read), (uint32_t)__popcll(wm));
                base = __shfl(base, leader);
                if (want) {
                    const uint32_t rr = base + (uint32_t)__popcll(wm & ((1ULL << lane) - 1));
                    if (rr >= n_reads) {
                        exhausted = true;
                    } else {
                        r = rr;
                        uint64_t o0;
                        if (!check_read(rd, P, O, r, m, maxd, o0)) {
                            ow = lane;
                            c.pd = own_pd;
                            c.cand = own_cand;
                            c.ncand = 0;
                            c.best = INF_SCORE;
                            c.expand = 0;
                            // the first strand the pre-pass left searchable,
                            // or nothing to search
                            const int dfl = as_global(A->dflag)[r];
                            has_n = (dfl & 4) != 0;
                            two = (dfl & 2) == 0;
                            strand = (dfl & 1) ? 1 : 0;
                            load = (dfl & 3) != 3;
                            if (!load) publish(c, P, O, r);
                            S = seed_of(P, m);
                            sh_st(&ws.best[lane], INF_SCORE);
                            sh_st(&ws.ncand[lane], 0);
                            sh_st(&ws.pending[lane], 0);
                            sh_st(&ws.flags[lane], 0);
                            sh_st(&ws.hexp[lane], 0);
                            if (A->X.budget) A->lane_read[gl] = r;
                        }
                    }
                }
            }
            if (cap < 64) exhausted = true;
            if (load) {
                load_drow(own_pd, drow_of(A->drows, A->dstride, r, strand), m);
                phase = PZ_SEARCH;
                cur = root_state(ix, m, P.minc * pd_d(c, m - 1));
                valid = true;
                c.sp = c.sbase = 0;
            }
        }
        if (__ballot(phase != PZ_IDLE) == 0) {
            if (__ballot(!exhausted) == 0) break;
            continue;
        }
        endgame = endgame || __ballot(exhausted) != 0;
        if (O.work) {
            w_iters++;
            w_busy += phase == PZ_SEARCH || phase == PZ_HELP;
        }

        if (endgame) {
            wave_fence();
            const bool searching = phase == PZ_SEARCH || phase == PZ_HELP;
            if (searching) {
                const int sb = sh_ld(&ws.best[ow]);
                if (sb < c.best) c.best = sb;
                if (sh_ld(&ws.flags[ow]) & SH_FAIL) {
                    // the read goes to the second pass: drop this lane's part
                    valid = false;
                    c.sp = c.sbase = 0;
                }
            }
            // hand the oldest pending state of busy lanes to idle lanes
            const int avail = searching ? (int)(c.sp - c.sbase) - (valid ? 0 : 1) : 0;
            const bool give = avail >= 1;
            const bool recv = phase == PZ_IDLE;
            const unsigned long long R = __ballot(recv), G = __ballot(give);
            if (R && G) {
                const int n = min(__popcll(R), __popcll(G));
                const unsigned long long lt = (1ULL << lane) - 1;
                if (give) {
                    const int gi = __popcll(G & lt);
                    if (gi < n) {
                        ws.box[gi] = c.stack[(size_t)c.sbase * c.sstride];
                        ws.meta[gi] = (uint32_t)ow | ((uint32_t)strand << 6) | ((uint32_t)maxd << 7) |
                                      ((uint32_t)m << 11) | ((uint32_t)has_n << 21);
                        c.sbase++;
                        atomicAdd(&ws.pending[ow], 1);
                        atomicOr(&ws.flags[ow], SH_HELPED);
                    }
                }
                wave_fence();
                if (recv) {
                    const int ri = __popcll(R & lt);
                    if (ri < n) {
                        cur = ws.box[ri];
                        const uint32_t mt = ws.meta[ri];
                        ow = (int)(mt & 63);
                        strand = (int)((mt >> 6) & 1);
                        maxd = (int)((mt >> 7) & 15);
                        m = (int)((mt >> 11) & 1023);
                        has_n = (mt >> 21) != 0;
                        S = seed_of(P, m);
                        valid = true;
                        c.sp = c.sbase = 0;
                        c.pd = lds_bytes + (size_t)(wave0 + ow) * lds_stride;
                        c.cand = own_cand + ((int)ow - lane) * (ptrdiff_t)FAST_CAND;
                        c.best = sh_ld(&ws.best[ow]);
                        c.expand = 0;
                        phase = PZ_HELP;
                    }
                }
                wave_fence();
            }
            // a part past the budget goes to the split searches, one lane
            // of the wave at a time (a read's slot is taken once); a part's
            // expansions count from the read's start for its owner and from
            // the hand-over for a helper
            uint32_t bud = A->X.budget;
            if (bud) {
                if ((eg_iter++ & 15) == 15 && !drain) drain = ld_agent(&A->X.ctl[SPLIT_DONE]) >= A->X.drain;
                if (drain) bud = min(bud, DRAIN_BUDGET);
                const bool want = (phase == PZ_SEARCH || phase == PZ_HELP) && c.sp > c.sbase && c.expand >= bud &&
                                  !(sh_ld(&ws.flags[ow]) & (SH_FAIL | SH_NOSPLIT));
                unsigned long long sm = __ballot(want);
                while (sm) {
                    const int L = __ffsll(sm) - 1;
                    if (lane == L) {
                        int fl = sh_ld(&ws.flags[ow]);
                        const uint32_t og = gl - (uint32_t)lane + (uint32_t)ow;  // the owner's global lane
                        const uint32_t rr = ow == lane ? r : A->lane_read[og];
                        if (split_part(A->X, rr, og, strand, m, maxd, has_n, sh_ld(&ws.best[ow]), c, cur, valid, fl))
                            valid = false;  // the lane's part is over
                        else
                            fl |= SH_NOSPLIT;  // no room: the read's parts go on in the wave
                        sh_st(&ws.flags[ow], fl);
                    }
                    wave_fence();
                    sm &= sm - 1;
                }
            }
        }

        // decide this lane's action and rank queries; a lane that changes
        // phase here acts in its new phase from the next iteration on
        bool go = false;  // cur takes a step
        bool hit = false;
        bool part_done = false;  // this lane's part of the strand's search is over
        if (phase == PZ_SEARCH || phase == PZ_HELP) {
            int rr = resolve(cur, valid, strand, P, c, PH_FAST, POPS_PER_STEP, ix, endgame);
            if (rr == 2) {
                // pop limit reached: keep popping next iteration
            } else if (rr == 3) {
                hit = true;
            } else if (rr < 0) {
                // only without endgame, so the lane owns its read alone
                send_to_second_pass(O, r);
                if (O.expand) O.expand[r] = c.expand;
                phase = PZ_IDLE;
            } else if (rr == 0) {
                part_done = true;
            }
            go = rr == 1;
            if (!endgame && phase == PZ_SEARCH) {
                sh_st(&ws.best[lane], c.best);
                sh_st(&ws.ncand[lane], (int)c.ncand);
            }
        }

        // completed hits found in the endgame, one lane at a time: lanes of
        // one read share its hit buffer
        if (endgame) {
            unsigned long long hm = __ballot(hit);
            while (hm) {
                const int L = __ffsll(hm) - 1;
                if (lane == L) {
                    c.ncand = (uint32_t)sh_ld(&ws.ncand[ow]);
                    const int sb = sh_ld(&ws.best[ow]);
                    if (sb < c.best) c.best = sb;
                    const int score = s_score(cur);
                    if (score < c.best) c.best = score;
                    const u2 kl = state_kl(ix, strand, cur);
                    const int rc = record(c, P,
                                          make_hit(strand, kl.x, kl.y, s_len(cur), score, s_nmm(cur), s_ngo(cur),
                                                   s_nge(cur)),
                                          PH_FAST);
                    sh_st(&ws.best[ow], c.best);
                    sh_st(&ws.ncand[ow], (int)c.ncand);
                    if (rc) {
                        atomicOr(&ws.flags[ow], SH_FAIL);
                        c.sp = c.sbase = 0;
                        part_done = true;
                    }
                    valid = false;
                }
                wave_fence();
                hm &= hm - 1;
            }
        }

        // the end of a lane's part: a helper reports back; an owner waits
        // for its helpers before the next strand or the publication
        if (part_done) {
            valid = false;
            c.sp = c.sbase = 0;
            if (phase == PZ_HELP) {
                atomicAdd(&ws.hexp[ow], (int)c.expand);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                atomicSub(&ws.pending[ow], 1);
                phase = PZ_IDLE;
            } else {
                phase = PZ_WAIT;
            }
        }
        if (phase == PZ_WAIT && sh_ld(&ws.pending[lane]) == 0) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            phase = PZ_TURN;
        }

        const DevDir qd = pick_dir(ix, strand == 0 ? 1 : 0);
        if (O.work) w_query += go;
        if (search_step<LW>(ix, qd, strand == 0 ? 1 : 0, go, cur, valid, m, maxd, has_n, S, P, c)) {
            // cannot happen with worst-case stacks; kept as a guard
            if (endgame) {
                atomicOr(&ws.flags[ow], SH_FAIL);  // every lane of the read drops out
            } else {
                send_to_second_pass(O, r);
                if (O.expand) O.expand[r] = c.expand;
                phase = PZ_IDLE;
            }
        }
    }
    if (A->X.budget && lane == 0) atomicAdd(as_global(&A->X.ctl[SPLIT_DONE]), 1u);
    if (A->O.work) {
        if (lane == 0) atomicAdd(&A->O.work[0], (unsigned long long)w_iters);
        atomicAdd(&A->O.work[1], (unsigned long long)w_busy);
        atomicAdd(&A->O.work[2], (unsigned long long)w_query);
    }
}

// Two builds of the batched kernel: the compiler's own register budget
// and one held to 128 VGPRs so that 4 waves stay resident per SIMD.  What
// bounds the search is the latency of its random accesses: a wave waits in
// each iteration for the slowest of 64 lanes' chains of one to three dependent
// loads out of tables, suffix arrays and stacks that together span gigabytes,
// and only other waves' loads fill that time.  2M reads of 100 bases on 100
// Mbp take 57 ms at 4 waves per SIMD, 65 at 3, 82 at 2 and 139 at 1.  The
// autotuner picks.
template <int LW>
__global__ __launch_bounds__(BLOCK) void k_align_persistent(DevIndex ix, Params P, const PersistentArgs *A) {
    persistent_body<LW>(ix, P, A);
}
template <int LW>
__global__ __launch_bounds__(BLOCK, 4) void k_align_persistent4(DevIndex ix, Params P, const PersistentArgs *A) {
    persistent_body<LW>(ix, P, A);
}

using PersistentKernel = void (*)(DevIndex, Params, const PersistentArgs *);

// the build serving a waves_per_simd setting: 0 and >= 4 take the 4-wave
// build, 1-3 the compiler's own
template <int LW>
PersistentKernel persistent_kernel(int waves_per_simd) {
    return (waves_per_simd == 0 || waves_per_simd >= 4) ? k_align_persistent4<LW> : k_align_persistent<LW>;
}

// Arguments of the task rounds, kept in device memory like PersistentArgs.
struct TaskArgs {
    LaneBufs B;
    SplitBufs X;
};

__global__ void k_set_task_args(TaskArgs *dst, TaskArgs a) {
    if (threadIdx.x == 0) *dst = a;
}

// One round of split searches: a persistent grid whose lanes take the
// tasks of generation g from a counter, one atomic per wave as the batched
// kernel takes reads.  A task is one state of a split read: its subtree is
// searched depth-first on the lane's own stack with the slot's row (read in
// place, so the kernel needs no LDS and as many lanes as its registers
// allow), budget and best score, one rank-query pair per lane and
// iteration.  Once the
// round's tasks are all taken (drain set), a lane that has expanded at
// least DRAIN_MIN states of its task hands its pending states to
// generation g + 1, so that the round ends soon and the next one spreads
// them over the grid; the last round has no drain.  At a task's end its
// hits go to the slot.
constexpr uint32_t DRAIN_MIN = 256;
// Idle lanes of a wave that make it take new tasks: few while a round holds
// TASK_MANY and more tasks for each lane of its grid, when the idle lanes cost
// most (2M reads of 250 bases at 10 / 32: 377 / 397 ms at the default split
// budget, 294 / 331 at 512), else half, so that a short round's tasks do not
// end up on few waves (150 k reads: 57 / 52 ms)
constexpr int TASK_REFILL_MANY = 10, TASK_REFILL = 32;
constexpr uint32_t TASK_MANY = 8;
// Waves per SIMD of the rounds.  Five (96 registers; the planar formats of 64
// and 128 bytes hold more and would spill) suit the long rounds of a batch of
// many reads, whose random fills they keep in flight; in short rounds they only
// cut the tasks finer, so a batch of fewer than TASK_READS reads a lane takes
// the lanes of four (128-byte sub-counted lines, 250 bases, 4 / 5 waves: 2M at
// a split budget of 512 293 / 273 ms, 1M 169 / 160, 600 k 150 / 150, 300 k 84 /
// 86, 150 k 53.9 / 55.9).  At 64-byte sub-counted lines five take 100 k reads
// as fast as four (40.3 / 41.5 ms).  The body as a function of its own takes 92
// registers at 128-byte sub-counted lines, as the kernel itself 100.
constexpr int TASK_WAVES = 5, TASK_WAVES_FEW = 4;
constexpr uint32_t TASK_READS = 2;
template <int LW>
__device__ __forceinline__ void tasks_body(const DevIndex &ix, const Params &P, const TaskArgs *Aarg, uint32_t g,
                                           uint32_t drain) {
    using GlobalArgs = const __attribute__((address_space(1))) TaskArgs;
    GlobalArgs *Ag = (GlobalArgs *)Aarg;
    const TaskArgs *A = (const TaskArgs *)Ag;
    const uint32_t ntask = min(ld_agent(&A->X.ctl[1 + g]), A->X.task_cap);
    if (ntask == 0) return;  // the whole grid: nothing was split
    const int lane = threadIdx.x & 63;
    const int refill = ntask / TASK_MANY >= gridDim.x * BLOCK ? TASK_REFILL_MANY : TASK_REFILL;
    LaneCtx c;
    init_ctx(c, A->B, blockIdx.x * blockDim.x + threadIdx.x);
    c.sstride = 1;
    c.cstride = 1;
    bool busy = false, exhausted = false, valid = false;
    bool drained = false;  // wave-uniform: the round's tasks are all taken
    uint32_t s = 0, texp = 0, witer = 0;
    int strand = 0, m = 0, maxd = 0;
    bool has_n = false;
    u4 cur = mk4(0, 0, 0, 0);
    Seed S{0, 0, 0};
    for (;;) {
        asm volatile("" : "+s"(Ag));
        A = (const TaskArgs *)Ag;
        const SplitBufs &X = A->X;
        witer++;
        // a wave learns that the round's tasks are all taken when one of
        // its lanes finds none left, else from one load of the counter
        // every 64 iterations (the same address for the whole wave)
        if (drain && !drained && (witer & 63) == 0) drained = ld_agent(&X.ctl[2 + SPLIT_ROUNDS + g]) >= ntask;
        // every 64 iterations, at once for the wave (lanes on one read share
        // the load), the bound takes the best score any part has found
        if ((witer & 63) == 32 && busy) {
            const int sb = (int)ld_agent(reinterpret_cast<const uint32_t *>(&X.slot_best[s]));
            if (sb < c.best) c.best = sb;
        }
        // idle lanes take the next tasks, one atomic per wave, once
        // `refill` lanes of the wave are idle (or none is busy): tasks
        // end every few hundred expansions, and one counter taken by every
        // wave at that rate held the rounds to half their speed
        const bool idle = !busy && !exhausted;
        const unsigned long long im = __ballot(idle);
        const bool bulk = __popcll(im) >= refill || __ballot(busy) == 0;
        const bool want = idle && bulk;
        const unsigned long long wm = bulk ? im : 0ull;
        uint32_t t = 0;
        if (wm) {
            const int leader = __ffsll(wm) - 1;
            uint32_t base = 0;
            if (lane == leader) base = atomicAdd(&X.ctl[2 + SPLIT_ROUNDS + g], (uint32_t)__popcll(wm));
            base = __shfl(base, leader);
            t = base + (uint32_t)__popcll(wm & ((1ULL << lane) - 1));
            if (want && t >= ntask) exhausted = true;
        }
        if (want && !exhausted) {
            const uint32_t ref = as_global(X.task_ref[g & 1])[t];
            // unused entries and the parts of failed reads are skipped (a
            // stale flag only costs the work)
            if (ref != TASK_EMPTY && !as_global(X.slot_fail)[ref & 0x7fffffffu]) {
                s = ref & 0x7fffffffu;
                strand = (int)(ref >> 31);
                const uint32_t meta = as_global(X.slot_meta)[s];
                m = (int)(meta & 1023);
                maxd = (int)((meta >> 10) & 15);
                has_n = (meta >> 14) != 0;
                // the slot's row, read in place: the tasks of one read share
                // it in the caches
                c.pd = as_global(X.slot_rows + ((size_t)s * 2 + (size_t)strand) * X.dstride);
                cur = as_global(X.tasks[g & 1])[t];
                valid = true;
                c.sp = c.sbase = 0;
                c.ncand = 0;
                c.best = as_global(X.slot_best)[s];  // a stale value only prunes less
                c.expand = 0;
                texp = 0;
                S = seed_of(P, m);
                busy = true;
            }
        }
        if (__ballot(busy) == 0) {
            if (__ballot(!exhausted) == 0) break;
            continue;
        }
        drained = drained || __ballot(exhausted) != 0;
        bool query = false, done = false;
        if (busy) {
            const int rr = resolve(cur, valid, strand, P, c, PH_FAST, POPS_PER_STEP, ix, true);
            if (rr == 3) {
                // a completed hit; a better score is shared with the read's
                // other parts at once, a full buffer is first delivered
                const int score = s_score(cur);
                if (score < c.best) {
                    c.best = score;
                    atomicMin(&X.slot_best[s], score);
                }
                const u2 kl = state_kl(ix, strand, cur);
                const u4 h = make_hit(strand, kl.x, kl.y, s_len(cur), score, s_nmm(cur), s_ngo(cur), s_nge(cur));
                if (record(c, P, h, PH_FAST)) {
                    flush_slot(X, P, s, c);
                    if (record(c, P, h, PH_FAST)) {
                        atomicOr(&X.slot_fail[s], 1u);
                        done = true;
                    }
                }
                valid = false;
            } else if (rr == 0) {
                done = true;
            } else if (rr == 1) {
                if (drain && drained && texp >= DRAIN_MIN && c.sp > c.sbase) {
                    uint32_t off = 0;
                    if (take_tasks(X, g + 1, task_count(c, cur, true), off)) {
                        put_tasks(X, g + 1, off, s | ((uint32_t)strand << 31), c, cur, true);
                        valid = false;
                        done = true;
                    }
                }
                query = !done;
            }
            // rr == 2: the pop limit; popping goes on next iteration
        }
        const DevDir qd = pick_dir(ix, strand == 0 ? 1 : 0);
        const uint32_t e0 = c.expand;
        if (search_step<LW>(ix, qd, strand == 0 ? 1 : 0, query, cur, valid, m, maxd, has_n, S, P, c)) {
            atomicOr(&X.slot_fail[s], 1u);  // cannot happen with worst-case stacks; kept as a guard
            done = true;
        }
        texp += c.expand - e0;
        if (done) {
            flush_slot(X, P, s, c);
            busy = false;
            valid = false;
        }
    }
}

template <int LW>
__global__ __launch_bounds__(BLOCK, LW == 16 || LW == 32 ? TASK_WAVES_FEW : TASK_WAVES) void k_align_tasks(
    DevIndex ix, Params P, const TaskArgs *A, uint32_t g, uint32_t drain) {
    tasks_body<LW>(ix, P, A, g, drain);
}

// Totals of the split searches for the work counters (work[3..5] start at
// zero): reads split, task entries handed out over all generations, split
// reads sent on to the second pass; then per generation the entries asked
// for (above the room when some found none).  One thread per slot.
__global__ void k_split_stats(SplitBufs X, unsigned long long *work) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t ns = min(X.ctl[0], X.slot_cap);
    if (s == 0) {
        unsigned long long t = 0;
        for (int g = 0; g <= SPLIT_ROUNDS; g++) t += min(X.ctl[1 + g], X.task_cap);
        work[3] = ns;
        work[4] = t;
        for (int g = 0; g < SPLIT_ROUNDS; g++) work[6 + g] = X.ctl[1 + g];
    }
    if (s < ns && (X.slot_fail[s] || X.slot_nhit[s] > SLOT_HITS)) atomicAdd(&work[5], 1ull);
}

// Second pass for the reads listed in slow_list (*O.n_slow of them, set by
// the first pass): a fixed grid pulls them from a counter.  Each read gets
// the worst-case stack; first the best score S*, then the hits with the
// bound fixed at S* + s_mm.  The reported hits go to the staging arena like
// the first pass's.
template <int LW>
__global__ __launch_bounds__(BLOCK) void k_align_slow(DevIndex ix, ReadsView rd, Params P, LaneBufs B, ReadOut O,
                                                      uint32_t *slow_next) {
    const uint32_t gl = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t ns = *O.n_slow;
    if (blockIdx.x * blockDim.x >= ns) return;  // the whole block has nothing to take
    LaneCtx c;
    init_ctx(c, B, gl);
    for (;;) {
        const uint32_t t = atomicAdd(slow_next, 1u);
        if (t >= ns) break;
        const uint32_t r = O.slow_list[t];
        uint64_t o0, len;
        bool bad;
        read_span(rd, r, o0, len, bad);
        const int m = (int)len;
        const int maxd = rd.maxd ? rd.maxd[r] : P.max_diff;
        c.expand = 0;
        c.best = INF_SCORE;
        align_read<LW>(ix, rd.bases + o0, m, maxd, P, c, PH_BEST);
        uint8_t st = 0;
        uint32_t a = 0, b = 0, nr = 0;
        if (c.best != INF_SCORE) {
            const int rc = align_read<LW>(ix, rd.bases + o0, m, maxd, P, c, PH_COLLECT);
            if (rc == R_CAND) {
                st = BWFM_ST_OVERFLOW;
                a = b = 0xffffffffu;
            } else {
                nr = finish(c, P, st, a, b);
            }
        }
        stage_hits(c, O, r, nr);
        O.n_rep[r] = nr;
        O.status[r] = st | ST_RESEARCH;
        O.c1[r] = a;
        O.c2[r] = b;
        if (O.expand) O.expand[r] += c.expand;
    }
}

// Copy each read's reported hits from the staging arena to the CSR output.
// Launched only when the output holds them all.
__global__ void k_compact(uint32_t n, const uint64_t *hoff, const u4 *stage, const uint64_t *stage_off,
                          u4 *hits, const uint64_t *n_dev, const uint32_t *err) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (err && *err) return;  // the output cannot hold the hits
    if (r >= count_of(n, n_dev)) return;
    const uint64_t o = hoff[r], e = hoff[r + 1];
    if (e == o) return;
    const u4 *src = stage + stage_off[r];
    for (uint64_t j = 0; j < e - o; j++) hits[o + j] = src[j];
}

// Fill n words with v (used instead of a memset node, so that a captured
// sequence replays it reliably).
__global__ void k_fill_u32(uint32_t *p, uint32_t n, uint32_t v) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ exclusive scan (u32 counts -> u64 offsets)

constexpr int SCAN_BLOCK = 1024;

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_reduce(const uint32_t *in, uint64_t n, uint64_t *part,
                                                            const uint64_t *n_dev) {
    __shared__ uint64_t s[SCAN_BLOCK / 64];
    n = count_of(n, n_dev);
    uint64_t i = (uint64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x;
    uint64_t v = i < n ? in[i] : 0;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int w = 0; w < SCAN_BLOCK / 64; w++) t += s[w];
        part[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_parts(uint64_t *part, uint64_t nb) {
    // exclusive scan of nb block sums by one workgroup, in chunks
    __shared__ uint64_t s[SCAN_BLOCK];
    __shared__ uint64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint64_t base = 0; base < nb; base += SCAN_BLOCK) {
        uint64_t i = base + threadIdx.x;
        uint64_t v = i < nb ? part[i] : 0;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < SCAN_BLOCK; o <<= 1) {
            uint64_t t = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0;
            __syncthreads();
            s[threadIdx.x] += t;
            __syncthreads();
        }
        uint64_t incl = s[threadIdx.x];
        if (i < nb) part[i] = carry + incl - v;
        __syncthreads();
        if (threadIdx.x == SCAN_BLOCK - 1) carry += incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) part[nb] = carry;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_apply(const uint32_t *in, uint64_t n, const uint64_t *part,
                                                           uint64_t *out, const uint64_t *n_dev) {
    __shared__ uint64_t s[SCAN_BLOCK];
    n = count_of(n, n_dev);
    uint64_t i = (uint64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x;
    if (n == 0) {
        if (i == 0) out[0] = 0;
        return;
    }
    uint64_t v = i < n ? in[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < SCAN_BLOCK; o <<= 1) {
        uint64_t t = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0;
        __syncthreads();
        s[threadIdx.x] += t;
        __syncthreads();
    }
    if (i < n) out[i] = part[blockIdx.x] + s[threadIdx.x] - v;
    if (i == n - 1) out[n] = part[blockIdx.x] + s[threadIdx.x];
}

// ------------------------------------------------------------------ locate

// per hit: number of positions to locate (width if <= max_occ, else 0)
__global__ void k_loc_count(uint64_t n_hits, const u4 *hits, uint32_t max_occ, uint32_t *cnt,
                            const uint64_t *n_dev) {
    uint64_t h = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= count_of(n_hits, n_dev)) return;
    u4 x = hits[h];
    uint64_t w = (uint64_t)x.y - x.x + 1;
    cnt[h] = (x.x <= x.y && w <= max_occ) ? (uint32_t)w : 0;
}

// position p of the located hits: its hit is the last h with poff[h] <= p
template <int LW>
__device__ void locate_one(const DevIndex &ix, uint64_t n_hits, const u4 *hits, const uint64_t *poff, uint64_t p,
                           uint32_t *pos) {
    uint64_t lo = 0, hi = n_hits;
    while (hi - lo > 1) {
        uint64_t mid = (lo + hi) / 2;
        if (poff[mid] <= p) lo = mid;
        else hi = mid;
    }
    u4 x = hits[lo];
    int strand = h_strand(x);
    const DevDir d = pick_dir(ix, strand == 0 ? 1 : 0);
    uint32_t j = x.x + (uint32_t)(p - poff[lo]);
    uint32_t steps = 0;
    const uint32_t smask = (1u << ix.sa_shift) - 1;
    uint32_t q;
    for (;;) {
        if (j == d.primary) { q = steps; break; }
        if ((j & smask) == 0) { q = d.sa[j >> ix.sa_shift] + steps; break; }
        j = lf_step<LW>(ix, d, j);
        steps++;
    }
    pos[p] = strand == 0 ? ix.n - q - (uint32_t)h_len(x) : q;
}

// one lane per position (grid-stride): find its hit, walk LF to a sampled row
template <int LW>
__global__ void k_loc_rows(DevIndex ix, uint64_t n_hits, const u4 *hits, const uint64_t *poff, uint64_t total,
                           uint32_t *pos, const uint64_t *n_hits_dev, const uint64_t *total_dev) {
    n_hits = count_of(n_hits, n_hits_dev);
    total = count_of(total, total_dev);
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (uint64_t)gridDim.x * blockDim.x)
        locate_one<LW>(ix, n_hits, hits, poff, p, pos);
}
// With the whole suffix array on the device a position is one load: one lane
// per hit, wide hits (more than LOC_LANE rows) by their wave, the widest (more
// than LOC_WAVE) listed for k_loc_wide.  The walk above takes a binary search
// over the hits and sa_sample rank lines on average for each position:
// 400 k reads of 36 bases located in 537 us with it, 175 us with this.
// A total of 0 means that the positions do not fit: nothing is written.
constexpr uint32_t LOC_LANE = 8, LOC_WAVE = 2048;
__device__ __forceinline__ uint32_t hit_pos(const DevIndex &ix, const uint32_t *full, u4 x, uint32_t t) {
    const uint32_t q = full[x.x + t];
    return h_strand(x) == 0 ? ix.n - q - (uint32_t)h_len(x) : q;
}
__global__ __launch_bounds__(256) void k_loc_hits(DevIndex ix, uint64_t n_hits, const u4 *hits, const uint64_t *poff,
                                                  uint32_t *pos, uint32_t *wide, uint32_t *n_wide,
                                                  const uint64_t *n_hits_dev, const uint64_t *total_dev) {
    const uint64_t h = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (total_dev && *total_dev == 0) return;
    uint64_t o = 0;
    uint32_t w = 0;
    u4 x = mk4(0, 0, 0, 0);
    if (h < count_of(n_hits, n_hits_dev)) {
        o = poff[h];
        w = (uint32_t)(poff[h + 1] - o);
        x = hits[h];
    }
    if (w && w <= LOC_LANE) {
        const uint32_t *full = h_strand(x) == 0 ? ix.dir[1].full : ix.dir[0].full;
        for (uint32_t t = 0; t < w; t++) pos[o + t] = hit_pos(ix, full, x, t);
    }
    if (w > LOC_WAVE) wide[atomicAdd(n_wide, 1u)] = (uint32_t)h;
    unsigned long long todo = __ballot(w > LOC_LANE && w <= LOC_WAVE);
    while (todo) {
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const uint64_t so = __shfl((unsigned long long)o, src);
        const uint32_t sw = __shfl(w, src);
        const u4 sx = mk4(__shfl(x.x, src), __shfl(x.y, src), __shfl(x.z, src), __shfl(x.w, src));
        const uint32_t *full = h_strand(sx) == 0 ? ix.dir[1].full : ix.dir[0].full;
        for (uint32_t t = threadIdx.x & 63; t < sw; t += 64) pos[so + t] = hit_pos(ix, full, sx, t);
    }
}
// the listed hits, each by the whole grid
__global__ __launch_bounds__(256) void k_loc_wide(DevIndex ix, const u4 *hits, const uint64_t *poff, uint32_t *pos,
                                                  const uint32_t *wide, const uint32_t *n_wide) {
    const uint32_t n = *n_wide;
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t h = wide[i];
        const uint64_t o = poff[h], w = poff[h + 1] - o;
        const u4 x = hits[h];
        const uint32_t *full = h_strand(x) == 0 ? ix.dir[1].full : ix.dir[0].full;
        for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t < w; t += (uint64_t)gridDim.x * blockDim.x)
            pos[o + t] = hit_pos(ix, full, x, (uint32_t)t);
    }
}

// sort each hit's positions: short segments by one lane, long ones by a
// workgroup running a bitonic network (pairs past the end count as +inf).
// A total of 0 means that the positions do not fit, as above: poff then
// reaches past pos, and nothing is sorted (n_big stays 0).
__global__ void k_sort_small(uint64_t n_hits, const uint64_t *poff, uint32_t *pos, uint32_t *big, uint32_t *n_big,
                             const uint64_t *n_dev, const uint64_t *total_dev) {
    uint64_t h = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (total_dev && *total_dev == 0) return;
    if (h >= count_of(n_hits, n_dev)) return;
    uint64_t o = poff[h], w = poff[h + 1] - o;
    if (w <= 1) return;
    if (w > 32) {
        big[atomicAdd(n_big, 1u)] = (uint32_t)h;
        return;
    }
    uint32_t *a = pos + o;
    for (uint64_t i = 1; i < w; i++) {
        uint32_t v = a[i];
        uint64_t q = i;
        while (q > 0 && a[q - 1] > v) { a[q] = a[q - 1]; q--; }
        a[q] = v;
    }
}

__global__ __launch_bounds__(256) void k_sort_big(const uint64_t *poff, uint32_t *pos, const uint32_t *big,
                                                  const uint32_t *n_big) {
    __shared__ uint32_t s[4096];
    const uint32_t nb = *n_big;
    for (uint32_t b = blockIdx.x; b < nb; b += gridDim.x) {
        uint32_t h = big[b];
        uint64_t o = poff[h], n = poff[h + 1] - o;
        uint32_t *a = pos + o;
        const bool lds = n <= 4096;
        if (lds) {
            for (uint64_t i = threadIdx.x; i < n; i += blockDim.x) s[i] = a[i];
            __syncthreads();
        }
        uint32_t *x = lds ? s : a;
        for (uint64_t k = 2; k < 2 * n; k <<= 1) {
            for (uint64_t j = k >> 1; j > 0; j >>= 1) {
                for (uint64_t i = threadIdx.x; i < n; i += blockDim.x) {
                    uint64_t q = (j == (k >> 1)) ? (i ^ (k - 1)) : (i ^ j);
                    if (q > i && q < n && x[i] > x[q]) {
                        uint32_t t = x[i];
                        x[i] = x[q];
                        x[q] = t;
                    }
                }
                __syncthreads();
            }
        }
        if (lds) {
            for (uint64_t i = threadIdx.x; i < n; i += blockDim.x) a[i] = s[i];
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ pairing

struct EndView {
    const uint64_t *hoff;
    const u4 *hits;
    const uint64_t *poff;  // per hit, indexed by (hit index - hbase)
    const uint32_t *pos;
    uint64_t hbase;        // hoff[0]
};

__device__ __forceinline__ uint64_t lower_bound(const uint32_t *a, uint64_t n, uint64_t v) {
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        uint64_t mid = (lo + hi) / 2;
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// single-end primary: smallest (score, diffs, strand, pos, len)
__device__ bool se_primary(const EndView &e, uint32_t q, uint32_t &pos, u4 &hit, bool &rep) {
    bool found = false;
    rep = false;
    for (uint64_t i = e.hoff[q]; i < e.hoff[q + 1]; i++) {
        uint64_t o = e.poff[i - e.hbase], w = e.poff[i - e.hbase + 1] - o;
        if (w == 0) { rep = true; continue; }
        u4 h = e.hits[i];
        uint32_t p = e.pos[o];  // sorted: the first is the smallest
        bool b;
        if (!found) b = true;
        else if (h_score(h) != h_score(hit)) b = h_score(h) < h_score(hit);
        else if (h_diffs(h) != h_diffs(hit)) b = h_diffs(h) < h_diffs(hit);
        else if (h_strand(h) != h_strand(hit)) b = h_strand(h) < h_strand(hit);
        else if (p != pos) b = p < pos;
        else b = h_len(h) < h_len(hit);
        if (b) { found = true; pos = p; hit = h; }
    }
    return found;
}

// One lane per pair.  With n_dev, the pair count is read on the device and
// end 2's reads follow end 1's in one batch (its offsets start at
// e1.hoff + n); a nonzero *err (an output was too small) makes every record
// that of an unplaced pair, which mate rescue and MAPQ launched after it
// leave alone (the hit offsets may then reach past the hits).
__global__ void k_pair(uint32_t n_pairs, EndView e1, EndView e2, int paired, int32_t lo, int32_t hi, int32_t mu,
                       bwfm_pair *out, const uint64_t *n_dev, const uint32_t *err) {
    uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (n_dev) {
        n_pairs = (uint32_t)count_of(n_pairs, n_dev);
        e2.hoff = e1.hoff + n_pairs;
    }
    if (q >= n_pairs) return;
    bwfm_pair o;
    memset(&o, 0, sizeof(o));
    o.pos1 = o.pos2 = 0xffffffffu;
    if (err && *err) {
        out[q] = o;
        return;
    }
    bool found = false;
    int64_t bs = 0, bd = 0, bpf = 0;
    if (paired) {
        for (uint64_t i = e1.hoff[q]; i < e1.hoff[q + 1]; i++) {
            u4 h1 = e1.hits[i];
            const uint32_t *P1 = e1.pos + e1.poff[i - e1.hbase];
            uint64_t n1 = e1.poff[i - e1.hbase + 1] - e1.poff[i - e1.hbase];
            for (uint64_t j = e2.hoff[q]; j < e2.hoff[q + 1]; j++) {
                u4 h2 = e2.hits[j];
                if (h_strand(h1) == h_strand(h2)) continue;
                const uint32_t *P2 = e2.pos + e2.poff[j - e2.hbase];
                uint64_t n2 = e2.poff[j - e2.hbase + 1] - e2.poff[j - e2.hbase];
                int64_t s = (int64_t)h_score(h1) + h_score(h2);
                for (uint64_t x = 0; x < n1; x++) {
                    int64_t p1 = P1[x];
                    // range of end-2 positions forming a proper pair with p1
                    int64_t a, b;
                    if (h_strand(h1) == 0) {  // end 1 is +: pf = p1, pr = p2, lr = len2
                        int64_t lr = h_len(h2);
                        a = p1 + lo - lr > p1 ? p1 + lo - lr : p1;
                        b = p1 + hi - lr;
                    } else {  // end 1 is -: pr = p1, lr = len1, pf = p2
                        int64_t lr = h_len(h1);
                        a = p1 + lr - hi;
                        b = p1 + lr - lo < p1 ? p1 + lr - lo : p1;
                    }
                    if (b < a || b < 0) continue;
                    uint64_t y = lower_bound(P2, n2, (uint64_t)(a < 0 ? 0 : a));
                    for (; y < n2 && (int64_t)P2[y] <= b; y++) {
                        int64_t p2 = P2[y];
                        int64_t pf = h_strand(h1) == 0 ? p1 : p2;
                        int64_t pr = h_strand(h1) == 0 ? p2 : p1;
                        int64_t lr = h_strand(h1) == 0 ? h_len(h2) : h_len(h1);
                        int64_t ins = pr + lr - pf;
                        int64_t d = ins > mu ? ins - mu : mu - ins;
                        bool bt;
                        if (!found) bt = true;
                        else if (s != bs) bt = s < bs;
                        else if (d != bd) bt = d < bd;
                        else if (pf != bpf) bt = pf < bpf;
                        else if ((uint32_t)h_strand(h1) != o.strand1) bt = (uint32_t)h_strand(h1) < o.strand1;
                        else if ((uint32_t)p1 != o.pos1) bt = (uint32_t)p1 < o.pos1;
                        else if ((uint32_t)h_len(h1) != o.len1) bt = (uint32_t)h_len(h1) < o.len1;
                        else if ((uint32_t)p2 != o.pos2) bt = (uint32_t)p2 < o.pos2;
                        else bt = (uint32_t)h_len(h2) < o.len2;
                        if (bt) {
                            found = true;
                            bs = s;
                            bd = d;
                            bpf = pf;
                            o.pos1 = (uint32_t)p1;
                            o.pos2 = (uint32_t)p2;
                            o.len1 = (uint16_t)h_len(h1);
                            o.len2 = (uint16_t)h_len(h2);
                            o.score1 = (uint16_t)h_score(h1);
                            o.score2 = (uint16_t)h_score(h2);
                            o.strand1 = (uint8_t)h_strand(h1);
                            o.strand2 = (uint8_t)h_strand(h2);
                            o.insert = (int32_t)ins;
                        }
                    }
                }
            }
        }
    }
    uint32_t pp;
    u4 hp;
    bool rep1 = false, rep2 = false;
    bool f1 = se_primary(e1, q, pp, hp, rep1);
    if (found) {
        o.flags = BWFM_PF_PAIRED | BWFM_PF_MAPPED1 | BWFM_PF_MAPPED2;
    } else if (f1) {
        o.pos1 = pp;
        o.len1 = (uint16_t)h_len(hp);
        o.score1 = (uint16_t)h_score(hp);
        o.strand1 = (uint8_t)h_strand(hp);
        o.flags |= BWFM_PF_MAPPED1;
    }
    if (paired) {
        bool f2 = se_primary(e2, q, pp, hp, rep2);
        if (!found && f2) {
            o.pos2 = pp;
            o.len2 = (uint16_t)h_len(hp);
            o.score2 = (uint16_t)h_score(hp);
            o.strand2 = (uint8_t)h_strand(hp);
            o.flags |= BWFM_PF_MAPPED2;
        }
    }
    if (rep1) o.flags |= BWFM_PF_REP1;
    if (rep2) o.flags |= BWFM_PF_REP2;
    out[q] = o;
}


// ------------------------------------------------------------------ short-string table

// Level d of direction `which`'s table at kt from level d - 1: one thread per
// string S of d - 1 bases writes the intervals of aS, a = 0..3, from the
// rank counts at S's k and l + 1 (the same step the search takes).  mark:
// strings that do not occur get (1 + the number of their first-prepended
// bases that do, 0) instead of the step's crossed pointers (a string that
// occurs has l >= 1, since row 0 is the empty suffix's).
template <int LW>
__global__ __launch_bounds__(256) void k_kt_level(DevIndex ix, int which, int d, uint32_t *kt, int mark) {
    const uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (p >= ((uint64_t)1 << (2 * (d - 1)))) return;
    const DevDir dd = pick_dir(ix, which);
    const uint64_t pe = kt_level_start(d - 1) + p;
    const u2 kl = reinterpret_cast<const u2 *>(kt)[pe];
    Kids k;
    if (mark && kl.y == 0) {
#pragma unroll
        for (int a = 0; a < 4; a++) {
            k.x[a] = kl.x;
            k.y[a] = 0;
        }
    } else {
        rank_children<LW>(ix, dd, kl.x, kl.y + 1, k);
        if (mark) {
#pragma unroll
            for (int a = 0; a < 4; a++)
                if (!(k.mask & (1u << a))) {
                    k.x[a] = (uint32_t)d;
                    k.y[a] = 0;
                }
        }
    }
    u4 *dst = reinterpret_cast<u4 *>(kt + 2 * (size_t)kt_children(d - 1, (uint32_t)p));
    dst[0] = mk4(k.x[0], k.y[0], k.x[1], k.y[1]);
    dst[1] = mk4(k.x[2], k.y[2], k.x[3], k.y[3]);
}

// Strings of the deepest level that occur once get their position in the
// direction's text: one thread per position of the text.
__global__ __launch_bounds__(256) void k_kt_single(DevIndex ix, int which, int levels, uint32_t *kt) {
    u2 *lv = reinterpret_cast<u2 *>(kt) + kt_level_start(levels);
    for (uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; p + levels <= ix.n;
         p += (uint64_t)gridDim.x * blockDim.x) {
        // the string at p: T[p, p + levels), or T[n - p - levels, n - p) backwards
        const uint32_t t0 = which == 0 ? (uint32_t)p : ix.n - (uint32_t)p - (uint32_t)levels;
        const u2w w = *reinterpret_cast<const u2w *>(ix.pac + (t0 >> 4));
        uint32_t code = __builtin_amdgcn_alignbit(w.y, w.x, 2 * (t0 & 15)) & ((1u << (2 * levels)) - 1u);
        if (which) code = rev_digits(code, levels);
        const u2 kl = lv[code];
        if (kl.x == kl.y) {
            uint32_t next = SINGLE;
            if (p >= (uint32_t)NEXT) {
                // the bases before p in the direction's text, the nearest first
                const uint32_t t1 = which == 0 ? (uint32_t)p - NEXT : ix.n - (uint32_t)p;
                const u2w v = *reinterpret_cast<const u2w *>(ix.pac + (t1 >> 4));
                next = __builtin_amdgcn_alignbit(v.y, v.x, 2 * (t1 & 15)) & ((1u << (2 * NEXT)) - 1u);
                if (which == 0) next = rev_digits(next, NEXT);
                next |= SINGLE0;
            }
            lv[code] = mk2((uint32_t)p, next);
        }
    }
}

// The whole suffix array and its inverse from the sampled rows: one thread
// per sampled row walks back through the text until the next sampled row (or
// the text's start), so that every row is visited once.
template <int LW>
__global__ __launch_bounds__(256) void k_full_sa(DevIndex ix, int which, uint64_t n_samples, uint32_t *sa,
                                                 uint32_t *isa) {
    const DevDir d = pick_dir(ix, which);
    const uint32_t mask = (1u << ix.sa_shift) - 1u;
    for (uint64_t s = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; s < n_samples;
         s += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t j = (uint32_t)(s << ix.sa_shift);
        uint32_t q = d.sa[s];
        for (;;) {
            sa[j] = q;
            isa[q] = j;
            if (q == 0) break;
            j = lf_step<LW>(ix, d, j);
            q--;
            if ((j & mask) == 0) break;
        }
    }
}

// level 0: the empty string's interval (0, n)
__global__ void k_kt_root(uint32_t *kt, uint32_t n) {
    if (threadIdx.x == 0) {
        kt[0] = 0;
        kt[1] = n;
    }
}

// ------------------------------------------------------------------ random-line probe

// Each lane performs `iters` dependent fetches of whole lines at
// pseudo-random line indices; the next index depends on the data just read,
// as in the search's pointer chase.  Every index is reduced into
// [0, n_lines), so any buffer contents are safe.
template <int LW>
__global__ __launch_bounds__(256) void k_probe_gather(const u4 *buf, uint64_t n_lines, uint32_t iters,
                                                      uint32_t *sink) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t x = 0x9E3779B97F4A7C15ULL * (t + 1);
    uint32_t acc = 0;
    for (uint32_t it = 0; it < iters; it++) {
        x ^= x >> 31;
        x *= 0xBF58476D1CE4E5B9ULL;
        x ^= x >> 29;
        const uint64_t line = __umul64hi(x, n_lines);
        const u4 *L = buf + line * (LW / 4);
#pragma unroll
        for (int q = 0; q < LW / 4; q++) {
            u4 v = L[q];
            acc += v.x ^ v.y ^ v.z ^ v.w;
        }
        x += acc;
    }
    sink[t] = acc;
}

// ------------------------------------------------------------------ host helpers

#define HIPCHK(expr)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(BWFM_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

inline uint32_t blocks(uint64_t n, uint32_t b) { return (uint32_t)((n + b - 1) / b); }

// ------------------------------------------------------------------ kernel timing

struct TimingStore {
    std::mutex mu;
    bool on = false;
    std::map<std::string, std::pair<double, uint64_t>> acc;
};
TimingStore &timing() {
    static TimingStore t;
    return t;
}

// Events around the launches of one API call; resolved when the call has
// synchronised its stream.
struct CallTimer {
    struct Rec {
        const char *name;
        hipEvent_t a, b;
    };
    std::vector<Rec> recs;
    bool on;
    hipStream_t st;
    explicit CallTimer(hipStream_t s, bool allowed = true) : on(false), st(s) {
        if (!allowed) return;  // callers that must not create events
        std::lock_guard<std::mutex> g(timing().mu);
        on = timing().on;
    }
    int begin(const char *name) {
        if (!on) return -1;
        Rec r{name, nullptr, nullptr};
        if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return -1;
        (void)hipEventRecord(r.a, st);
        recs.push_back(r);
        return (int)recs.size() - 1;
    }
    void end(int i) {
        if (i >= 0) (void)hipEventRecord(recs[i].b, st);
    }
    ~CallTimer() {
        if (recs.empty()) return;
        (void)hipStreamSynchronize(st);
        std::lock_guard<std::mutex> g(timing().mu);
        for (auto &r : recs) {
            float ms = 0;
            if (hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
                auto &e = timing().acc[r.name];
                e.first += ms;
                e.second += 1;
            }
            (void)hipEventDestroy(r.a);
            (void)hipEventDestroy(r.b);
        }
    }
};

DevIndex dev_index(const bwfm_index *ix) {
    DevIndex d;
    memset(&d, 0, sizeof(d));
    for (int k = 0; k < 2; k++) {
        d.dir[k].lines = (const uint32_t *)ix->d_lines[k];
        d.dir[k].sa = (const uint32_t *)ix->d_sa[k];
        for (int a = 0; a < 4; a++) d.dir[k].C[a] = (uint32_t)ix->dir[k].C[a];
        d.dir[k].primary = (uint32_t)ix->dir[k].primary;
        d.dir[k].kt = (const uint32_t *)ix->d_jt[k];
        d.dir[k].full = (const uint32_t *)ix->d_full[k];
    }
    d.pac = (const uint32_t *)ix->d_pac;
    d.kt_levels = ix->jt_levels;
    d.magic = (uint64_t)(((unsigned __int128)1 << 64) / ix->bpl) + 1;
    d.n = (uint32_t)ix->n;
    d.bpl = ix->bpl;
    uint32_t s = 0;
    while ((1u << s) < ix->sa_sample) s++;
    d.sa_shift = s;
    d.line_words = ix->line_bytes / 4;
    return d;
}

Params make_params(const bwfm_aln_params &p) {
    Params P;
    P.max_diff = p.max_diff;
    P.max_gapo = p.max_gapo;
    P.max_gape = p.max_gape;
    P.seed_len = p.seed_len;
    P.seed_diff = p.seed_diff;
    P.ies = p.indel_end_skip;
    P.s_mm = p.s_mm;
    P.s_gapo = p.s_gapo;
    P.s_gape = p.s_gape;
    P.mode = p.mode;
    P.max_best = p.max_best;
    P.max_hits = p.max_hits;
    P.minc = std::min(p.s_mm, std::min(p.s_gapo, p.s_gape));
    (void)p.form;
    P.s1 = std::max(p.indel_end_skip, 1);
    return P;
}

// The workspace of a stream on this index, created on first use.
bwfm::Workspace &stream_ws(bwfm_index *ix, hipStream_t st) {
    std::lock_guard<std::mutex> g(ix->ws_mu);
    auto &w = ix->ws[(void *)st];
    if (!w) w.reset(new bwfm::Workspace());
    return *w;
}

// Grow a workspace buffer to at least `bytes` (grow-only).  The stream's
// earlier work may still read the old buffer, so it is drained first.
int ws_grow(void *&ptr, size_t &have, size_t bytes, hipStream_t st) {
    if (have >= bytes && ptr) return BWFM_OK;
    if (ptr) {
        HIPCHK(hipStreamSynchronize(st));
        dev_free(ptr);
    }
    ptr = nullptr;
    have = 0;
    const size_t want = std::max<size_t>(bytes + bytes / 8, 4096);
    if (dev_malloc(&ptr, want) != hipSuccess) {
        ptr = nullptr;
        (void)hipGetLastError();
        return fail(BWFM_E_NOMEM, "workspace allocation of " + std::to_string(want) + " bytes failed");
    }
    have = want;
    return BWFM_OK;
}

int ws_reserve(bwfm::Workspace &w, size_t bytes, hipStream_t st, void **out) {
    if (int rc = ws_grow(w.ptr, w.bytes, bytes, st)) return rc;
    *out = w.ptr;
    return BWFM_OK;
}

struct Carver {
    char *p;
    size_t used = 0;
    template <typename T>
    T *take(size_t n) {
        used = (used + 255) & ~size_t(255);
        T *r = reinterpret_cast<T *>(p + used);
        used += n * sizeof(T);
        return r;
    }
};

// Exclusive scan of n u32 counts into n + 1 u64 offsets (out[n] = total).
// With n_dev the count is read on the device (at most n; the grid covers n).
int scan_counts(const uint32_t *cnt, uint64_t n, uint64_t *out, uint64_t *part, hipStream_t st,
                const uint64_t *n_dev = nullptr) {
    uint64_t nb = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    if (n == 0) {
        k_fill_u32<<<1, 64, 0, st>>>(reinterpret_cast<uint32_t *>(out), 2, 0u);
        HIPCHK(hipGetLastError());
        return BWFM_OK;
    }
    k_scan_reduce<<<(uint32_t)nb, SCAN_BLOCK, 0, st>>>(cnt, n, part, n_dev);
    k_scan_parts<<<1, SCAN_BLOCK, 0, st>>>(part, nb);
    k_scan_apply<<<(uint32_t)nb, SCAN_BLOCK, 0, st>>>(cnt, n, part, out, n_dev);
    HIPCHK(hipGetLastError());
    return BWFM_OK;
}

size_t scan_part_elems(uint64_t n) { return (n + SCAN_BLOCK - 1) / SCAN_BLOCK + 1; }

// Lanes of a persistent grid that fit on the device at once, for a block
// size and its dynamic LDS, at most waves_per_simd waves per SIMD (0 = no
// cap; a CU has 4 SIMDs).
template <int LW>
uint32_t persistent_lanes(uint32_t bs, size_t lds, int waves_per_simd) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<LW>(waves_per_simd), (int)bs, lds) !=
            hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    if (waves_per_simd > 0) {
        const int cap = std::max(1, waves_per_simd * 4 * 64 / (int)bs);
        per_cu = std::min(per_cu, cap);
    }
    return (uint32_t)cus * (uint32_t)per_cu * bs;
}

// Lanes of the batched form for n reads: the lanes that fit, but no more
// than a wave per read (a wave's other lanes help its reads) up to 1024
// reads, 16 lanes per read from 4096 on (each lane needs its buffers: 17 KB
// at 100 bases).  1000 pairs take 2.5 ms at a wave per read, 2.9 ms at 16
// lanes; 5000 pairs 3.7 ms either way.  lean: a lane per read, where memory is
// short (a call that finds no memory for its workspace is tried once more in
// this shape, with the fewest task entries and slots too: 1000 reads of 512
// bases 1.2 GB instead of 4.6).
inline uint32_t batched_lanes(uint32_t fit, uint32_t n, uint32_t bs, bool lean) {
    const uint64_t per = lean ? std::max(n, 1u)
                              : std::min<uint64_t>(64ull * std::max(n, 1u), std::max<uint64_t>(65536, 16ull * n));
    const uint64_t want = ((per + bs - 1) / bs) * bs;
    return (uint32_t)std::min<uint64_t>(fit, want);
}

// LDS bytes per lane for reads up to mlen bases (an odd number of dwords,
// which spreads the lanes' rows over the banks) and the largest block that
// keeps a block's LDS (rows plus the per-wave sharing blocks) within 64 KB.
inline uint32_t lds_stride_for(uint32_t mlen) {
    uint32_t dw = (mlen + 3) / 4;
    if ((dw & 1) == 0) dw++;
    return dw * 4;
}
inline uint32_t block_for(uint32_t stride) {
    uint32_t bs = BLOCK;
    while (bs > 64 && (size_t)bs * stride + (bs / 64) * sizeof(WaveShare) > 65536) bs /= 2;
    return bs;
}

// waves of a first pass of `lanes` that must have ended before its parts are
// split early
inline uint32_t drain_waves(uint32_t lanes) { return (lanes / 64 * DRAIN_EIGHTHS + 7) / 8; }
// whether the declared read length leaves a CU of 160 KB so few of these
// blocks (bs lanes, lds bytes) that they make a wave a SIMD or fewer
inline uint32_t drain_at_once(uint32_t bs, size_t lds) { return 163840 / lds * (bs / 64) <= 4; }

constexpr uint32_t SLOW_LANES = BWFM_SLOW_LANES;  // most lanes of the second pass
constexpr uint32_t SPLIT_DEFAULT = 16384;         // split budget unless the caller sets one

// Expansions between splits for a parameter block; 0: no splitting (the
// plain form never splits).
inline uint32_t split_budget_of(const bwfm_aln_params &p) {
    if (p.form == BWFM_FORM_PLAIN || p.split_budget < 0) return 0;
    return p.split_budget == 0 ? SPLIT_DEFAULT : (uint32_t)p.split_budget;
}

// Room of the split searches for a batch of n reads of at most mlen bases:
// in batches of long reads, which are split early, a slot for every read that
// can be in flight when the batch runs dry (one a lane of the first pass); of
// others a slot for one read in eight (at least 64, at most 2^26).  Per
// generation sixteen task entries a read, in smaller batches 1024 a read up to
// 2^23 (at most 2^26 in all): a split hands out a few hundred entries on long
// reads.  Running out is not an error, but a read or task that finds no room
// goes on alone, which can take seconds (2.2 s for 150 k reads of 250 bases
// whose splits outgrew sixteen entries a read; 300 k / 600 k of them at a split
// budget of 512 with a slot for one in eight 2.6 / 2.9 s, so 77 / 119 ms).
struct SplitShape {
    uint32_t slot_cap, task_cap, dstride;
};
inline SplitShape split_shape(uint32_t n, uint32_t mlen, uint32_t lanes, bool lean) {
    SplitShape z;
    const uint64_t least = lean ? 4096 : 1024ull * std::min(std::max(n, 1u), 8192u);
    const uint32_t slots = mlen >= LONG_READ && !lean ? lanes : std::min(std::max(64u, n / 8), 1u << 26);
    z.slot_cap = std::min(std::max(n, 1u), slots);
    z.task_cap = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(16ull * n, least), 1ull << 26);
    z.dstride = ((mlen + 15) / 16) * 16;
    return z;
}
inline size_t split_bytes(const SplitShape &z) {
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    return 9 * al((size_t)z.slot_cap * 4) + al((size_t)z.slot_cap * 2 * z.dstride) +
           al((size_t)z.slot_cap * SLOT_HITS * 16) + 2 * al((size_t)z.task_cap * 16) + 2 * al((size_t)z.task_cap * 4) +
           al(SPLIT_CTL * 4) + al(sizeof(TaskArgs)) + 256;
}
inline SplitBufs carve_split(Carver &cv, const SplitShape &z, uint32_t budget, TaskArgs **targs) {
    SplitBufs X{};
    X.slot_read = cv.take<uint32_t>(z.slot_cap);
    X.slot_meta = cv.take<uint32_t>(z.slot_cap);
    X.slot_best = cv.take<int>(z.slot_cap);
    X.slot_nhit = cv.take<uint32_t>(z.slot_cap);
    X.slot_fail = cv.take<uint32_t>(z.slot_cap);
    X.slot_exp = cv.take<uint32_t>(z.slot_cap);
    X.slot_owner = cv.take<uint32_t>(z.slot_cap);
    X.slot_own = cv.take<uint32_t>(z.slot_cap);
    X.slot_obest = cv.take<int>(z.slot_cap);
    X.slot_rows = cv.take<uint8_t>((size_t)z.slot_cap * 2 * z.dstride);
    X.slot_hits = cv.take<u4>((size_t)z.slot_cap * SLOT_HITS);
    for (int k = 0; k < 2; k++) {
        X.tasks[k] = cv.take<u4>(z.task_cap);
        X.task_ref[k] = cv.take<uint32_t>(z.task_cap);
    }
    X.ctl = cv.take<uint32_t>(SPLIT_CTL);
    *targs = cv.take<TaskArgs>(1);
    X.slot_cap = z.slot_cap;
    X.task_cap = z.task_cap;
    X.dstride = z.dstride;
    X.budget = budget;
    return X;
}

// Lanes of the task rounds' grid (blocks of BLOCK lanes, no LDS): as many
// as fit on the device at once, but at most sixteen per read of the batch
// (n_up lanes) or the first pass's lanes, whichever is more, since they
// all need lane buffers.
template <int LW>
uint32_t task_lanes(uint32_t n_up, uint32_t lanes) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_align_tasks<LW>, (int)BLOCK, 0) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    if (LW != LW_SUB && (uint64_t)n_up < (uint64_t)cus * (uint64_t)per_cu * BLOCK * TASK_READS)
        per_cu = std::min(per_cu, TASK_WAVES_FEW * 4 * 64 / BLOCK);
    const uint64_t fit = (uint64_t)cus * (uint64_t)per_cu * BLOCK;
    const uint64_t want = std::max<uint64_t>(lanes, ((16ull * n_up + BLOCK - 1) / BLOCK) * BLOCK);
    return (uint32_t)std::max<uint64_t>(std::min(fit, want), BLOCK);
}

// After the first pass (split searches on): the collection of the split
// reads' first-pass hits, the task rounds on their own grid of tlanes
// lanes, on the first pass's lane buffers (allocated for both grids), the
// last round without a drain, then the publication of the split reads.  Every
// launch reads its counts on the device, so the sequence can be captured.
template <int LW>
void enqueue_split(const DevIndex &D, const Params &P, const SplitBufs &X, TaskArgs *targs, const LaneBufs &lb,
                   const ReadOut &O, uint32_t tlanes, hipStream_t st) {
    SplitBufs Xc = X;
    Xc.lane_cand = lb.cand;
    k_split_collect<<<blocks(X.slot_cap, 256), 256, 0, st>>>(Xc);
    k_set_task_args<<<1, 64, 0, st>>>(targs, TaskArgs{lb, X});
    for (uint32_t g = 0; g < (uint32_t)SPLIT_ROUNDS; g++)
        k_align_tasks<LW><<<tlanes / BLOCK, BLOCK, 0, st>>>(D, P, targs, g, g + 1 < (uint32_t)SPLIT_ROUNDS ? 1u : 0u);
    k_split_publish<<<blocks(X.slot_cap, 256), 256, 0, st>>>(P, X, O);
}

template <int LW>
int align_impl(bwfm_index *ix, bwfm::Workspace &ws, const bwfm_reads *rd, const bwfm_aln_params *p,
               bwfm_aln_result *res, hipStream_t st, uint32_t *expand, uint64_t *work = nullptr) {
    const uint32_t n = rd->n_reads;
    const DevIndex D = dev_index(ix);
    const Params P = make_params(*p);
    ReadsView rv{rd->bases, rd->offsets, rd->lengths, rd->max_diff, rd->n_reads, rd->max_len, nullptr};
    const uint32_t mlen = std::max<uint32_t>(rd->max_len, 1);
    const uint32_t worst_stack = 8 * (mlen + BWFM_MAX_DIFF) + 1;  // never overflows
    const uint32_t lstride = lds_stride_for(mlen);
    const bool plain = p->form == BWFM_FORM_PLAIN;
    const uint32_t sbud = plain ? 0u : split_budget_of(*p);  // split searches (batched form)
    const uint32_t bs = block_for(lstride);
    const size_t lds = (size_t)bs * lstride + (plain ? 0 : (bs / 64) * sizeof(WaveShare));
    const uint32_t nr_up = ((std::max<uint32_t>(n, 1) + bs - 1) / bs) * bs;
    const uint32_t fit = plain ? 0 : persistent_lanes<LW>(bs, lds, p->waves_per_simd);
    const uint32_t stack_cap = plain ? std::min<uint32_t>(worst_stack, PLAIN_STACK) : worst_stack;
    // the staging arena holds the reported hits of every read: as many as
    // the output can take
    const uint64_t stage_cap = res->hit_capacity;
    const uint32_t slow_lanes = std::min<uint32_t>(nr_up, SLOW_LANES);
    const uint32_t scap = P.max_hits + 1;
    const uint32_t dstride = ((mlen + 15) / 16) * 16;  // of the D-array pre-pass's rows
    uint32_t lanes = 0, tlanes = 0, blanes = 0;
    SplitShape zs{};
    void *w;
    auto reserve = [&](bool lean) {
        lanes = plain ? nr_up : batched_lanes(fit, n, bs, lean);
        // the task rounds' grid shares the lane buffers: room for the larger one
        tlanes = sbud ? task_lanes<LW>(nr_up, lanes) : 0u;
        blanes = std::max(lanes, tlanes);
        zs = split_shape(n, mlen, lanes, lean);
        size_t need = (size_t)blanes * stack_cap * 16 + (size_t)blanes * FAST_CAND * 16;
        need += (size_t)slow_lanes * worst_stack * 16 + (size_t)slow_lanes * scap * 16;
        need += (size_t)n * 4 * 2 + (size_t)n * 8 + stage_cap * 16 + scan_part_elems(n) * 8 + 16 * 256;
        need += sizeof(PersistentArgs) + 256;
        if (!plain) need += (size_t)n * 2 * dstride + n + 2 * 256;
        if (sbud) need += split_bytes(zs) + (size_t)lanes * 4 + 256;
        return ws_reserve(ws, need, st, &w);
    };
    int rc = reserve(false);
    if (rc == BWFM_E_NOMEM && !plain) rc = reserve(true);
    if (rc) return rc;
    Carver cv{(char *)w};
    u4 *lstack = cv.take<u4>((size_t)blanes * stack_cap);
    u4 *lcand = cv.take<u4>((size_t)blanes * FAST_CAND);
    u4 *sstack = cv.take<u4>((size_t)slow_lanes * worst_stack);
    u4 *scand = cv.take<u4>((size_t)slow_lanes * scap);
    uint32_t *n_rep = cv.take<uint32_t>(n);
    uint32_t *slow_list = cv.take<uint32_t>(n);
    uint64_t *stage_off = cv.take<uint64_t>(n);
    u4 *stage = cv.take<u4>(stage_cap);
    uint64_t *part = cv.take<uint64_t>(scan_part_elems(n));
    PersistentArgs *pargs = cv.take<PersistentArgs>(1);
    uint8_t *drows = plain ? nullptr : cv.take<uint8_t>((size_t)n * 2 * dstride);
    uint8_t *dflag = plain ? nullptr : cv.take<uint8_t>(n);
    TaskArgs *targs = nullptr;
    SplitBufs X = sbud ? carve_split(cv, zs, sbud, &targs) : SplitBufs{};
    X.count = expand != nullptr;
    X.drain = drain_waves(lanes);
    uint32_t *lane_read = sbud ? cv.take<uint32_t>(lanes) : nullptr;
    uint32_t *ctl = cv.take<uint32_t>(16);  // n_slow, next_read, stage_used (64-bit), slow_next
    uint32_t *n_slow = ctl, *next_read = ctl + 1, *slow_next = ctl + 4;
    unsigned long long *stage_used = reinterpret_cast<unsigned long long *>(ctl + 2);
    k_fill_u32<<<1, 64, 0, st>>>(ctl, 16, 0u);
    // plain lanes start together and stay roughly in step: interleave their
    // buffers; persistent lanes drift apart: give each a contiguous run
    LaneBufs lb = plain ? LaneBufs{lstack, lcand, 1, lanes, stack_cap, 1, lanes, FAST_CAND, lstride}
                        : LaneBufs{lstack, lcand, stack_cap, 1, stack_cap, FAST_CAND, 1, FAST_CAND, lstride};
    ReadOut O{n_rep,     res->c1,   res->c2,   res->status, slow_list,
              n_slow,    stage,     stage_used, stage_cap,  stage_off,
              expand,    reinterpret_cast<unsigned long long *>(work)};
    if (work) k_fill_u32<<<1, 64, 0, st>>>(reinterpret_cast<uint32_t *>(work), 2 * (6 + SPLIT_ROUNDS), 0u);
    if (sbud) k_fill_u32<<<1, 64, 0, st>>>(X.ctl, SPLIT_CTL, 0u);
    CallTimer tm(st);
    if (n) {
        if (plain) {
            int t = tm.begin("align_plain");
            k_align_plain<LW><<<nr_up / bs, bs, lds, st>>>(D, rv, P, lb, O);
            tm.end(t);
        } else {
            int td = tm.begin("dscan");
            k_dscan<LW><<<nr_up / bs, bs, (size_t)bs * lstride, st>>>(D, rv, P, drows, dflag, dstride, lstride,
                                                                      sbud ? X.ctl + SPLIT_LONG : nullptr);
            tm.end(td);
            k_set_args<<<1, 64, 0, st>>>(
                pargs, PersistentArgs{rv, lb, O, next_read, drows, dflag, dstride, X, lane_read},
                drain_at_once(bs, lds));
            int ts = tm.begin("align_search");
            int t = tm.begin("align_persistent");
            hipLaunchKernelGGL(persistent_kernel<LW>(p->waves_per_simd), dim3(lanes / bs), dim3(bs), lds, st, D, P,
                               (const PersistentArgs *)pargs);
            tm.end(t);
            if (sbud) {
                int tt = tm.begin("align_tasks");
                enqueue_split<LW>(D, P, X, targs, lb, O, tlanes, st);
                tm.end(tt);
            }
            tm.end(ts);
        }
        // the second pass reads its count on the device: no host round trip
        const size_t slds = (size_t)bs * lstride;
        LaneBufs sb{sstack, scand, worst_stack, 1, worst_stack, scap, 1, scap, lstride};
        int t = tm.begin("align_slow");
        k_align_slow<LW><<<slow_lanes / bs, bs, slds, st>>>(D, rv, P, sb, O, slow_next);
        tm.end(t);
        if (work && sbud)
            k_split_stats<<<blocks(X.slot_cap, 256), 256, 0, st>>>(X, reinterpret_cast<unsigned long long *>(work));
        HIPCHK(hipGetLastError());
    }
    rc = scan_counts(n_rep, n, res->hit_offsets, part, st);
    if (rc) return rc;
    uint64_t total = 0;
    HIPCHK(hipMemcpyAsync(&total, res->hit_offsets + n, 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (total > res->hit_capacity)
        return fail(BWFM_E_CAPACITY,
                    "hit capacity " + std::to_string(res->hit_capacity) + " < " + std::to_string(total));
    if (n && total) {
        int t = tm.begin("compact");
        k_compact<<<blocks(n, 256), 256, 0, st>>>(n, res->hit_offsets, stage, stage_off,
                                                  reinterpret_cast<u4 *>(res->hits), nullptr, nullptr);
        tm.end(t);
        HIPCHK(hipGetLastError());
    }
    HIPCHK(hipStreamSynchronize(st));
    return BWFM_OK;
}

// Enqueue the counts of positions per hit and their offsets (pos_off: n_hits
// + 1 entries, the last one the total).
int locate_count(uint64_t n_hits, const u4 *hits, uint32_t max_occ, uint64_t *pos_off, uint32_t *cnt, uint64_t *part,
                 hipStream_t st) {
    if (n_hits) {
        k_loc_count<<<blocks(n_hits, 256), 256, 0, st>>>(n_hits, hits, max_occ, cnt, nullptr);
        HIPCHK(hipGetLastError());
    }
    return scan_counts(cnt, n_hits, pos_off, part, st);
}

// Enqueue the positions of every hit.  total, or with the _dev counts (a
// captured step) its bound, sizes the grids; big: n_hits words; n_big: two.
template <int LW>
int locate_fill(const DevIndex &D, uint64_t n_hits, const u4 *hits, const uint64_t *pos_off, uint64_t total,
                uint32_t *pos, uint32_t *big, uint32_t *n_big, const uint64_t *n_hits_dev, const uint64_t *total_dev,
                hipStream_t st) {
    if (D.kt_levels) {
        k_loc_hits<<<blocks(n_hits, 256), 256, 0, st>>>(D, n_hits, hits, pos_off, pos, big, n_big + 1, n_hits_dev,
                                                        total_dev);
        k_loc_wide<<<512, 256, 0, st>>>(D, hits, pos_off, pos, big, n_big + 1);
    } else {
        // (a captured step's bound may be 0, its grid not)
        const uint64_t grid = std::min<uint64_t>(std::max(blocks(total, 256), 1u), total_dev ? 2048 : 65536);
        k_loc_rows<LW><<<(uint32_t)grid, 256, 0, st>>>(D, n_hits, hits, pos_off, total, pos, n_hits_dev, total_dev);
    }
    HIPCHK(hipGetLastError());
    return BWFM_OK;
}

// ... and their order, eagerly.
int locate_rows(const bwfm_index *ix, uint64_t n_hits, const u4 *hits, const uint64_t *pos_off, uint64_t total,
                uint32_t *pos, uint32_t *big, uint32_t *n_big, hipStream_t st, bool timed);

bool check_index(const bwfm_index *ix) { return ix && ix->device >= 0; }

// result buffers: per-read arrays may be NULL only for an empty batch
int check_result(const bwfm_aln_result *r, uint32_t n) {
    return r && r->hit_offsets && (n == 0 || (r->c1 && r->c2 && r->status)) && (r->hits || r->hit_capacity == 0);
}

}  // namespace

// Call f with the index's rank-line format as a compile-time tag.
template <class F> auto by_layout(const bwfm_index *ix, F &&f) {
    if (ix->rank_format == BWFM_RANK_SUBCOUNTS) return f(std::integral_constant<int, LW_SUB>());
    if (ix->rank_format == BWFM_RANK_SUB128) return f(std::integral_constant<int, LW_SUB128>());
    if (ix->line_bytes == 128) return f(std::integral_constant<int, 32>());
    if (ix->line_bytes == 32) return f(std::integral_constant<int, 8>());
    return f(std::integral_constant<int, 16>());
}

namespace {
int locate_rows(const bwfm_index *ix, uint64_t n_hits, const u4 *hits, const uint64_t *pos_off, uint64_t total,
                uint32_t *pos, uint32_t *big, uint32_t *n_big, hipStream_t st, bool timed) {
    if (!total) return BWFM_OK;
    const DevIndex D = dev_index(ix);
    k_fill_u32<<<1, 64, 0, st>>>(n_big, 2, 0u);
    CallTimer tm(st, timed);
    int t = tm.begin("locate_rows");
    const int rc = by_layout(ix, [&](auto lw) {
        return locate_fill<decltype(lw)::value>(D, n_hits, hits, pos_off, total, pos, big, n_big, nullptr, nullptr, st);
    });
    tm.end(t);
    if (rc) return rc;
    t = tm.begin("sort");
    k_sort_small<<<blocks(n_hits, 256), 256, 0, st>>>(n_hits, pos_off, pos, big, n_big, nullptr, nullptr);
    k_sort_big<<<1024, 256, 0, st>>>(pos_off, pos, big, n_big);
    tm.end(t);
    HIPCHK(hipGetLastError());
    return BWFM_OK;
}
}  // namespace

// ===================================================================== C ABI

// table bytes per direction, padded to a multiple of 256 so that a lane's
// line-sized, line-aligned read around its 32 entry bytes stays inside
static uint64_t kt_bytes(uint32_t levels) {
    return levels ? (kt_level_start((int)levels + 1) * 8 + 255) / 256 * 256 : 0;
}

// Enqueue the levels of direction d's interval table at kt.
static void fill_table(const bwfm_index *ix, int d, uint32_t *kt, int levels, int mark, hipStream_t st) {
    const DevIndex D = dev_index(ix);
    k_kt_root<<<1, 64, 0, st>>>(kt, (uint32_t)ix->n);
    for (int lv = 1; lv <= levels; lv++) {
        const uint64_t np = (uint64_t)1 << (2 * (lv - 1));
        by_layout(ix, [&](auto t) {
            k_kt_level<decltype(t)::value><<<blocks(np, 256), 256, 0, st>>>(D, d, lv, kt, mark);
            return 0;
        });
    }
}

// The search's interval table, made once the rank lines are on the device.
// Depth, unless the caller set one: the least with 4^depth >= 2 n, at most 15,
// so that most of the deepest strings are absent or unique and a run of exact
// matches ends in its one entry: 100 Mbp: 14 levels, 2.9 GB per direction (its
// iterations per read: 1031, with 13 levels 1223, with 12 1421).  With it come
// the whole suffix array and its inverse, 8 bytes a base and direction, which
// turn rows into text positions and back (the deepest level names unique
// strings by position, so neither is of use alone).  All of it takes at most
// half of the free memory (less deep, or not made at all, where that is short:
// results do not depend on it).
int bwfm::build_search_tables(bwfm_index *ix, hipStream_t st) {
    if (ix->jt_want == 0 || ix->n >= SINGLE0) return BWFM_OK;
    size_t free_b = 0, total_b = 0;
    HIPCHK(hipMemGetInfo(&free_b, &total_b));
    free_b += dev_cached();
    int levels = ix->jt_want > 0 ? ix->jt_want : 1;
    if (ix->jt_want < 0)
        while (levels < 15 && ((uint64_t)1 << (2 * levels)) < 2 * ix->n) levels++;
    while (levels > 0 && 2 * (kt_bytes((uint32_t)levels) + 2 * (ix->n + 1) * 4) > free_b / 2) levels--;
    if (levels == 0) return BWFM_OK;
    const uint64_t bytes = kt_bytes((uint32_t)levels), full = 2 * (ix->n + 1) * 4;
    for (int d = 0; d < 2; d++)
        if (dev_malloc(&ix->d_jt[d], bytes) || dev_malloc(&ix->d_full[d], full)) {
            free_search_tables(ix);
            return BWFM_OK;
        }
    DevIndex D = dev_index(ix);  // no levels yet: the builders read rank lines
    for (int d = 0; d < 2; d++) {
        uint32_t *kt = (uint32_t *)ix->d_jt[d], *sa = (uint32_t *)ix->d_full[d];
        fill_table(ix, d, kt, levels, 1, st);
        k_kt_single<<<(uint32_t)std::min<uint64_t>(blocks(ix->n, 256), 1u << 16), 256, 0, st>>>(D, d, levels, kt);
        by_layout(ix, [&](auto t) {
            k_full_sa<decltype(t)::value><<<(uint32_t)std::min<uint64_t>(blocks(ix->n_samples, 256), 1u << 16), 256, 0,
                                            st>>>(D, d, ix->n_samples, sa, sa + ix->n + 1);
            return 0;
        });
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        free_search_tables(ix);
        return fail(BWFM_E_DEVICE, std::string("the search's tables: ") + hipGetErrorString(e));
    }
    ix->jt_levels = (uint32_t)levels;
    ix->device_bytes += 2 * (bytes + full);
    return BWFM_OK;
}

// Drop the search's tables; the caller has waited for the work that reads them.
void bwfm::free_search_tables(bwfm_index *ix) {
    for (int d = 0; d < 2; d++) {
        dev_free(ix->d_jt[d]);
        dev_free(ix->d_full[d]);
        ix->d_jt[d] = ix->d_full[d] = nullptr;
    }
    if (ix->jt_levels) ix->device_bytes -= 2 * (kt_bytes(ix->jt_levels) + 2 * (ix->n + 1) * 4);
    ix->jt_levels = 0;
    ix->jt_gen++;
}

extern "C" int bwfm_index_search_tables(bwfm_index *ix, int levels, void *stream) {
    if (!ix) return fail(BWFM_E_INVAL, "search_tables: NULL index");
    if (levels < -1 || levels > 15) return fail(BWFM_E_INVAL, "search_tables: levels must be -1, 0 or 1..15");
    std::unique_lock<std::shared_mutex> g(ix->mu);
    if (ix->device >= 0) {
        int dev = -1;
        HIPCHK(hipGetDevice(&dev));
        if (dev != ix->device) return fail(BWFM_E_INVAL, "search_tables: the index's device must be current");
        HIPCHK(hipDeviceSynchronize());  // captured steps on any stream may still read the tables
        free_search_tables(ix);
    }
    ix->jt_want = levels;
    return ix->device >= 0 ? build_search_tables(ix, (hipStream_t)stream) : (int)BWFM_OK;
}

extern "C" int bwfm_index_upload(bwfm_index *ix, void *stream) {
    if (!ix) return fail(BWFM_E_INVAL, "upload: NULL index");
    std::unique_lock<std::shared_mutex> g(ix->mu);
    if (ix->device >= 0) return BWFM_OK;
    hipStream_t st = (hipStream_t)stream;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    uint64_t bytes = 0;
    for (int d = 0; d < 2; d++) {
        size_t lb = ix->dir[d].lines.size() * 4, sb = ix->dir[d].sa.size() * 4;
        if (dev_malloc(&ix->d_lines[d], lb) != hipSuccess || dev_malloc(&ix->d_sa[d], sb) != hipSuccess)
            return fail(BWFM_E_NOMEM, "index upload: device allocation failed");
        HIPCHK(hipMemcpyAsync(ix->d_lines[d], ix->dir[d].lines.data(), lb, hipMemcpyHostToDevice, st));
        HIPCHK(hipMemcpyAsync(ix->d_sa[d], ix->dir[d].sa.data(), sb, hipMemcpyHostToDevice, st));
        bytes += lb + sb;
    }
    const size_t pb = (ix->pac.size() + 2) * 4;  // two words of padding (text_word)
    if (dev_malloc(&ix->d_pac, pb) != hipSuccess) return fail(BWFM_E_NOMEM, "index upload: device allocation failed");
    if (!ix->pac.empty())
        HIPCHK(hipMemcpyAsync(ix->d_pac, ix->pac.data(), ix->pac.size() * 4, hipMemcpyHostToDevice, st));
    bytes += pb;
    HIPCHK(hipStreamSynchronize(st));
    ix->device_bytes = bytes;
    if (int rc = build_search_tables(ix, st)) return rc;
    ix->device = dev;
    return BWFM_OK;
}


extern "C" int bwfm_index_kmer_table(bwfm_index *ix, int levels, void *stream) {
    if (!ix) return fail(BWFM_E_INVAL, "kmer_table: NULL index");
    std::unique_lock<std::shared_mutex> g(ix->mu);
    if (ix->device < 0) return fail(BWFM_E_INVAL, "kmer_table: the index is not uploaded");
    if (levels < -1 || levels > 15) return fail(BWFM_E_INVAL, "kmer_table: levels must be -1, 0 or 1..15");
    if (levels == -1) {
        levels = 1;
        while (levels < 14 && ((uint64_t)1 << (2 * levels)) < ix->n) levels++;
    }
    hipStream_t st = (hipStream_t)stream;
    HIPCHK(hipStreamSynchronize(st));
    ix->device_bytes -= 2 * kt_bytes(ix->kt_levels);
    ix->kt_levels = 0;
    for (int d = 0; d < 2; d++) {
        dev_free(ix->d_kt[d]);
        ix->d_kt[d] = nullptr;
    }
    if (levels == 0) return BWFM_OK;
    const uint64_t bytes = kt_bytes((uint32_t)levels);
    for (int d = 0; d < 2; d++)
        if (dev_malloc(&ix->d_kt[d], bytes) != hipSuccess) {
            for (int e = 0; e < 2; e++) {
                dev_free(ix->d_kt[e]);
                ix->d_kt[e] = nullptr;
            }
            (void)hipGetLastError();
            return fail(BWFM_E_NOMEM, "kmer_table: device allocation failed");
        }
    for (int d = 0; d < 2; d++) fill_table(ix, d, (uint32_t *)ix->d_kt[d], levels, 0, st);
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(st));
    ix->kt_levels = (uint32_t)levels;
    ix->device_bytes += 2 * bytes;
    return BWFM_OK;
}

extern "C" int bwfm_index_kmer_get(const bwfm_index *ix, int which, int level, uint64_t first, uint64_t count,
                                   uint32_t *out) {
    if (!ix || !out || (which != 0 && which != 1)) return fail(BWFM_E_INVAL, "kmer_get: bad argument");
    if (level < 0 || (uint32_t)level > ix->kt_levels || !ix->d_kt[which])
        return fail(BWFM_E_INVAL, "kmer_get: no such table level");
    const uint64_t codes = (uint64_t)1 << (2 * level);
    if (first > codes || count > codes - first) return fail(BWFM_E_INVAL, "kmer_get: codes out of range");
    if (!count) return BWFM_OK;
    const char *src = (const char *)ix->d_kt[which] + (kt_level_start(level) + first) * 8;
    HIPCHK(hipMemcpy(out, src, count * 8, hipMemcpyDeviceToHost));
    return BWFM_OK;
}

extern "C" void bwfm_index_free(bwfm_index *ix) {
    if (!ix) return;
    for (int d = 0; d < 2; d++) {
        dev_free(ix->d_lines[d]);
        dev_free(ix->d_sa[d]);
        dev_free(ix->d_kt[d]);
    }
    free_search_tables(ix);
    dev_free(ix->d_pac);
    for (auto &kv : ix->ws) {
        dev_free(kv.second->ptr);
        dev_free(kv.second->pos);
    }
    delete ix;
}

// Search parameters in range; 0 or a bwfm_err.
static int check_aln_params(const bwfm_aln_params *p) {
    if (p->max_diff < 0 || p->max_diff > BWFM_MAX_DIFF || p->max_gapo < 0 || p->seed_len < 0 || p->seed_diff < 0 ||
        p->indel_end_skip < 0 || p->s_mm < 0 || p->s_gapo < 0 || p->s_gape < 0 ||
        (p->mode != BWFM_MODE_ALL && p->mode != BWFM_MODE_BEST) || p->max_best < 0 || p->max_hits < 1 ||
        (p->form != BWFM_FORM_BATCHED && p->form != BWFM_FORM_PLAIN) || p->waves_per_simd < 0 ||
        p->waves_per_simd > 8 || p->max_hits > 65536 || p->s_mm > 63 || p->s_gapo > 63 || p->s_gape > 63)
        return fail(BWFM_E_INVAL, "align_batch: parameter out of range");
    const int32_t b = p->split_budget;
    if (b != 0 && b != -1 && (b < 16 || b > (1 << 24)))
        return fail(BWFM_E_INVAL, "align_batch: split_budget must be 0, -1 or in [16, 2^24]");
    return BWFM_OK;
}

// Argument checks shared by the align entry points; 0 or a bwfm_err.
static int check_align_args(bwfm_index *ix, const bwfm_reads *rd, const bwfm_aln_params *p,
                            const bwfm_aln_result *res) {
    if (!ix || !rd || !p || !check_result(res, rd->n_reads)) return fail(BWFM_E_INVAL, "align_batch: NULL argument");
    if (!check_index(ix)) return fail(BWFM_E_STATE, "align_batch: index not uploaded");
    if (rd->n_reads && (!rd->bases || !rd->offsets)) return fail(BWFM_E_INVAL, "align_batch: NULL reads");
    if (rd->max_len > BWFM_MAX_READ) return fail(BWFM_E_TOOLONG, "align_batch: max_len above 512");
    return check_aln_params(p);
}

extern "C" int bwfm_align_batch(const bwfm_index *cix, const bwfm_reads *rd, const bwfm_aln_params *p,
                                bwfm_aln_result *res, void *stream) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (int rc = check_align_args(ix, rd, p, res)) return rc;
    std::shared_lock<std::shared_mutex> g(ix->mu);
    hipStream_t st = (hipStream_t)stream;
    bwfm::Workspace &ws = stream_ws(ix, st);
    std::lock_guard<std::mutex> wg(ws.mu);
    return by_layout(ix, [&](auto lw) { return align_impl<decltype(lw)::value>(ix, ws, rd, p, res, st, nullptr); });
}

// Same as bwfm_align_batch, also writing per-read search work (states
// expanded, summed over both passes) to expand (device, n_reads).
extern "C" int bwfm_align_batch_counted(const bwfm_index *cix, const bwfm_reads *rd, const bwfm_aln_params *p,
                                        bwfm_aln_result *res, uint32_t *expand, uint64_t *work, void *stream) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (!expand) return fail(BWFM_E_INVAL, "align_batch_counted: NULL counter array");
    if (int rc = check_align_args(ix, rd, p, res)) return rc;
    std::shared_lock<std::shared_mutex> g(ix->mu);
    hipStream_t st = (hipStream_t)stream;
    bwfm::Workspace &ws = stream_ws(ix, st);
    std::lock_guard<std::mutex> wg(ws.mu);
    return by_layout(ix, [&](auto lw) {
        return align_impl<decltype(lw)::value>(ix, ws, rd, p, res, st, expand, work);
    });
}

extern "C" int bwfm_locate(const bwfm_index *cix, uint32_t n_reads, const bwfm_aln_result *res, uint32_t max_occ,
                           uint64_t *pos_off, uint32_t *pos, uint64_t cap, void *stream) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (!ix || !check_result(res, n_reads) || !pos_off || (!pos && cap))
        return fail(BWFM_E_INVAL, "locate: NULL argument");
    if (!check_index(ix)) return fail(BWFM_E_STATE, "locate: index not uploaded");
    std::shared_lock<std::shared_mutex> g(ix->mu);
    hipStream_t st = (hipStream_t)stream;
    bwfm::Workspace &ws = stream_ws(ix, st);
    std::lock_guard<std::mutex> wg(ws.mu);
    uint64_t h0 = 0, h1 = 0;
    HIPCHK(hipMemcpyAsync(&h0, res->hit_offsets, 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipMemcpyAsync(&h1, res->hit_offsets + n_reads, 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (h1 < h0) return fail(BWFM_E_INVAL, "locate: hit offsets decrease");
    const uint64_t n_hits = h1 - h0;
    size_t need = n_hits * 4 + scan_part_elems(n_hits) * 8 + n_hits * 4 + 4096;
    void *w;
    int rc = ws_reserve(ws, need, st, &w);
    if (rc) return rc;
    Carver cv{(char *)w};
    uint32_t *cnt = cv.take<uint32_t>(n_hits);
    uint64_t *part = cv.take<uint64_t>(scan_part_elems(n_hits));
    uint32_t *big = cv.take<uint32_t>(n_hits);
    uint32_t *n_big = cv.take<uint32_t>(2);
    uint64_t total = 0;
    const u4 *hits = (const u4 *)res->hits + h0;
    rc = locate_count(n_hits, hits, max_occ, pos_off, cnt, part, st);
    if (rc) return rc;
    HIPCHK(hipMemcpyAsync(&total, pos_off + n_hits, 8, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (total > cap) return fail(BWFM_E_CAPACITY, "position capacity too small");
    rc = locate_rows(ix, n_hits, hits, pos_off, total, pos, big, n_big, st, true);
    if (rc) return rc;
    HIPCHK(hipStreamSynchronize(st));
    return BWFM_OK;
}

namespace {

// Buffers of one pair_reads call: `ctl` returns the control area (counts,
// scan partials, per-hit position offsets of both ends), `pos` the located
// positions of both ends; either may fail with an error code.
struct PairMem {
    std::function<int(size_t, void **)> ctl, pos;
};

// Locate every hit of both ends, then pair: the body shared by the
// allocating and the non-allocating entry points.  The stream must be held
// by the caller (workspace mutex or the scratch contract).
int pair_impl(bwfm_index *ix, uint32_t n_pairs, const bwfm_aln_result *r1, const bwfm_aln_result *r2,
              const bwfm_pair_params *pp, bwfm_pair *out, hipStream_t st, const PairMem &mem, bool timed) {
    const bwfm_aln_result *rr[2] = {r1, r2};
    uint64_t hb[2] = {0, 0}, he[2] = {0, 0}, nh[2] = {0, 0};
    for (int e = 0; e < 2; e++)
        if (rr[e]) {
            HIPCHK(hipMemcpyAsync(&hb[e], rr[e]->hit_offsets, 8, hipMemcpyDeviceToHost, st));
            HIPCHK(hipMemcpyAsync(&he[e], rr[e]->hit_offsets + n_pairs, 8, hipMemcpyDeviceToHost, st));
        }
    HIPCHK(hipStreamSynchronize(st));
    for (int e = 0; e < 2; e++) {
        if (he[e] < hb[e]) return fail(BWFM_E_INVAL, "pair_reads: hit offsets decrease");
        nh[e] = he[e] - hb[e];
    }
    // control buffers and each end's position offsets first; the positions
    // of both ends in the second buffer, sized by a counting pass
    const uint64_t nmax = std::max(nh[0], nh[1]);
    const size_t ctl = nmax * 4 * 2 + scan_part_elems(nmax) * 8 + 4096 + (nh[0] + nh[1] + 2) * 8 + 6 * 256;
    void *wmem;
    if (int rc = mem.ctl(ctl, &wmem)) return rc;
    Carver cv{(char *)wmem};
    uint32_t *cnt = cv.take<uint32_t>(nmax);
    uint32_t *big = cv.take<uint32_t>(nmax);
    uint64_t *part = cv.take<uint64_t>(scan_part_elems(nmax));
    uint32_t *n_big = cv.take<uint32_t>(2);
    uint64_t *poff[2] = {cv.take<uint64_t>(nh[0] + 1), cv.take<uint64_t>(nh[1] + 1)};
    uint64_t total[2] = {0, 0};
    for (int e = 0; e < 2; e++)
        if (rr[e]) {
            if (int rc = locate_count(nh[e], (const u4 *)rr[e]->hits + hb[e], pp->max_occ, poff[e], cnt, part, st))
                return rc;
            HIPCHK(hipMemcpyAsync(&total[e], poff[e] + nh[e], 8, hipMemcpyDeviceToHost, st));
        }
    HIPCHK(hipStreamSynchronize(st));
    void *pmem;
    if (int rc = mem.pos((total[0] + total[1] + 1) * 4, &pmem)) return rc;
    uint32_t *pos[2] = {(uint32_t *)pmem, (uint32_t *)pmem + total[0]};
    for (int e = 0; e < 2; e++)
        if (rr[e])
            if (int rc = locate_rows(ix, nh[e], (const u4 *)rr[e]->hits + hb[e], poff[e], total[e], pos[e], big, n_big,
                                     st, timed))
                return rc;
    if (n_pairs) {
        EndView e1{r1->hit_offsets, (const u4 *)r1->hits, poff[0], pos[0], hb[0]};
        EndView e2 = e1;
        if (r2) e2 = EndView{r2->hit_offsets, (const u4 *)r2->hits, poff[1], pos[1], hb[1]};
        CallTimer tm(st, timed);
        int t = tm.begin("pair");
        k_pair<<<blocks(n_pairs, 256), 256, 0, st>>>(n_pairs, e1, e2, r2 ? 1 : 0, pp->lo, pp->hi, pp->mu, out, nullptr,
                                                     nullptr);
        tm.end(t);
        HIPCHK(hipGetLastError());
    }
    HIPCHK(hipStreamSynchronize(st));
    return BWFM_OK;
}

int check_pair_args(const bwfm_index *ix, uint32_t n_pairs, const bwfm_aln_result *r1, const bwfm_aln_result *r2,
                    const bwfm_pair_params *pp, const bwfm_pair *out) {
    if (!ix || !check_result(r1, n_pairs) || (r2 && !check_result(r2, n_pairs)) || !pp || (!out && n_pairs))
        return fail(BWFM_E_INVAL, "pair_reads: NULL argument");
    if (!check_index(ix)) return fail(BWFM_E_STATE, "pair_reads: index not uploaded");
    if (pp->lo > pp->hi) return fail(BWFM_E_INVAL, "pair_reads: lo > hi");
    return BWFM_OK;
}

}  // namespace

extern "C" int bwfm_pair_reads(const bwfm_index *cix, uint32_t n_pairs, const bwfm_aln_result *r1,
                               const bwfm_aln_result *r2, const bwfm_pair_params *pp, bwfm_pair *out, void *stream) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (int rc = check_pair_args(ix, n_pairs, r1, r2, pp, out)) return rc;
    std::shared_lock<std::shared_mutex> g(ix->mu);
    hipStream_t st = (hipStream_t)stream;
    bwfm::Workspace &ws = stream_ws(ix, st);
    std::lock_guard<std::mutex> wg(ws.mu);
    PairMem mem{[&](size_t b, void **p) { return ws_reserve(ws, b, st, p); },
                [&](size_t b, void **p) {
                    if (int rc = ws_grow(ws.pos, ws.pos_bytes, b, st)) return rc;
                    *p = ws.pos;
                    return (int)BWFM_OK;
                }};
    return pair_impl(ix, n_pairs, r1, r2, pp, out, st, mem, true);
}

// ------------------------------------------------------------------ fixed scratch

// Device scratch of bwfm_pair_reads_noalloc: the control area at its start,
// the located positions after it.  Each device holds its own copy; in host
// code `scratch` names a host-side stand-in, so only the address returned
// by hipGetSymbolAddress (kept per device below) reaches kernels.
static __device__ __align__(256) uint8_t scratch[BWFM_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_ptr[SCRATCH_MAX_DEVICES] = {};

// the device address of `scratch` on device dev, looked up on the first
// call made with that device current
int scratch_of(int dev, uint8_t **out) {
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return fail(BWFM_E_DEVICE, "noalloc: device ordinal out of range");
    std::lock_guard<std::mutex> g(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(BWFM_E_DEVICE, std::string("noalloc: scratch address lookup failed: ") + hipGetErrorString(e));
        scratch_ptr[dev] = p;
    }
    *out = (uint8_t *)scratch_ptr[dev];
    return BWFM_OK;
}
}  // namespace

extern "C" int bwfm_pair_reads_noalloc(const bwfm_index *cix, uint32_t n_pairs, const bwfm_aln_result *r1,
                                       const bwfm_aln_result *r2, const bwfm_pair_params *pp, bwfm_pair *out,
                                       void *stream) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (int rc = check_pair_args(ix, n_pairs, r1, r2, pp, out)) return rc;
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev != ix->device) return fail(BWFM_E_INVAL, "pair_reads_noalloc: the index's device must be current");
    uint8_t *base;
    if (int rc = scratch_of(dev, &base)) return rc;
    std::shared_lock<std::shared_mutex> g(ix->mu);
    hipStream_t st = (hipStream_t)stream;
    size_t ctl_end = 0;
    PairMem mem{[&](size_t b, void **p) {
                    if (b > BWFM_NOALLOC_SCRATCH_BYTES)
                        return fail(BWFM_E_CAPACITY, "pair_reads_noalloc: the hits need " + std::to_string(b) +
                                                         " bytes of control buffers, more than the " +
                                                         std::to_string((size_t)BWFM_NOALLOC_SCRATCH_BYTES) +
                                                         "-byte scratch");
                    ctl_end = (b + 255) & ~(size_t)255;
                    *p = base;
                    return (int)BWFM_OK;
                },
                [&](size_t b, void **p) {
                    if (ctl_end + b > BWFM_NOALLOC_SCRATCH_BYTES)
                        return fail(BWFM_E_CAPACITY, "pair_reads_noalloc: control buffers and positions need " +
                                                         std::to_string(ctl_end + b) + " bytes, more than the " +
                                                         std::to_string((size_t)BWFM_NOALLOC_SCRATCH_BYTES) +
                                                         "-byte scratch");
                    *p = base + ctl_end;
                    return (int)BWFM_OK;
                }};
    return pair_impl(ix, n_pairs, r1, r2, pp, out, st, mem, false);
}

extern "C" int bwfm_max_diff_rule(uint32_t len, double err, double thres) {
    // accumulate the Poisson(err * len) distribution until its tail drops
    // below thres
    double lambda = err * (double)len;
    double pk = std::exp(-lambda);
    double cdf = pk;
    for (int k = 0; k < 1000; k++) {
        if (1.0 - cdf < thres) return k;
        pk = pk * lambda / (double)(k + 1);
        cdf += pk;
    }
    return 1000;
}

extern "C" int bwfm_estimate_insert(const int32_t *ins, uint64_t n, bwfm_pair_params *out) {
    if (!out || (!ins && n)) return fail(BWFM_E_INVAL, "estimate_insert: NULL argument");
    if (n < 100) {
        out->lo = 0;
        out->hi = 500;
        out->mu = 250;
        return BWFM_OK;
    }
    std::vector<int32_t> v(ins, ins + n);
    std::sort(v.begin(), v.end());
    const double q1 = v[(size_t)std::floor(0.25 * (double)(n - 1))];
    const double q3 = v[(size_t)std::floor(0.75 * (double)(n - 1))];
    const double lo_k = q1 - 2 * (q3 - q1), hi_k = q3 + 2 * (q3 - q1);
    double sum = 0;
    uint64_t cnt = 0;
    for (int32_t x : v)
        if (x >= lo_k && x <= hi_k) {
            sum += x;
            cnt++;
        }
    const double mu = sum / (double)cnt;
    double ss = 0;
    for (int32_t x : v)
        if (x >= lo_k && x <= hi_k) ss += ((double)x - mu) * ((double)x - mu);
    const double sd = std::sqrt(ss / (double)cnt);
    const double lo = std::floor(mu - 4 * sd);
    out->lo = (int32_t)(lo < 0 ? 0 : lo);
    out->hi = (int32_t)std::ceil(mu + 4 * sd);
    out->mu = (int32_t)std::nearbyint(mu);
    return BWFM_OK;
}

extern "C" int bwfm_timing_enable(int on) {
    std::lock_guard<std::mutex> g(timing().mu);
    timing().on = on != 0;
    return BWFM_OK;
}

extern "C" int bwfm_timing_reset(void) {
    std::lock_guard<std::mutex> g(timing().mu);
    timing().acc.clear();
    return BWFM_OK;
}

extern "C" int bwfm_timing_get(const char *kernel, double *total_ms, uint64_t *launches) {
    if (!kernel || !total_ms || !launches) return fail(BWFM_E_INVAL, "timing_get: NULL argument");
    std::lock_guard<std::mutex> g(timing().mu);
    auto it = timing().acc.find(kernel);
    *total_ms = it == timing().acc.end() ? 0.0 : it->second.first;
    *launches = it == timing().acc.end() ? 0 : it->second.second;
    return BWFM_OK;
}

extern "C" int bwfm_probe_gather(const void *buf, uint64_t bytes, uint32_t line_bytes, uint32_t lanes, uint32_t iters,
                                 uint32_t *sink, double *ms_out, void *stream) {
    if (!buf || !sink || !ms_out || (line_bytes != 32 && line_bytes != 64 && line_bytes != 128) || lanes == 0 ||
        lanes % 256 ||
        bytes < line_bytes)
        return fail(BWFM_E_INVAL, "probe_gather: bad argument");
    hipStream_t st = (hipStream_t)stream;
    const uint64_t n_lines = bytes / line_bytes;
    hipEvent_t a, b;
    HIPCHK(hipEventCreate(&a));
    HIPCHK(hipEventCreate(&b));
    HIPCHK(hipEventRecord(a, st));
    if (line_bytes == 128)
        k_probe_gather<32><<<lanes / 256, 256, 0, st>>>((const u4 *)buf, n_lines, iters, sink);
    else if (line_bytes == 32)
        k_probe_gather<8><<<lanes / 256, 256, 0, st>>>((const u4 *)buf, n_lines, iters, sink);
    else
        k_probe_gather<16><<<lanes / 256, 256, 0, st>>>((const u4 *)buf, n_lines, iters, sink);
    hipError_t e = hipGetLastError();
    HIPCHK(hipEventRecord(b, st));
    HIPCHK(hipEventSynchronize(b));
    float ms = 0;
    HIPCHK(hipEventElapsedTime(&ms, a, b));
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (e != hipSuccess) return fail(BWFM_E_DEVICE, std::string("k_probe_gather: ") + hipGetErrorString(e));
    *ms_out = ms;
    return BWFM_OK;
}

// ------------------------------------------------------------------ captured pipeline

namespace {

// control words of a pipeline (uint64 indices)
enum {
    PC_PAIRS = 0,     // pairs in this run
    PC_READS = 1,     // reads in this run (2 * pairs)
    PC_HITS = 2,      // reported hits, 0 when they do not fit
    PC_POS = 3,       // located positions, 0 when they do not fit
    PC_NEED_HITS = 4, // reported hits
    PC_NEED_POS = 5,  // located positions
    PC_ERR = 6,       // BWFM_PIPE_E_* bits (low 32 bits)
    PC_BIG = 7,       // hits sorted by a workgroup (low 32 bits), hits located by the grid (high 32)
    PC_ALIGN = 8,     // 16 uint32 of the align kernels' counters
    PC_WORDS = 16
};

__global__ void k_pipe_begin(uint64_t *ctl, uint32_t n_pairs, uint32_t ends) {
    const uint32_t i = threadIdx.x;
    if (i < PC_WORDS) ctl[i] = i == PC_PAIRS ? n_pairs : (i == PC_READS ? (uint64_t)ends * n_pairs : 0ull);
}

// dst = offs[*n_dev], the total of a scan, or 0 with an error bit when it
// exceeds cap or an earlier stage already failed; need keeps the total
__global__ void k_take_total(const uint64_t *offs, const uint64_t *n_dev, uint64_t cap, uint64_t *dst, uint64_t *need,
                             uint32_t *err, uint32_t bit) {
    if (threadIdx.x != 0) return;
    const uint64_t t = (*err) ? 0 : offs[*n_dev];
    *need = t;
    if (t > cap) *err |= bit;
    *dst = (*err) ? 0 : t;
}

}  // namespace

struct bwfm_pipeline {
    bwfm_index *ix = nullptr;
    bwfm_aln_params ap{};
    bwfm_pair_params pp{};
    bwfm_pipeline_params q{};
    void *mem = nullptr;
    // inputs
    uint8_t *bases = nullptr;
    uint64_t *offsets = nullptr;
    uint8_t *maxd = nullptr;
    // search buffers
    u4 *lstack = nullptr, *lcand = nullptr, *sstack = nullptr, *scand = nullptr, *stage = nullptr;
    uint32_t *n_rep = nullptr, *slow_list = nullptr;
    uint64_t *stage_off = nullptr, *part = nullptr;
    // outputs
    uint64_t *hoff = nullptr, *poff = nullptr;
    u4 *hits = nullptr;
    uint32_t *c1 = nullptr, *c2 = nullptr, *cnt = nullptr, *big = nullptr, *pos = nullptr;
    uint8_t *status = nullptr;
    bwfm_pair *pairs = nullptr;
    uint64_t *ctl = nullptr;
    PersistentArgs *pargs = nullptr;
    uint8_t *drows = nullptr, *dflag = nullptr;  // D-array pre-pass output
    uint32_t dstride = 0;
    SplitBufs X{};               // split searches (X.budget 0: off)
    TaskArgs *targs = nullptr;
    uint32_t *lane_read = nullptr;
    // launch shape
    uint32_t lanes = 0, slow_lanes = 0, bs = 0, lstride = 0, stack_cap = 0, worst_stack = 0, scap = 0;
    uint32_t tlanes = 0;  // the split searches' round grid (shares the lane buffers)
    size_t lds = 0;
    uint32_t n_pairs = 0;  // of the batch last set
    uint32_t ends = 2;     // reads per pair record
    bool bound = false;    // input from caller-owned buffers
    bwfm_reads in{};       // the bound input
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};  // first pass start, end; the search's end
    hipStream_t cap = nullptr;  // capture only: nothing runs on it
    bool timed_graph = false, timed_last = false;
    uint64_t jt_gen = 0;        // the index's search tables that the graph was captured with
    bool timing_uncapturable = false;  // a capture with event nodes failed once
};

namespace {

// Enqueue the step.  Every count comes from the control words.
template <int LW>
int pipe_enqueue(bwfm_pipeline *pl, hipStream_t st, bool timed, bool capture) {
    const DevIndex D = dev_index(pl->ix);
    const Params P = make_params(pl->ap);
    const uint32_t nmax = pl->ends * pl->q.max_pairs;
    uint64_t *ctl = pl->ctl;
    uint32_t *actl = reinterpret_cast<uint32_t *>(ctl + PC_ALIGN);
    uint32_t *err = reinterpret_cast<uint32_t *>(ctl + PC_ERR);
    ReadsView rv = pl->bound ? ReadsView{pl->in.bases, pl->in.offsets, pl->in.lengths, pl->in.max_diff, nmax,
                                         pl->in.max_len, ctl + PC_READS}
                             : ReadsView{pl->bases,      pl->offsets,    nullptr, pl->maxd, nmax,
                                         pl->q.max_len, ctl + PC_READS};
    const bool plain = pl->ap.form == BWFM_FORM_PLAIN;
    LaneBufs lb = plain ? LaneBufs{pl->lstack, pl->lcand, 1, pl->lanes, pl->stack_cap, 1, pl->lanes, FAST_CAND,
                                   pl->lstride}
                        : LaneBufs{pl->lstack, pl->lcand, pl->stack_cap, 1, pl->stack_cap, FAST_CAND, 1, FAST_CAND,
                                   pl->lstride};
    ReadOut O{pl->n_rep, pl->c1, pl->c2, pl->status, pl->slow_list, actl, pl->stage,
              reinterpret_cast<unsigned long long *>(actl + 2), pl->q.hit_capacity, pl->stage_off, nullptr, nullptr};
    // under capture the events become event-record nodes of the graph
    auto mark = [&](hipEvent_t e) {
        return capture ? hipEventRecordWithFlags(e, st, hipEventRecordExternal) : hipEventRecord(e, st);
    };
    if (pl->X.budget) k_fill_u32<<<1, 64, 0, st>>>(pl->X.ctl, SPLIT_CTL, 0u);
    if (!plain) {
        const uint32_t nr_up = ((nmax + pl->bs - 1) / pl->bs) * pl->bs;
        k_dscan<LW><<<nr_up / pl->bs, pl->bs, (size_t)pl->bs * pl->lstride, st>>>(
            D, rv, P, pl->drows, pl->dflag, pl->dstride, pl->lstride, pl->X.budget ? pl->X.ctl + SPLIT_LONG : nullptr);
        k_set_args<<<1, 64, 0, st>>>(pl->pargs,
                                     PersistentArgs{rv, lb, O, actl + 1, pl->drows, pl->dflag, pl->dstride, pl->X,
                                                    pl->lane_read},
                                     drain_at_once(pl->bs, pl->lds));
    }
    if (timed) HIPCHK(mark(pl->ev[0]));
    if (plain)
        k_align_plain<LW><<<pl->lanes / pl->bs, pl->bs, pl->lds, st>>>(D, rv, P, lb, O);
    else
        hipLaunchKernelGGL(persistent_kernel<LW>(pl->ap.waves_per_simd), dim3(pl->lanes / pl->bs),
                           dim3(pl->bs),
                           pl->lds, st, D, P, (const PersistentArgs *)pl->pargs);
    if (timed) HIPCHK(mark(pl->ev[1]));
    if (pl->X.budget) enqueue_split<LW>(D, P, pl->X, pl->targs, lb, O, pl->tlanes, st);
    if (timed) HIPCHK(mark(pl->ev[2]));
    LaneBufs sb{pl->sstack, pl->scand, pl->worst_stack, 1, pl->worst_stack, pl->scap, 1, pl->scap, pl->lstride};
    k_align_slow<LW><<<pl->slow_lanes / pl->bs, pl->bs, (size_t)pl->bs * pl->lstride, st>>>(D, rv, P, sb, O, actl + 4);
    HIPCHK(hipGetLastError());
    int rc = scan_counts(pl->n_rep, nmax, pl->hoff, pl->part, st, ctl + PC_READS);
    if (rc) return rc;
    k_take_total<<<1, 64, 0, st>>>(pl->hoff, ctl + PC_READS, pl->q.hit_capacity, ctl + PC_HITS, ctl + PC_NEED_HITS, err,
                                   BWFM_PIPE_E_HITS);
    k_compact<<<blocks(nmax, 256), 256, 0, st>>>(nmax, pl->hoff, pl->stage, pl->stage_off, pl->hits, ctl + PC_READS,
                                                 err);
    // every hit of both ends is located in one pass
    const uint64_t hcap = std::max<uint64_t>(pl->q.hit_capacity, 1);
    k_loc_count<<<blocks(hcap, 256), 256, 0, st>>>(hcap, pl->hits, pl->pp.max_occ, pl->cnt, ctl + PC_HITS);
    rc = scan_counts(pl->cnt, hcap, pl->poff, pl->part, st, ctl + PC_HITS);
    if (rc) return rc;
    k_take_total<<<1, 64, 0, st>>>(pl->poff, ctl + PC_HITS, pl->q.pos_capacity, ctl + PC_POS, ctl + PC_NEED_POS, err,
                                   BWFM_PIPE_E_POSITIONS);
    uint32_t *n_big = reinterpret_cast<uint32_t *>(ctl + PC_BIG);
    rc = locate_fill<LW>(D, hcap, pl->hits, pl->poff, pl->q.pos_capacity, pl->pos, pl->big, n_big, ctl + PC_HITS,
                         ctl + PC_POS, st);
    if (rc) return rc;
    k_sort_small<<<blocks(hcap, 256), 256, 0, st>>>(hcap, pl->poff, pl->pos, pl->big, n_big, ctl + PC_HITS,
                                                  ctl + PC_POS);
    k_sort_big<<<1024, 256, 0, st>>>(pl->poff, pl->pos, pl->big, n_big);
    EndView e1{pl->hoff, pl->hits, pl->poff, pl->pos, 0};
    EndView e2{pl->hoff, pl->hits, pl->poff, pl->pos, 0};  // offsets moved by n on the device
    k_pair<<<blocks(pl->q.max_pairs, 256), 256, 0, st>>>(pl->q.max_pairs, e1, e2, pl->ends == 2 ? 1 : 0, pl->pp.lo,
                                                         pl->pp.hi, pl->pp.mu, pl->pairs, ctl + PC_PAIRS, err);
    HIPCHK(hipGetLastError());
    return BWFM_OK;
}

int pipe_enqueue_any(bwfm_pipeline *pl, hipStream_t st, bool timed, bool capture) {
    return by_layout(pl->ix, [&](auto lw) { return pipe_enqueue<decltype(lw)::value>(pl, st, timed, capture); });
}

}  // namespace

namespace {

void drop_graph(bwfm_pipeline *pl) {
    if (pl->exec) (void)hipGraphExecDestroy(pl->exec);
    if (pl->graph) (void)hipGraphDestroy(pl->graph);
    pl->exec = nullptr;
    pl->graph = nullptr;
}

}  // namespace

extern "C" int bwfm_pipeline_create(const bwfm_index *cix, const bwfm_aln_params *ap, const bwfm_pair_params *pp,
                                    const bwfm_pipeline_params *q, bwfm_pipeline **out) {
    bwfm_index *ix = const_cast<bwfm_index *>(cix);
    if (!out) return fail(BWFM_E_INVAL, "pipeline_create: NULL argument");
    *out = nullptr;
    if (!ix || !ap || !pp || !q) return fail(BWFM_E_INVAL, "pipeline_create: NULL argument");
    if (!check_index(ix)) return fail(BWFM_E_STATE, "pipeline_create: index not uploaded");
    if (q->max_pairs == 0 || q->max_len == 0 || q->max_bases == 0 || q->max_pairs > (1u << 30))
        return fail(BWFM_E_INVAL, "pipeline_create: empty or oversized capacity");
    if (q->max_len > BWFM_MAX_READ) return fail(BWFM_E_TOOLONG, "pipeline_create: max_len above 512");
    if (pp->lo > pp->hi) return fail(BWFM_E_INVAL, "pipeline_create: lo > hi");
    if (int rc = check_aln_params(ap)) return rc;
    std::unique_ptr<bwfm_pipeline> pl(new (std::nothrow) bwfm_pipeline);
    if (!pl) return fail(BWFM_E_NOMEM, "out of host memory");
    pl->ix = ix;
    pl->ap = *ap;
    pl->pp = *pp;
    pl->q = *q;
    pl->ends = q->paired ? 2 : 1;
    const uint32_t nmax = pl->ends * q->max_pairs;
    const uint32_t mlen = q->max_len;
    pl->worst_stack = 8 * (mlen + BWFM_MAX_DIFF) + 1;
    pl->lstride = lds_stride_for(mlen);
    const bool plain = ap->form == BWFM_FORM_PLAIN;
    const uint32_t sbud = plain ? 0u : split_budget_of(*ap);
    pl->bs = block_for(pl->lstride);
    pl->lds = (size_t)pl->bs * pl->lstride + (plain ? 0 : (pl->bs / 64) * sizeof(WaveShare));
    const uint32_t nr_up = ((nmax + pl->bs - 1) / pl->bs) * pl->bs;
    const uint32_t fit = plain ? 0 : by_layout(ix, [&](auto lw) {
        return persistent_lanes<decltype(lw)::value>(pl->bs, pl->lds, ap->waves_per_simd);
    });
    pl->stack_cap = plain ? std::min<uint32_t>(pl->worst_stack, PLAIN_STACK) : pl->worst_stack;
    pl->slow_lanes = std::min<uint32_t>(nr_up, SLOW_LANES);
    pl->scap = ap->max_hits + 1;
    const uint64_t hcap = std::max<uint64_t>(q->hit_capacity, 1);
    const uint64_t pcap = std::max<uint64_t>(q->pos_capacity, 1);
    pl->dstride = ((mlen + 15) / 16) * 16;
    uint32_t blanes = 0;
    SplitShape zs{};
    auto reserve = [&](bool lean) {
        pl->lanes = plain ? nr_up : batched_lanes(fit, nmax, pl->bs, lean);
        pl->tlanes = 0;
        if (sbud) pl->tlanes = by_layout(ix, [&](auto lw) { return task_lanes<decltype(lw)::value>(nr_up, pl->lanes); });
        blanes = std::max(pl->lanes, pl->tlanes);
        zs = split_shape(nmax, mlen, pl->lanes, lean);
        size_t need = 0;
        auto add = [&](size_t b) { need += (b + 255) & ~size_t(255); };
        add(q->max_bases); add((size_t)(nmax + 1) * 8); add(nmax);
        add((size_t)blanes * pl->stack_cap * 16); add((size_t)blanes * FAST_CAND * 16);
        add((size_t)pl->slow_lanes * pl->worst_stack * 16); add((size_t)pl->slow_lanes * pl->scap * 16);
        add((size_t)nmax * 4); add((size_t)nmax * 4); add((size_t)nmax * 8); add(hcap * 16);
        add(scan_part_elems(std::max<uint64_t>(nmax, hcap)) * 8);
        add((size_t)(nmax + 1) * 8); add(hcap * 16); add((size_t)nmax * 4); add((size_t)nmax * 4); add(nmax);
        add(hcap * 4); add(hcap * 4); add((hcap + 1) * 8); add(pcap * 4); add((size_t)q->max_pairs * sizeof(bwfm_pair));
        add(PC_WORDS * 8);
        add(sizeof(PersistentArgs));
        if (!plain) {
            add((size_t)nmax * 2 * pl->dstride);
            add(nmax);
        }
        if (sbud) need += split_bytes(zs) + (size_t)pl->lanes * 4 + 256;
        need += 4096;
        return dev_malloc(&pl->mem, need);
    };
    if (reserve(false) != hipSuccess && (plain || reserve(true) != hipSuccess))
        return fail(BWFM_E_NOMEM, "pipeline: device allocation failed");
    Carver cv{(char *)pl->mem};
    pl->bases = cv.take<uint8_t>(q->max_bases);
    pl->offsets = cv.take<uint64_t>(nmax + 1);
    pl->maxd = cv.take<uint8_t>(nmax);
    pl->lstack = cv.take<u4>((size_t)blanes * pl->stack_cap);
    pl->lcand = cv.take<u4>((size_t)blanes * FAST_CAND);
    pl->sstack = cv.take<u4>((size_t)pl->slow_lanes * pl->worst_stack);
    pl->scand = cv.take<u4>((size_t)pl->slow_lanes * pl->scap);
    pl->n_rep = cv.take<uint32_t>(nmax);
    pl->slow_list = cv.take<uint32_t>(nmax);
    pl->stage_off = cv.take<uint64_t>(nmax);
    pl->stage = cv.take<u4>(hcap);
    pl->part = cv.take<uint64_t>(scan_part_elems(std::max<uint64_t>(nmax, hcap)));
    pl->hoff = cv.take<uint64_t>(nmax + 1);
    pl->hits = cv.take<u4>(hcap);
    pl->c1 = cv.take<uint32_t>(nmax);
    pl->c2 = cv.take<uint32_t>(nmax);
    pl->status = cv.take<uint8_t>(nmax);
    pl->cnt = cv.take<uint32_t>(hcap);
    pl->big = cv.take<uint32_t>(hcap);
    pl->poff = cv.take<uint64_t>(hcap + 1);
    pl->pos = cv.take<uint32_t>(pcap);
    pl->pairs = cv.take<bwfm_pair>(q->max_pairs);
    pl->ctl = cv.take<uint64_t>(PC_WORDS);
    pl->pargs = cv.take<PersistentArgs>(1);
    if (!plain) {
        pl->drows = cv.take<uint8_t>((size_t)nmax * 2 * pl->dstride);
        pl->dflag = cv.take<uint8_t>(nmax);
    }
    if (sbud) {
        pl->X = carve_split(cv, zs, sbud, &pl->targs);
        pl->X.drain = drain_waves(pl->lanes);
        pl->lane_read = cv.take<uint32_t>(pl->lanes);
    }
    if (hipEventCreate(&pl->ev[0]) != hipSuccess || hipEventCreate(&pl->ev[1]) != hipSuccess ||
        hipEventCreate(&pl->ev[2]) != hipSuccess ||
        hipStreamCreateWithFlags(&pl->cap, hipStreamNonBlocking) != hipSuccess) {
        bwfm_pipeline_destroy(pl.release());
        return fail(BWFM_E_DEVICE, "pipeline: event or stream creation failed");
    }
    *out = pl.release();
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_set_reads(bwfm_pipeline *pl, const bwfm_reads *rd, uint32_t n_pairs, void *stream) {
    if (!pl || !rd) return fail(BWFM_E_INVAL, "pipeline_set_reads: NULL argument");
    if (rd->lengths) return fail(BWFM_E_INVAL, "pipeline_set_reads: lengths must be NULL");
    if (rd->n_reads != pl->ends * n_pairs)
        return fail(BWFM_E_INVAL, "pipeline_set_reads: n_reads must be n_pairs times the reads per pair");
    if (n_pairs > pl->q.max_pairs) return fail(BWFM_E_CAPACITY, "pipeline_set_reads: more pairs than max_pairs");
    if (rd->max_len > pl->q.max_len) return fail(BWFM_E_CAPACITY, "pipeline_set_reads: max_len above the pipeline's");
    if (n_pairs && (!rd->bases || !rd->offsets)) return fail(BWFM_E_INVAL, "pipeline_set_reads: NULL reads");
    hipStream_t st = (hipStream_t)stream;
    const uint32_t n = pl->ends * n_pairs;
    if (pl->bound) drop_graph(pl);
    pl->bound = false;
    if (n) {
        uint64_t o[2] = {0, 0};
        HIPCHK(hipMemcpyAsync(&o[0], rd->offsets, 8, hipMemcpyDeviceToHost, st));
        HIPCHK(hipMemcpyAsync(&o[1], rd->offsets + n, 8, hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        if (o[0] != 0) return fail(BWFM_E_INVAL, "pipeline_set_reads: offsets must start at 0");
        if (o[1] > pl->q.max_bases) return fail(BWFM_E_CAPACITY, "pipeline_set_reads: more bases than max_bases");
        if (o[1]) HIPCHK(hipMemcpyAsync(pl->bases, rd->bases, o[1], hipMemcpyDeviceToDevice, st));
        HIPCHK(hipMemcpyAsync(pl->offsets, rd->offsets, (size_t)(n + 1) * 8, hipMemcpyDeviceToDevice, st));
        if (rd->max_diff)
            HIPCHK(hipMemcpyAsync(pl->maxd, rd->max_diff, n, hipMemcpyDeviceToDevice, st));
        else
            HIPCHK(hipMemsetAsync(pl->maxd, pl->ap.max_diff, n, st));
    }
    pl->n_pairs = n_pairs;
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_bind_reads(bwfm_pipeline *pl, const bwfm_reads *rd) {
    if (!pl || !rd || !rd->bases || !rd->offsets) return fail(BWFM_E_INVAL, "pipeline_bind_reads: NULL argument");
    if (rd->n_reads < pl->ends * pl->q.max_pairs)
        return fail(BWFM_E_CAPACITY, "pipeline_bind_reads: fewer read slots than the pipeline's maximum");
    if (rd->max_len > pl->q.max_len) return fail(BWFM_E_CAPACITY, "pipeline_bind_reads: max_len above the pipeline's");
    drop_graph(pl);
    pl->in = *rd;
    pl->in.max_len = pl->q.max_len;  // reads longer than the LDS rows allow are flagged invalid
    pl->bound = true;
    pl->n_pairs = 0;
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_set_count(bwfm_pipeline *pl, uint32_t n_pairs) {
    if (!pl || !pl->bound) return fail(BWFM_E_INVAL, "pipeline_set_count: no bound reads");
    if (n_pairs > pl->q.max_pairs) return fail(BWFM_E_CAPACITY, "pipeline_set_count: more pairs than max_pairs");
    pl->n_pairs = n_pairs;
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_run(bwfm_pipeline *pl, int graph, void *stream) {
    if (!pl) return fail(BWFM_E_INVAL, "pipeline_run: NULL pipeline");
    hipStream_t st = (hipStream_t)stream;
    // the search's tables stay as they are until the step is enqueued
    std::shared_lock<std::shared_mutex> ig(pl->ix->mu);
    bool timed;
    {
        std::lock_guard<std::mutex> g(timing().mu);
        timed = timing().on;
    }
    // the batch size goes in by a launch of its own: the graph's kernels
    // read it from the control words
    k_pipe_begin<<<1, 64, 0, st>>>(pl->ctl, pl->n_pairs, pl->ends);
    HIPCHK(hipGetLastError());
    if (!graph) {
        pl->timed_last = timed;
        return pipe_enqueue_any(pl, st, timed, false);
    }
    if (pl->timing_uncapturable) timed = false;
    if (pl->exec && (pl->timed_graph != timed || pl->jt_gen != pl->ix->jt_gen)) drop_graph(pl);
    if (!pl->exec) {
        // recorded on the pipeline's own stream (the caller's may be the
        // null stream, which cannot be captured); launched on the caller's
        hipGraph_t gph = nullptr;
        for (;;) {
            HIPCHK(hipStreamBeginCapture(pl->cap, hipStreamCaptureModeThreadLocal));
            int rc = pipe_enqueue_any(pl, pl->cap, timed, true);
            hipError_t e = hipStreamEndCapture(pl->cap, &gph);
            (void)hipGetLastError();
            if (!rc && e == hipSuccess) break;
            if (gph) (void)hipGraphDestroy(gph);
            gph = nullptr;
            if (!timed) {
                if (rc) return rc;
                return fail(BWFM_E_DEVICE, std::string("pipeline capture: ") + hipGetErrorString(e));
            }
            // without event nodes: the step still runs, its kernel time is not taken
            pl->timing_uncapturable = true;
            timed = false;
        }
        hipGraphExec_t ex = nullptr;
        hipError_t e;
        e = hipGraphInstantiate(&ex, gph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(gph);
            return fail(BWFM_E_DEVICE, std::string("pipeline graph instantiation: ") + hipGetErrorString(e));
        }
        pl->graph = gph;
        pl->exec = ex;
        pl->timed_graph = timed;
        pl->jt_gen = pl->ix->jt_gen;
    }
    pl->timed_last = pl->timed_graph;
    HIPCHK(hipGraphLaunch(pl->exec, st));
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_finish(bwfm_pipeline *pl, void *stream, bwfm_pipeline_status *out) {
    if (!pl || !out) return fail(BWFM_E_INVAL, "pipeline_finish: NULL argument");
    hipStream_t st = (hipStream_t)stream;
    uint64_t c[PC_WORDS];
    HIPCHK(hipMemcpyAsync(c, pl->ctl, sizeof c, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    out->n_pairs = (uint32_t)c[PC_PAIRS];
    out->error = (uint32_t)c[PC_ERR];
    out->n_hits = c[PC_NEED_HITS];
    out->n_positions = c[PC_NEED_POS];
    out->kernel_ms = 0;
    if (pl->timed_last) {
        float ms = 0;
        float ms_all = 0;
        if (hipEventElapsedTime(&ms, pl->ev[0], pl->ev[1]) == hipSuccess &&
            hipEventElapsedTime(&ms_all, pl->ev[0], pl->ev[2]) == hipSuccess) {
            out->kernel_ms = ms_all;
            std::lock_guard<std::mutex> g(timing().mu);
            auto &e = timing().acc[pl->ap.form == BWFM_FORM_PLAIN ? "align_plain" : "align_persistent"];
            e.first += ms;
            e.second += 1;
            if (pl->ap.form != BWFM_FORM_PLAIN) {
                auto &f = timing().acc["align_search"];
                f.first += ms_all;
                f.second += 1;
            }
        }
    }
    return BWFM_OK;
}

extern "C" int bwfm_pipeline_outputs(bwfm_pipeline *pl, int end, bwfm_aln_result *res, uint64_t **pos_offsets,
                                     uint32_t **positions, bwfm_pair **pairs) {
    if (!pl || (end != 0 && end != 1)) return fail(BWFM_E_INVAL, "pipeline_outputs: bad argument");
    if (end == 1 && pl->ends == 1) return fail(BWFM_E_INVAL, "pipeline_outputs: single-end pipeline has no end 2");
    const uint64_t base = end ? pl->n_pairs : 0;
    if (res) {
        res->hit_offsets = pl->hoff + base;
        res->hits = reinterpret_cast<bwfm_hit *>(pl->hits);
        res->hit_capacity = pl->q.hit_capacity;
        res->c1 = pl->c1 + base;
        res->c2 = pl->c2 + base;
        res->status = pl->status + base;
    }
    if (pos_offsets) *pos_offsets = pl->poff;
    if (positions) *positions = pl->pos;
    if (pairs) *pairs = pl->pairs;
    return BWFM_OK;
}

extern "C" void bwfm_pipeline_destroy(bwfm_pipeline *pl) {
    if (!pl) return;
    drop_graph(pl);
    for (auto &e : pl->ev)
        if (e) (void)hipEventDestroy(e);
    if (pl->cap) (void)hipStreamDestroy(pl->cap);
    dev_free(pl->mem);
    delete pl;
}

extern "C" const char *bwfm_last_error(void) { return last_error().c_str(); }
