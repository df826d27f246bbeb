// Mate rescue on the device: the end of a pair left without a partner is
// aligned locally (affine gaps) inside the reference window that the insert
// bounds allow around its mate's primary (section 3.7 closes the pipeline
// with BWA's pairing step, of which this is the rescue part).
//
// A group of 16, 32 or 64 lanes works on a pair.  The mate's m bases
// are the rows of the dynamic-programming matrices, R consecutive rows per
// lane; the window's reference bases are its columns.  The group sweeps the
// columns in skewed order -- lane l works on column t - l at step t -- so
// each lane receives the row above its first row (the previous lane's last
// row) one step after it was made, through a one-lane DPP shift.  Every cell
// is computed once; a step costs R cells per lane.  A cell is one int32 key
// holding its score, the move it prefers on ties and the window column its
// alignment starts at, so the recurrence's maxima carry the tie order and
// the start along at no extra cost.  The window is decoded from the packed
// reference into LDS first.  Work per pair is m x window cells, a few
// hundred steps: the kernel is bound by integer ALU work, not memory.
//
// Groups of 16 lanes with many rows each, four pairs a wave, are the rule: a
// step's fixed work (the shift, the window base, loop and range checks) is
// then spread over up to 16 cells a lane instead of 2, the rows of a mate
// leave at most one lane's worth idle, and the skew is 15 columns instead of
// 63.  A wave with fewer pairs at hand gives each of them more lanes.  Pairs
// are listed by block and its four waves take from the list, longest mates
// first.  Bound by VALU issue: 89 instructions a step of a wave, 13 a cell
// (four of them for each gap matrix), issued 82% of the time.  Against
// one wave a pair with 1, 2, 4 or 8 rows a lane and a check of every cell
// against the best: 300 k pairs of 36-150 bases, a sixth to rescue, 2.17 ->
// 1.38 ms; of 250 bases 6.6 -> 5.6; 30 k of 150 bases 0.88 -> 0.41; 1 k of
// mixed lengths 0.33 -> 0.12 (a wave there worked off four records in turn).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>

#include "bwfm_internal.h"

using namespace bwfm;

namespace {

constexpr int RB = 256, WAVES = RB / 64;  // threads of a block, waves
// cell keys: score * KS + preference * KP + start column
constexpr int KS = 1 << 15, KP = 1 << 13;
constexpr int NEGK = -(1 << 30);  // no alignment can end here (score -32768)

struct EndView {
    const uint8_t *bases;
    const uint64_t *off;
    const uint32_t *len;  // or NULL: read r ends where read r + 1 starts
};

struct Scores {
    int a, b, o, e, min_score;
};

__device__ __forceinline__ void end_span(const EndView &v, uint32_t r, uint64_t &o0, int &m) {
    o0 = v.off[r];
    if (v.len) {
        m = (int)min(v.len[r], 1u << 20);
    } else {
        const uint64_t o1 = v.off[r + 1];
        m = o1 < o0 ? -1 : (int)min(o1 - o0, (uint64_t)1 << 20);
    }
}

// order this wave's LDS writes before its later reads by other lanes
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// v from the previous lane of the group of G lanes (a DPP shift right by one
// lane); a group's first lane, which has no previous lane, gets 0
template <int G> __device__ __forceinline__ int row_above(int v) {
    if constexpr (G == 16) return __builtin_amdgcn_mov_dpp(v, 0x111 /* row_shr:1 */, 0xF, 0xF, true);
    const int up = __builtin_amdgcn_mov_dpp(v, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
    return G == 64 || (threadIdx.x & (G - 1)) ? up : 0;
}

// One pair record that needs a rescue, as the lane that read it found it.
struct Mate {
    const uint8_t *q;  // the mate's bases
    uint32_t pair, pa;    // the record; where the anchor lies
    int end, m, la, sa;
};

// Rescue a pair per group of G lanes (c: the group's pair, the same in all its
// lanes; on: it has one).  m <= G * R.
template <int G, int R>
__device__ __forceinline__ void rescue_groups(const uint32_t *pac, uint64_t n, const Mate &c, bool on, int lo, int hi,
                              const Scores &S, uint8_t *win, bwfm_rescue *out) {
    int lane = threadIdx.x & (G - 1);
    // (keeps the builds' code from being merged, which held the registers of
    // all: 167 instead of 87)
    asm volatile("" : "+v"(lane));
    const int m = on ? c.m : 0;
    int64_t w0, w1;
    if (c.sa == 0) {
        w0 = c.pa;
        w1 = std::min<int64_t>((int64_t)c.pa + hi, (int64_t)n);
    } else {
        w1 = std::min<int64_t>((int64_t)c.pa + c.la, (int64_t)n);
        w0 = std::max<int64_t>(w1 - hi, 0);
    }
    const int w = on ? (int)std::max<int64_t>(w1 - w0, 0) : 0;
    // the window, in the orientation the query reads it: forward after a +
    // anchor, reversed (from pr + lr - 1 down) after a - anchor
    // (each base stored times 8: the bit offset of its score in a row's profile)
    for (int j = lane; j < w; j += G) {
        const uint64_t p = c.sa == 0 ? (uint64_t)(w0 + j) : (uint64_t)(w1 - 1 - j);
        win[j] = (uint8_t)(8 * ((pac[p >> 4] >> (2 * (p & 15))) & 3));
    }
    // this lane's rows: query base i is mate base m - 1 - i, complemented
    // after a + anchor (the mate then lies on -).  Each row keeps its
    // substitution scores against A, C, G, T as four signed bytes.
    int prof[R];
    const uint8_t *q = c.q + (m - 1 - lane * R);
    const uint32_t miss = (uint8_t)(int8_t)-S.b * 0x01010101u, flip = (uint8_t)(S.a ^ -S.b);
#pragma unroll
    for (int r = 0; r < R; r++) {
        int b = 5;  // rows past the mate: match nothing, never reported
        if (lane * R + r < m) {
            b = q[-r];
            if (c.sa == 0 && b < 4) b = 3 - b;
        }
        prof[r] = (int)(b < 4 ? miss ^ flip << (8 * b) : miss);
    }
    wave_sync();
    const int used = (m + R - 1) / R;        // lanes holding rows
    const int e_min = lo > 0 ? lo - 1 : -1;  // the alignment must end at column >= lo - 1
    // Cells are int32 keys: score * 2^15 + preference * 2^13 + the window
    // column the cell's alignment starts at (< 2^13).  One max over keys then
    // takes the highest score and, on equal scores, the preferred move
    // (diagonal 3 > gap along the reference 2 > gap along the read 1 > no
    // alignment 0), carrying the start column along.  H keys are kept with
    // preference 3, so a gap opened from H arrives with preference 3 and
    // beats the extension of a gap (E kept at 2, F at 1) on equal scores;
    // clearing one bit then brings E back to 2 and F back to 1.  A cell of
    // score 0 in column j is kept as preference 3 and start j + 1, the
    // highest key of score 0 that column can have: a cell one step down the
    // diagonal extends it or starts at its own column, by the same addition.
    // Ho is H less the cost of a gap's first base, which the next column's E
    // and the next row's F both start from.
    const int oek = (S.o + S.e) * KS, ek = S.e * KS;
    int Hp[R], Ho[R], Ep[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        Hp[r] = 3 * KP;
        Ho[r] = 3 * KP - oek;
        Ep[r] = NEGK;
    }
    int outH = 0, outF = 0;  // last row of this lane, current column
    int j = -lane;
    int prevH = 3 * KP + max(j, 0);  // row above, previous column (edge row: score 0)
    int bestK = 0, bj = -1, bi = 0;
    int bestT = KS;  // a cell reports when its key reaches this: a score above the best
    int steps = m > 0 && w > 0 ? w + used - 1 : 0;
#pragma unroll
    for (int k = G; k < 64; k <<= 1) steps = max(steps, __shfl_xor(steps, k));
    steps = __builtin_amdgcn_readfirstlane(steps);
    const int wl = lane < used ? w : 0;  // columns of this lane
    for (int t = 0; t < steps; t++, j++) {
        // the row above this lane's first row, from the previous lane
        const int upH = row_above<G>(outH), upF = row_above<G>(outF);
        const int z = 3 * KP + min(j + 1, KP - 1);
        if ((unsigned)j < (unsigned)wl) {
            const int sh = win[j];
            int Hd = prevH, Huo = upH - oek, F = upF, top = 0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                const int E = max(Ho[r], Ep[r] - ek) & ~KP;
                F = max(Huo, F - ek) & ~(2 * KP);
                const int dg = Hd + __builtin_amdgcn_sbfe(prof[r], sh, 8) * KS;
                const int H = max(max(max(dg, E), F), z) | (3 * KP);
                Hd = Hp[r];
                Hp[r] = H;
                Ep[r] = E;
                Ho[r] = Huo = H - oek;
                top = max(top, H);
            }
            outH = Hp[R - 1];
            outF = F;
            if (top >= bestT && j >= e_min) {
#pragma unroll
                for (int r = 0; r < R; r++)
                    if (Hp[r] >= bestT && lane * R + r < m) {
                        bestK = Hp[r];
                        bestT = (bestK & ~(KS - 1)) + KS;
                        bj = j;
                        bi = lane * R + r + 1;
                    }
            }
        }
        prevH = max(upH, z);  // (a group's first lane: score 0)
    }
    // the first best cell in column order: highest score, then smallest
    // column, then smallest row (each cell lives in exactly one lane)
    const int best = bestK >> 15;
    const uint64_t key = best >= S.min_score ? ((uint64_t)(uint32_t)best << 32) |
                                                   ((uint64_t)(0xFFFFu - (uint32_t)bj) << 16) |
                                                   (uint64_t)(0xFFFFu - (uint32_t)bi)
                                             : 0;
    uint64_t top = key;
    for (int k = G / 2; k > 0; k >>= 1) {
        const uint64_t o = __shfl_xor(top, k);
        top = o > top ? o : top;
    }
    if (on && (top ? key == top : lane == 0)) {
        bwfm_rescue res;
        std::memset(&res, 0, sizeof res);
        if (top) {
            const int start = bestK & (KP - 1);
            res.end = (uint8_t)c.end;
            res.score = (int16_t)best;
            res.len = (uint16_t)(bj - start + 1);
            res.insert = bj + 1;
            if (c.sa == 0) {
                res.strand = 1;
                res.pos = (uint32_t)(w0 + start);
            } else {
                res.strand = 0;
                res.pos = (uint32_t)(w1 - 1 - bj);
            }
        }
        out[c.pair] = res;
    }
    wave_sync();  // the windows are rewritten for the next pairs
}

// the build of the fewest rows per lane that hold m rows (at most ML)
template <int G, int ML>
__device__ __forceinline__ void rescue_by_rows(const uint32_t *pac, uint64_t n, const Mate &c, bool on, int m, int lo,
                                               int hi, const Scores &S, uint8_t *win, bwfm_rescue *out) {
    const int need = (m + G - 1) / G;
#define BWFM_ROWS(R)                                                                \
    if constexpr (G * (R) <= ML)                                                    \
        if (need <= (R)) return rescue_groups<G, (R)>(pac, n, c, on, lo, hi, S, win, out);
    BWFM_ROWS(1) BWFM_ROWS(2) BWFM_ROWS(3) BWFM_ROWS(4) BWFM_ROWS(5) BWFM_ROWS(6) BWFM_ROWS(7) BWFM_ROWS(8)
    BWFM_ROWS(10) BWFM_ROWS(12) BWFM_ROWS(14) BWFM_ROWS(16)
#undef BWFM_ROWS
}

// ML: bound of the mates' lengths (up to 128 the registers leave 5 waves per
// SIMD and more; above, 4 are held to).  A block takes `take` (<= RB) pair
// records, a thread each, and lists those that need a rescue, long mates
// first, so that the mates a wave works on together are of like lengths.  Its
// waves take from the list, each at most `most` (1, 2 or 4) mates at a time,
// fewer where the list holds fewer for each wave.
template <int ML>
__global__ __launch_bounds__(RB, ML <= 128 ? 1 : 4) void k_rescue(const uint32_t *pac, uint64_t n, EndView e1,
                                                                  EndView e2, const bwfm_pair *pairs,
                                                                  uint32_t n_pairs, int lo, int hi, int max_len,
                                                                  Scores S, uint32_t take, int most, int win_stride,
                                                                  bwfm_rescue *out) {
    extern __shared__ uint8_t lds[];
    __shared__ Mate list[RB];
    __shared__ int len[RB];  // 0: no rescue
    __shared__ int count, next;
    const int tid = threadIdx.x;
    const uint32_t p = blockIdx.x * take + (uint32_t)tid;
    Mate c{};
    bool cand = false;
    if ((uint32_t)tid < take && p < n_pairs) {
        const bwfm_pair pr = pairs[p];
        const bool m1 = (pr.flags & BWFM_PF_MAPPED1) != 0, m2 = (pr.flags & BWFM_PF_MAPPED2) != 0;
        // the anchor: the mapped end, or of two the lower search score (end 1 on ties)
        const int anchor = (m1 && m2) ? (pr.score1 <= pr.score2 ? 1 : 2) : (m1 ? 1 : 2);
        c.pair = p;
        c.end = 3 - anchor;
        c.pa = anchor == 1 ? pr.pos1 : pr.pos2;
        c.la = anchor == 1 ? pr.len1 : pr.len2;
        c.sa = anchor == 1 ? pr.strand1 : pr.strand2;
        if (!(pr.flags & BWFM_PF_PAIRED) && (m1 || m2)) {
            const EndView &ev = c.end == 1 ? e1 : e2;
            uint64_t o0;
            end_span(ev, p, o0, c.m);
            c.q = ev.bases + o0;
            cand = c.m > 0 && c.m <= max_len;
        }
        if (!cand) {
            bwfm_rescue z;
            std::memset(&z, 0, sizeof z);
            out[p] = z;
        }
    }
    len[tid] = cand ? c.m : 0;
    if (tid == 0) count = next = 0;
    __syncthreads();
    if (cand) {
        int place = 0;
        for (int i = 0; i < (int)take; i++) place += len[i] > c.m || (len[i] == c.m && i < tid);
        list[place] = c;
        atomicAdd(&count, 1);
    }
    __syncthreads();
    const int all = __builtin_amdgcn_readfirstlane(count), wv = tid >> 6;
    const int share = (all + WAVES - 1) / WAVES;
    most = min(most, share >= 3 ? 4 : share);
    uint8_t *wins = lds + (size_t)wv * most * win_stride;
    for (;;) {
        int i = 0;
        if ((tid & 63) == 0) i = atomicAdd(&next, most);
        i = __builtin_amdgcn_readfirstlane(i);
        if (i >= all) break;
        const int left = min(all - i, most);
        const int at_once = left >= 3 ? 4 : left;
        const int g = (tid & 63) / (64 / at_once);
        const bool on = g < left;
        const Mate x = list[on ? i + g : i];
        const int m0 = __builtin_amdgcn_readfirstlane(list[i].m);  // the longest
        uint8_t *win = wins + (size_t)g * win_stride;
        if (at_once == 4) {
            if constexpr (ML <= 256) rescue_by_rows<16, ML>(pac, n, x, on, m0, lo, hi, S, win, out);
        } else if (at_once == 2) {
            rescue_by_rows<32, ML>(pac, n, x, on, m0, lo, hi, S, win, out);
        } else {
            rescue_by_rows<64, ML>(pac, n, x, on, m0, lo, hi, S, win, out);
        }
    }
}

}  // namespace

extern "C" int bwfm_rescue_mates(const bwfm_index *ix, const bwfm_reads *end1, const bwfm_reads *end2,
                                 uint32_t n_pairs, const bwfm_pair *pairs, const bwfm_pair_params *pp,
                                 const bwfm_rescue_params *rp, bwfm_rescue *out, void *stream) {
    if (!ix || !end1 || !end2 || !pp || (n_pairs && (!pairs || !out)))
        return fail(BWFM_E_INVAL, "rescue_mates: NULL argument");
    if (ix->device < 0 || !ix->d_pac) return fail(BWFM_E_STATE, "rescue_mates: index not uploaded");
    if (n_pairs && (!end1->bases || !end1->offsets || !end2->bases || !end2->offsets))
        return fail(BWFM_E_INVAL, "rescue_mates: NULL reads");
    if (end1->n_reads < n_pairs || end2->n_reads < n_pairs)
        return fail(BWFM_E_INVAL, "rescue_mates: fewer reads than pairs");
    if (pp->lo > pp->hi) return fail(BWFM_E_INVAL, "rescue_mates: lo > hi");
    if (pp->hi > BWFM_RESCUE_MAX_WINDOW) return fail(BWFM_E_INVAL, "rescue_mates: hi above the largest window");
    const bwfm_rescue_params q = rp ? *rp : bwfm_rescue_params BWFM_RESCUE_DEFAULTS;
    if (q.match < 1 || q.match > 32 || q.mismatch < 0 || q.mismatch > 64 || q.gap_open < 0 || q.gap_open > 64 ||
        q.gap_extend < 0 || q.gap_extend > 64 || q.min_score < 1)
        return fail(BWFM_E_INVAL, "rescue_mates: scores out of range");
    const uint32_t max_len = std::max(end1->max_len, end2->max_len);
    if (max_len > BWFM_MAX_READ) return fail(BWFM_E_TOOLONG, "rescue_mates: max_len above 512");
    if (n_pairs == 0) return BWFM_OK;
    hipStream_t st = (hipStream_t)stream;
    const EndView e1{end1->bases, end1->offsets, end1->lengths}, e2{end2->bases, end2->offsets, end2->lengths};
    const Scores S{q.match, q.mismatch, q.gap_open, q.gap_extend, q.min_score};
    const int hi = std::max(pp->hi, 0);
    const int win_stride = std::max((hi + 15) & ~15, 16);
    // records a block takes: as many as it has waves while all blocks run at
    // once (eight a CU), more of a larger batch so that its waves find four
    // mates at a time.  Blocks of 256 records end less evenly than of 128 unless
    // there are many (300 k pairs of 36-150 bases at 64 / 128 / 256: 1.45 /
    // 1.38 / 1.55 ms; 1 M of 100 bases, 6% to rescue: 1.54 at 128, 1.46 at 256)
    uint32_t take = WAVES;
    while (take < RB && (uint64_t)take * 2048 < n_pairs && (take < 128 || (uint64_t)take * 4096 <= n_pairs)) take *= 2;
    const uint32_t grid = (n_pairs - 1) / take + 1;
    // mates a wave works on at once: as many as its lanes hold the rows of
    // and 48 KB of LDS hold the windows of
    int most = max_len <= 256 ? 4 : 2;
    while (most > 1 && (size_t)WAVES * most * win_stride > 48 * 1024) most /= 2;
    const size_t lds = (size_t)WAVES * most * win_stride;
    const uint32_t *pac = (const uint32_t *)ix->d_pac;
    const int ml = (int)max_len;
    const auto kernel = max_len <= 64 ? k_rescue<64> : max_len <= 128 ? k_rescue<128> : max_len <= 256 ? k_rescue<256>
                                                                                                       : k_rescue<512>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(RB), lds, st, pac, ix->n, e1, e2, pairs, n_pairs, pp->lo, hi, ml, S,
                       take, most, win_stride, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(BWFM_E_DEVICE, std::string("rescue_mates: launch: ") + hipGetErrorString(e));
    return BWFM_OK;
}
