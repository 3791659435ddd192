// knnf_kernels.hip -- KNN filtering kernels for CDNA4 (gfx950), wave64.
//
// Method (Lazcano et al., Sec. II.C.3): for each pixel q, find the K nearest
// window pixels under the Eq. 1 distance of the features (I, lambda*row,
// lambda*col) and average their class probabilities (Eq. 2); the class map is
// the argmax of the summed probabilities.  The window is R rows above and below
// q at full width, clipped at the frame edges (Sec. III.A.3).
//
// Arithmetic contract (identical bits to any other conforming implementation):
//   fr(x) = fl32(lambda * (float)x)
//   a = fl32(fr(r) - fr(i)), b = fl32(fr(c) - fr(j)), e = fl32(I_q - I_p)
//   d = fmaf(e, e, fmaf(b, b, fl32(a * a)))
//   order: key = (bits(d) << 32) | (i*W + j), ascending (d >= +0, so the bit
//   pattern orders like the value)
//   S_c = ((+0 + P[n_0][c]) + P[n_1][c]) + ... in key order; O_c = fl32(S_c/K)
//   class = lowest c with maximal S_c
// The file is built with -ffp-contract=off, so every * and - below is one
// binary32 operation and fmaf is the only fused operation.
//
// Work decomposition (not the paper's; designed for 64-wide wavefronts):
//   * One wavefront task = a tile of QR x QC query pixels (default 1 x 8).
//     Per-query state lives in VGPRs and a small per-wavefront LDS block.
//   * pass A (bound): the 64 or 128 candidates (see SMALL_K) of a compact block
//     around each query (8 rows x 8 or 16 columns where the window allows) are
//     evaluated and ranked for all Q queries at once by a segmented network;
//     any distance with at least K block candidates at or below it bounds the
//     query's final K-th key from above.  The block is ranked as two interleaved
//     groups (16-bit keys, both in one packed network); the bound is the larger
//     of the groups' ceil(K/2)-th keys.
//   * pass B (collect): candidates with d <= d_K are appended to a per-query
//     LDS buffer with ballot + mbcnt; a full buffer is cut down by a tighter
//     bound, and a tile that keeps filling them is done over in parts with larger
//     ones (crowded_tile).  Two scans:
//       - pruned (default): patches of 64 candidates, as high as the block of
//         rows, swept over the rows and columns whose spatial lower bound is
//         within some query's bound (bit-identical: every term of Eq. 1 is
//         >= 0 and rounding is monotone);
//       - exhaustive: every window row in 64-column chunks, four rows per
//         group, one coalesced 256-byte load per row shared by all queries.
//   * Final selection: one segmented sort of 32-bit packed keys (distance
//     bits | buffer slot) with exact (d, idx) repair of equal distance parts.
//   * The tail is fused: gather the K neighbours' probabilities (L2-resident),
//     sum in key order, divide, argmax, and write the outputs.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "knnf_device.h"
#include "knnf_networks.h"
#include "knnf_select.h"

namespace knnf {
namespace {

constexpr uint64_t KEY_INF = ~0ull;
constexpr int WAVE = 64;
constexpr int A2ROWS = 64;  // window rows per block of the LDS a2 table
constexpr int A2PAD = 4;    // padding rows (NaN) so a 4-row group may start anywhere
constexpr int MAXC = 16;
// Pass A looks at 64 candidates per query for K up to SMALL_K (8-query tiles),
// 128 beyond.  The larger block's tighter bound lets fewer candidates through
// (K = 40: 45 instead of 48 of the 64 buffer slots, and 1 % instead of 4 % of
// the queries overflow them), but takes twice the distances and a network of
// twice the registers.  380 x 480, smaller against larger block: lambda 0.01,
// K = 32 49.5 against 51.3 us, K = 40 53.7 / 54.1 (1000 x 1000: 205 / 216),
// K = 48 71 / 64; lambda 1, K = 36 41.0 / 47.5, K = 44 43.7 / 49.6, K = 52
// 79 / 52.
constexpr int SMALL_K = 40;
// A tile of such a K with a bound wider than eight pixels' spatial distance (its
// K nearest reach far beyond the 8 x 8 block: outliers, about 1 % of the tiles)
// takes the larger block after all: its own bound let whole regions through
// (a 50 x 50 frame with a few such pixels 11.4 instead of 9.6 us; five pixels
// instead of eight, 26 % of the tiles, cost 1024 frames of 50 x 50 708 instead of
// 666 us).
constexpr float WIDE2 = 64.0f;

__device__ __forceinline__ int lane_id() {
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
// The same, computed where it stands: the compiler moves what depends on the lane
// alone out of loops.  The rare paths use it (the 21 lane masks of a 64-key sort
// cost every tile 110 vector instructions in front of the scan), and the
// persistent kernel's tiles, whose lane constants its claim loop kept in registers
// (108 bytes of them spilled).
__device__ __forceinline__ int lane_id_here() {
    int L = lane_id();
    asm volatile("" : "+v"(L));
    return L;
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniu(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ int mbcnt(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Orders LDS traffic of one wavefront (lanes exchange data through LDS).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ uint64_t make_key(float d, int idx) {
    return ((uint64_t)__float_as_uint(d) << 32) | (uint64_t)(uint32_t)idx;
}

// ---- cross-lane exchange with the partner lane L ^ J (no LDS traffic
// except J = 4, which uses the LDS crossbar swizzle)
template <int J>
__device__ __forceinline__ uint32_t xlane(uint32_t v, int L) {
    if constexpr (J == 1) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false);
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false);
    } else if constexpr (J == 4) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (4 << 10));
    } else if constexpr (J == 8) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xF, 0xF, false);
    } else if constexpr (J == 16) {
        // permlane16_swap(v, v) yields rows {0,0,2,2} and {1,1,3,3}
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (L & 16) ? r[0] : r[1];
    } else {
        // permlane32_swap(v, v) yields halves {lo,lo} and {hi,hi}
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (L & 32) ? r[0] : r[1];
    }
}

// Compare-exchange of 64-bit keys (hi, lo) with partner L ^ J inside bitonic
// stage S (S = 64: the final, all-ascending stage).
template <int S, int J>
__device__ __forceinline__ void cx_key(uint32_t& hi, uint32_t& lo, int L) {
    const uint32_t ph = xlane<J>(hi, L), pl = xlane<J>(lo, L);
    const uint64_t me = ((uint64_t)hi << 32) | lo, ot = ((uint64_t)ph << 32) | pl;
    const bool flip = ((L & J) != 0) != (S < WAVE && (L & S) != 0);
    const bool take = (ot < me) != flip;  // keys are unique apart from KEY_INF
    hi = take ? ph : hi;
    lo = take ? pl : lo;
}

template <int S, int J>
__device__ __forceinline__ void stage_key(uint32_t& hi, uint32_t& lo, int L) {
    cx_key<S, J>(hi, lo, L);
    if constexpr (J > 1) stage_key<S, J / 2>(hi, lo, L);
}

// Ascending bitonic sort of one 64-bit key per lane across the wavefront.
__device__ __forceinline__ uint64_t sort64(uint64_t key, int L) {
    uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
    stage_key<2, 1>(hi, lo, L);
    stage_key<4, 2>(hi, lo, L);
    stage_key<8, 4>(hi, lo, L);
    stage_key<16, 8>(hi, lo, L);
    stage_key<32, 16>(hi, lo, L);
    stage_key<64, 32>(hi, lo, L);
    return ((uint64_t)hi << 32) | lo;
}

// ---- segmented networks: the Q queries of a tile together.  A segment of P
// lanes (4, 8 or 16) holds one query's P * E elements, E registers a lane; the
// sorted order is element lp * E + r in register r of the segment's lane lp.
//
// Each lane sorts its E elements, then runs of E, 2E, 4E elements are merged
// bitonically: stage KS compares e with its mirror e ^ (KS - 1) (both runs
// ascending -> the smaller half in the lower lanes, as two bitonic halves), then
// half-cleaners compare e with e ^ D across lanes (D >= E) and within the lane.
// The tiles issue one vector instruction after another, so the count of
// instructions is what a network costs.
//
// 32-bit keys (final selection).  The median of an element, its partner and 0 or
// all ones is the smaller or the larger of the two, so a cross-lane comparison
// is a DPP move and a v_med3_u32 with a constant of the lane.  Within a lane,
// with lo / md / hi the sorted three of four elements, the fourth is inserted by
// min(lo, d), med3(lo, md, d), med3(md, hi, d), max(hi, d): 7 instructions for a
// sort of 4 where 5 compare-exchanges take 10.  Two sorted pairs merge in 5 (6):
// a cyclic bitonic sequence a, b, c, d in 6 (8), because min(b, d) never exceeds
// max(a, c) in it nor max(b, d) falls below min(a, c).  8 queries x 64 elements:
// 186 instructions (214 with compare-exchanges, negating the values of the lanes
// that keep the larger element).
//
// Pairs of 16-bit keys (pass A: two groups of candidates a query, one in each
// half).  There is no packed median; lanes that keep the larger element hold
// their keys complemented and keep the smaller of their own and the partner's
// complement (v_not_b32 with DPP, v_pk_min_u16, and v_xor_b32 where the set of
// such lanes changes).  Within a lane a bitonic sequence may lie in either
// direction, so odd lanes stay complemented, hence sorted the other way round,
// while lanes merge their own elements; a mirror stage, whose partner lane
// differs in bit 0, then pairs equal registers, and a half-cleaner with lane ^ 1
// opposite ones.

// Ascending sort of each segment of P lanes.
template <int P, int E>
__device__ __forceinline__ void seg_sort(uint32_t (&x)[E], int lp) {
    static_assert(P == 4 || P == 8 || P == 16, "segment width");
    const uint32_t k0 = (lp & 1) ? ~0u : 0u, k1 = (lp & 2) ? ~0u : 0u;
    lane_sort<E>(x);
    cross<DPP_XOR1, true>(x, k0);  // runs of 2E
    lane_merge<E>(x);
    cross<DPP_XOR3, true>(x, k1);  // runs of 4E
    cross<DPP_XOR1, false>(x, k0);
    if constexpr (P >= 8) {
        const uint32_t k2 = (lp & 4) ? ~0u : 0u;
        lane_merge<E>(x);
        cross<DPP_XOR7, true>(x, k2);  // runs of 8E
        cross<DPP_XOR2, false>(x, k1);
        cross<DPP_XOR1, false>(x, k0);
        if constexpr (P == 16) {
            lane_merge<E>(x);
            cross<DPP_XOR15, true>(x, (lp & 8) ? ~0u : 0u);  // runs of 16E
            cross_xor4(x, k2);
            cross<DPP_XOR2, false>(x, k1);
            cross<DPP_XOR1, false>(x, k0);
        }
    }
    lane_merge<E>(x);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ void pk_cx(uint32_t& a, uint32_t& b) {
    const uint32_t lo = pk_min(a, b);
    b = pk_max(a, b);
    a = lo;
}

// n0 .. n3 = ~y0 .. ~y3 of the lanes CTRL selects (a DPP operand must not have
// been written in the two instructions before: s_nop 1)
#define KNNF_NOT4(CTRL)                                                          \
    asm("s_nop 1\n\t"                                                            \
        "v_not_b32_dpp %0, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"           \
        "v_not_b32_dpp %1, %5 " CTRL " row_mask:0xf bank_mask:0xf\n\t"           \
        "v_not_b32_dpp %2, %6 " CTRL " row_mask:0xf bank_mask:0xf\n\t"           \
        "v_not_b32_dpp %3, %7 " CTRL " row_mask:0xf bank_mask:0xf"               \
        : "=&v"(n[r]), "=&v"(n[r + 1]), "=&v"(n[r + 2]), "=&v"(n[r + 3])         \
        : "v"(x[r]), "v"(x[r + 1]), "v"(x[r + 2]), "v"(x[r + 3]))
// Each register keeps the smaller of its own keys and the complemented ones of
// lane L ^ X (X = 1, 2, 3: quad_perm; 7: row_half_mirror), in the same register
// or (OPP) registers paired r, E-1-r.
template <int X, bool OPP, int E>
__device__ __forceinline__ void pk_cross(uint32_t (&x)[E]) {
    uint32_t n[E];
#pragma unroll
    for (int r = 0; r < E; r += 4) {
        if constexpr (X == 1) KNNF_NOT4("quad_perm:[1,0,3,2]");
        else if constexpr (X == 2) KNNF_NOT4("quad_perm:[2,3,0,1]");
        else if constexpr (X == 3) KNNF_NOT4("quad_perm:[3,2,1,0]");
        else KNNF_NOT4("row_half_mirror");
    }
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = pk_min(x[r], n[OPP ? E - 1 - r : r]);
}
#undef KNNF_NOT4
template <int E>
__device__ __forceinline__ void pk_lane_merge(uint32_t (&x)[E]) {
#pragma unroll
    for (int d = E / 2; d >= 1; d /= 2)
#pragma unroll
        for (int r = 0; r < E; ++r)
            if (!(r & d)) pk_cx(x[r], x[r | d]);
}
template <int E>
__device__ __forceinline__ void pk_flip(uint32_t (&x)[E], uint32_t mask) {
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] ^= mask;
}
// The segment's sorted element lp * E + rank in each lane (rank uniform): the last
// merge within the lane follows the one path to it, E - 1 minima of keys that are
// complemented on the levels where the larger half is wanted.
template <int P, int E>
__device__ __forceinline__ uint32_t pk_seg_rank(uint32_t (&x)[E], int lp, int rank) {
    static_assert(P == 4 || P == 8, "segment width");
    const uint32_t m0 = (lp & 1) ? ~0u : 0u, m1 = (lp & 2) ? ~0u : 0u;
    pk_flip(x, m0);
    // Batcher's odd-even merge sort of the lane's elements
#pragma unroll
    for (int p = 1; p < E; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < E; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < E && (i + j) / (2 * p) == (i + j + k) / (2 * p))
                        pk_cx(x[i + j], x[i + j + k]);
    pk_cross<1, false>(x);  // runs of 2E
    pk_lane_merge(x);
    pk_flip(x, m0 ^ m1);
    pk_cross<3, false>(x);  // runs of 4E
    pk_flip(x, m0 ^ m1);
    pk_cross<1, true>(x);
    if constexpr (P == 8) {
        const uint32_t m2 = (lp & 4) ? ~0u : 0u;
        pk_lane_merge(x);
        pk_flip(x, m0 ^ m2);
        pk_cross<7, false>(x);  // runs of 8E
        pk_flip(x, m2 ^ m1);
        pk_cross<2, false>(x);
        pk_flip(x, m1 ^ m0);
        pk_cross<1, true>(x);
    }
    uint32_t was = m0;
#pragma unroll
    for (int d = E / 2; d >= 1; d /= 2) {
        const uint32_t up = (rank & d) ? ~0u : 0u;
#pragma unroll
        for (int r = 0; r < 2 * d; ++r) x[r] ^= was ^ up;
#pragma unroll
        for (int r = 0; r < d; ++r) x[r] = pk_min(x[r], x[r + d]);
        was = up;
    }
    return x[0] ^ was;
}

// The upper halves of two binary32 bit patterns as a pair of 16-bit keys
// (rounded down: d < (key + 1) << 16).
__device__ __forceinline__ uint32_t pack_hi(uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

// Buffer slots are prefilled with the query's own index and, as distance bits,
// PAD + 64 slot: above those of any candidate that the packed final selection
// orders (distance bits up to BIG; queries with a larger bound take the exact
// merge), and no two empty slots alike once the slot bits are set aside.
constexpr uint32_t PAD = 0x7f7f0000u;
constexpr uint32_t BIG = PAD - 1;

// When a tile counts as crowded (see crowded_tile).  A cut of a full buffer costs about 400
// cycles and frees a part of the 64 - K slots beyond the K that stay, so the larger K, the
// fewer cuts are worth making: pruned scan, 64 - K cuts for eight queries (380 x 480, K =
// 40 and 64, lambda 0.01: 56.4 and 144 us; 16 cuts for every K 56.4 and 160, 48 cuts 57 and
// 191; without crowded tiles 56.2 and 175), and more than eight steps of the block to go (K =
// 60, lambda 1: 86 us, 107 wherever it stands).  The whole-window scan meets the nearest
// candidates first and crowds only for K near 64: 48 cuts there (K = 64, lambda 0.001: 945
// us; 80 cuts 1,109, without 1,414; lambda 0.01 506, 514, 472), else 32 a query.
__device__ __forceinline__ int crowded_cuts(int Q, int K) { return max(1, (64 - K) * Q / 8); }
__device__ __forceinline__ int crowded_cuts_all(int Q, int K) { return Q * (K < 58 || Q > 8 ? 32 : 6); }
constexpr int CROWDED_STEPS = 8;
// Candidates that a cut leaves where it stops early: the middle between K and 64; with 128
// slots, which fill up slowly, a quarter of the way (uniform noise, K = 52: 373 us, 390).
template <int SLOTS>
__device__ __forceinline__ int cut_target(int K) { return SLOTS > WAVE ? (3 * K + SLOTS) / 4 : (K + SLOTS) / 2; }
constexpr int ROWS = 32;  // neighbour rows staged at a time in Eq. 2 (four classes)

// Per-wavefront LDS state of one tile of QR x QC query pixels.
template <int E>
__device__ __forceinline__ int row_at(int r) { return E >= 8 ? r + (r >> 3) : r; }

template <int QR, int QC, int NSLOT = WAVE>
struct alignas(16) TileState {
    static constexpr int Q = QR * QC, SLOTS = NSLOT;
    union {
        uint32_t pend[Q][2][SLOTS]; // candidates that passed the bound, unsorted: distance
                                 // bits, linear indices
        // four classes: the neighbours' probability rows, in order; where a lane
        // stores eight, one row is skipped after them (row_at: without the gap half
        // the lanes of a segment met on each bank; 1000 x 1000, K = 40: 203 us
        // against 210)
        float4 rows[Q][ROWS + ROWS / 8 + 1];
        struct {                 // other class counts:
            // neighbours' linear indices in order; rows padded by 16 bytes so that
            // the queries' rows start on different banks (Eq. 2 reads the same
            // entry of every query at once)
            uint32_t list[Q][WAVE + 4];
            float sums[Q][MAXC + 1]; // class sums for the argmax; the odd row stride
                                 // spreads the queries over the banks
        };
    };
    uint32_t tauhi[Q];        // distance bits of the current bound on the K-th key
    float iq[Q];              // I of each query pixel (NaN for pixels off the frame)
    int cnt[Q];               // pending entries (mirror of the scan's registers)
};

// The exhaustive scan also keeps a table of row terms; the pruned scan
// computes them per lane.
template <int QR, int QC, bool PRUNE, int NSLOT = WAVE>
struct alignas(16) TileLds : TileState<QR, QC, NSLOT> {
    float a2t[A2ROWS + A2PAD][QR];  // fl32(a*a) for a block of window rows (NaN: inactive)
};
template <int QR, int QC, int NSLOT>
struct alignas(16) TileLds<QR, QC, true, NSLOT> : TileState<QR, QC, NSLOT> {};

// Coordinate feature fr(x) = fl32(lambda * (float)x).
__device__ __forceinline__ float feat(float lam, int x) { return lam * (float)x; }

// Put query q's cnt candidates in exact (d, idx) order and write its neighbour
// outputs, for bounds beyond the packed keys' range.  The buffer then holds the
// indices in order under distance parts that only number them.
template <int QR, int QC, int NSLOT>
__device__ __forceinline__ void order_query(TileState<QR, QC, NSLOT>& S, const FrameDesc& f, int r0, int c0,
                                            int q, int cnt) {
    const int L = lane_id_here();
    const int W = f.W, K = f.K;
    const int r = r0 + q / QC, c = c0 + q % QC;
    uint64_t key = KEY_INF;
    if (L < cnt) key = make_key(__uint_as_float(S.pend[q][0][L]), (int)S.pend[q][1][L]);
    key = sort64(key, L);
    wave_sync();
    // a slot without a candidate (only with non-finite inputs, or inputs that
    // change during the launch) gathers the query pixel's own row, never an
    // address outside the frame
    S.pend[q][0][L] = (uint32_t)L << 6;
    S.pend[q][1][L] = key == KEY_INF ? (uint32_t)r * (uint32_t)W + (uint32_t)c : (uint32_t)key;
    if (L < K) {
        const size_t pix = (size_t)r * W + c;
        if (f.out_nbr) f.out_nbr[pix * K + L] = (int32_t)(uint32_t)key;
        if (f.out_dist) f.out_dist[pix * K + L] = __uint_as_float((uint32_t)(key >> 32));
    }
    wave_sync();
}

// Cut query q's buffer down to at most `room` candidates: nb pending ones and this
// step's (dn: each lane's distance bits, all ones for none; idx its linear index), more
// than room of them within the bound.  Any distance t with at least K candidates at or
// below it bounds the K-th key, so a t that leaves few enough of them is found by
// bisection (its counts are ballots; it stops early at `few`), the buffer keeps those,
// and the bound becomes t.  Where equal distances leave no such t, the smallest t with K
// candidates is taken, and of those at t the ones up to an index that is found
// the same way: ties go by the index.  About 100 instructions, 200 with ties.
template <int QR, int QC, int NSLOT>
__device__ __forceinline__ void tighten(TileState<QR, QC, NSLOT>& S, int q, int nb, uint32_t dn, uint32_t idx,
                                        uint32_t bound, int K, uint32_t own, int room, int few) {
    constexpr int B = NSLOT / WAVE;  // a lane's slots
    const int L = lane_id_here();
    uint32_t kb[B], ib[B], db[B];
#pragma unroll
    for (int v = 0; v < B; ++v) {
        kb[v] = S.pend[q][0][WAVE * v + L];
        ib[v] = S.pend[q][1][WAVE * v + L];
        db[v] = WAVE * v + L < nb ? kb[v] : ~0u;
    }
    auto count = [&](uint32_t t) {
        int n = __builtin_popcountll(ballot(dn <= t));
#pragma unroll
        for (int v = 0; v < B; ++v) n += __builtin_popcountll(ballot(db[v] <= t));
        return n;
    };
    int n = NSLOT + WAVE;
    uint32_t hi = cut_distance(bound, K, few, n, count), ih = 0;  // ih: of those at hi, indices below it
    if (n > room) {
        if (hi == 1 && count(0) >= K) hi = 0;  // (the bisection never looks at 0)
        ih = 0x80000000u;
        n = count(hi);
        if (n > room) {
            const uint64_t ln = ballot(dn < hi), en = ballot(dn == hi);
            uint64_t lb[B], eb[B];
#pragma unroll
            for (int v = 0; v < B; ++v) {
                lb[v] = ballot(db[v] < hi);  // fewer than K, all in all
                eb[v] = ballot(db[v] == hi);
            }
            ih = cut_index(K, few, n, [&](uint32_t i) {
                int c = __builtin_popcountll(ln | (en & ballot(idx < i)));
#pragma unroll
                for (int v = 0; v < B; ++v) c += __builtin_popcountll(lb[v] | (eb[v] & ballot(ib[v] < i)));
                return c;
            });
        }
    } else {
        ih = 0x80000000u;
    }
    wave_sync();
    auto put = [&](int slot, uint32_t dist, uint32_t id) {
        S.pend[q][0][slot] = dist;
        S.pend[q][1][slot] = id;
    };
    int at = 0;
#pragma unroll
    for (int v = 0; v < B; ++v) {
        const bool keep = db[v] < hi || (db[v] == hi && ib[v] < ih);
        const uint64_t m = ballot(keep);
        if (keep) put(at + mbcnt(m), kb[v], ib[v]);
        at += __builtin_popcountll(m);
    }
    const bool keep = dn < hi || (dn == hi && idx < ih);
    const uint64_t m = ballot(keep);
    if (keep) put(at + mbcnt(m), dn, idx);
#pragma unroll
    for (int v = 0; v < B; ++v)
        if (WAVE * v + L >= n) put(WAVE * v + L, PAD + 64u * (uint32_t)(WAVE * v + L), own);
    if (L == 0) {
        S.cnt[q] = n;
        S.tauhi[q] = hi;
    }
    wave_sync();
}

// Buffer counts as the pruned scan holds them: 4 * (n + SLOTS - 1), the byte offset of
// the next slot plus a bias for which a count beyond SLOTS sets the bit 8 * SLOTS.
template <int SLOTS>
__device__ __forceinline__ int pend_code(int n) { return 4 * (n + SLOTS - 1); }
template <int SLOTS>
__device__ __forceinline__ int pend_count(int code) { return code / 4 - (SLOTS - 1); }

// Append to the buffers of queries q .. q + 3 the lanes of masks m (distances d,
// linear index idx); cnt: the queries' counts before, slot0: the buffers' LDS
// address, less the counts' bias, in words.  Written out because the compiler
// guards each store by a branch: 16 scalar instructions per query and step where
// two are needed, with nearly every query storing in nearly every step.  The
// caller's branch on the counts orders the compares before the masks' first
// vector read; all 64 lanes are active.  LDS accesses of a wavefront stay in order.
template <int SLOTS>
__device__ __forceinline__ void append4(int q, const uint64_t* m, const float* d, const int* cnt,
                                        uint32_t idx, uint32_t slot0) {
    constexpr int B = SLOTS / WAVE;  // a buffer half in units of the store's offsets
    uint32_t t;
#define KNNF_APPEND(M, D, N, O)                                    \
    "s_mov_b64 exec, %[" #M "]\n\t"                                \
    "s_cbranch_execz .Lskip%=_" #O "\n\t"                          \
    "v_mbcnt_lo_u32_b32 %[t], exec_lo, %[s]\n\t"                   \
    "v_mbcnt_hi_u32_b32 %[t], exec_hi, %[t]\n\t"                   \
    "v_lshl_add_u32 %[t], %[t], 2, %[" #N "]\n\t"                  \
    "ds_write2st64_b32 %[t], %[" #D "], %[i] offset0:%[" #O "0] offset1:%[" #O "1]\n"  \
    ".Lskip%=_" #O ":\n\t"
    asm volatile(KNNF_APPEND(ma, da, na, a) KNNF_APPEND(mb, db, nb, b) KNNF_APPEND(mc, dc, nc, c)
                     KNNF_APPEND(md, dd, nd, d) "s_mov_b64 exec, -1"
                 : [t] "=&v"(t)
                 : [ma] "s"(m[0]), [mb] "s"(m[1]), [mc] "s"(m[2]), [md] "s"(m[3]), [da] "v"(d[0]),
                   [db] "v"(d[1]), [dc] "v"(d[2]), [dd] "v"(d[3]), [na] "s"(cnt[0]), [nb] "s"(cnt[1]),
                   [nc] "s"(cnt[2]), [nd] "s"(cnt[3]), [i] "v"(idx), [s] "v"(slot0), [a0] "i"(2 * B * q),
                   [a1] "i"(2 * B * q + B), [b0] "i"(2 * B * (q + 1)), [b1] "i"(2 * B * (q + 1) + B),
                   [c0] "i"(2 * B * (q + 2)), [c1] "i"(2 * B * (q + 2) + B), [d0] "i"(2 * B * (q + 3)),
                   [d1] "i"(2 * B * (q + 3) + B)
                 : "memory");
#undef KNNF_APPEND
}

// Pruned scan (bit-identical to the exhaustive one).  Every term of Eq. 1 is
// >= 0 and binary32 rounding is monotone, so fmaf(b, b, a2) with the smallest
// |b| and a2 of a set of candidates bounds all their distances from below;
// a set whose bound exceeds every query's current bound tau cannot hold a
// neighbour.  The scan visits the window in patches of PR rows x SW = 64/PR
// columns: lane L holds row blk + (L % PR), column jc + L / PR, so a lane's row
// term stays fixed while a row block is swept column step by column step.
//   * live rows: rows where some query's row term alone is within its bound
//     (its own column has b = 0), in equal blocks of at most 2^(lpr+1) = 16, 32 or
//     64 rows (the plan's window chunk);
//   * per block of live rows: the tile's own columns and those right and left of
//     it whose bound is within some query's (a prefix on each side).
// A patch has the block's height whatever that is, so nearly every lane holds a
// row that can matter and both ends of the sweep are used: K = 16 at 380 x 480
// 32.2 us against 36.2 with patches of 16 x 4, 400 x 400 at lambda = 1 40.7
// against 45.3, K = 40 56.3 against 58.7 (blocks of at most 16 rows 57.6, 12: 57.0,
// 8: 59.0; 1000 x 1000 231, 233, 236, 248).
// Survivors (d <= tau's distance) are appended per query with ballot +
// mbcnt; a full buffer is cut down to the candidates within a tighter bound
// (tighten).  After `cuts` of those the scan is given up and returns true (see
// crowded_tile); the bounds that it reached stay.
template <int QR, int QC, int NSLOT>
__device__ __forceinline__ bool scan_pruned(TileState<QR, QC, NSLOT>& S, const FrameDesc& f, int r0,
                                            int c0, int nqr, int nqc, int lpr, int L,
                                            const float (&iq)[QR * QC],
                                            uint32_t (&th)[QR * QC], int (&cnt)[QR * QC],
                                            unsigned long long& pairs, int cuts) {
    constexpr int Q = QR * QC, FULL = 8 * NSLOT;
    const int H = f.H, W = f.W, R = f.R;
    const float lam = f.lambda;
    const float* __restrict__ pc1 = f.pc1;
    const float pinf = __int_as_float(0x7f800000), qnan = __int_as_float(0x7fc00000);
    const int rlo = max(0, r0 - R), rhi = min(H - 1, r0 + nqr - 1 + R);

    // the counts are kept as buffer offsets (see append4)
#pragma unroll
    for (int q = 0; q < Q; ++q) cnt[q] = pend_code<NSLOT>(cnt[q]);
    const uint32_t slot0 = ((uint32_t)(uintptr_t)&S.pend[0][0][0] - (uint32_t)pend_code<NSLOT>(0)) / 4;
    const bool stats = f.stats != nullptr;
    bool given_up = false;

    // ---- live rows
    int lo = 0x7fffffff, hi = -1;
    {
        uint32_t thr[QR];  // loosest bound of each query row
#pragma unroll
        for (int qr = 0; qr < QR; ++qr) {
            thr[qr] = th[qr * QC];
#pragma unroll
            for (int qc = 1; qc < QC; ++qc) thr[qr] = max(thr[qr], th[qr * QC + qc]);
        }
        for (int base = rlo; base <= rhi; base += WAVE) {
            const int i = base + L;
            const float fi = feat(lam, i);
            bool live = false;
#pragma unroll
            for (int qr = 0; qr < QR; ++qr) {
                const int r = r0 + qr;
                const float a = feat(lam, r) - fi;
                live |= qr < nqr && i <= rhi && i >= r - R && i <= r + R &&
                        __float_as_uint(a * a) <= thr[qr];
            }
            const uint64_t m = ballot(live);
            if (m) {
                lo = min(lo, base + (int)__builtin_ctzll(m));
                hi = max(hi, base + 63 - (int)__builtin_clzll(m));
            }
        }
    }

    const int nrows = hi - lo + 1;
    if (nrows <= 0) return false;
    const int nblk = (nrows + (2 << lpr) - 1) >> (lpr + 1);
    int PR = nrows;
    if (nblk > 1) PR = (nrows + nblk - 1) / nblk;
    // x / PR by a reciprocal: (x + 0.5) / PR is at least 1/128 from an integer
    const float rp = __builtin_amdgcn_rcpf((float)PR);
    const int lc = (int)(((float)L + 0.5f) * rp), lr = L - lc * PR;
    const int SW = uni((int)((WAVE + 0.5f) * rp));
    for (int blk = lo; blk <= hi; blk += PR) {
        const int bhi = min(blk + PR - 1, hi);
        const int i = blk + lr;
        float a2[QR];   // this lane's row term per query row (NaN outside the block's rows
                        // or the query row's window: no distance is within a bound)
        float a2n[QR];  // smallest row term of the block per query row (uniform)
#pragma unroll
        for (int qr = 0; qr < QR; ++qr) {
            const int r = r0 + qr;
            const float a = feat(lam, r) - feat(lam, i);
            a2[qr] = qr < nqr && lc < SW && i <= bhi && i >= r - R && i <= r + R ? a * a : qnan;
            const int wl = max(blk, r - R), wh = min(bhi, r + R);
            const float an = feat(lam, r) - feat(lam, min(max(r, wl), wh));
            a2n[qr] = (qr < nqr && wl <= wh) ? an * an : pinf;
        }
        // live columns right and left of the tile's own: a prefix each, found P at
        // a time, one (query, column) pair per lane
        constexpr int P = WAVE / Q;
        const int sq = L / P, lp = L % P;
        const uint32_t thl = S.tauhi[sq];
        const float fcl = feat(lam, c0 + sq % QC);
        float a2l = a2n[0];
#pragma unroll
        for (int qr = 1; qr < QR; ++qr) a2l = sq / QC == qr ? a2n[qr] : a2l;
        int nside[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            int n = 0;
            for (;;) {
                const int jn = side == 0 ? c0 + nqc + n + lp : c0 - 1 - n - lp;
                const float b = fcl - feat(lam, jn);
                uint64_t m = ballot(__float_as_uint(fmaf(b, b, a2l)) <= thl) &
                             ballot(side == 0 ? jn < W : jn >= 0);
#pragma unroll
                for (int d = WAVE / 2; d >= P; d /= 2) m |= m >> d;  // any query's, in bits 0 .. P-1
                const int k = (int)__builtin_ctzll(~m | (1ull << P));
                n += k;
                if (k < P) break;
            }
            nside[side] = n;
        }
        const int cl = c0 - nside[1];
        int cr = c0 + nqc - 1 + nside[0];

        // rows past the frame or the window and columns past the frame are loaded clamped
        const float* __restrict__ rowp = pc1 + (size_t)min(i, rhi) * W;
        float ipn = rowp[(uint32_t)min(cl + lc, W - 1)];
        for (int jc = cl; jc <= cr; jc += SW) {
            const int j = jc + lc;
            const bool jok = j < W;
            const float ip = jok ? ipn : qnan;
            if (jc + SW <= cr) ipn = rowp[(uint32_t)min(j + SW, W - 1)];
            const uint32_t idx = (uint32_t)i * (uint32_t)W + (uint32_t)j;
            float b[QC];
#pragma unroll
            for (int qc = 0; qc < QC; ++qc) b[qc] = feat(lam, c0 + qc) - feat(lam, j);
            if (stats) {
#pragma unroll
                for (int qr = 0; qr < QR; ++qr)
                    pairs += (unsigned long long)__builtin_popcountll(ballot(jok && a2[qr] == a2[qr])) * nqc;
            }
            float d[Q];
            uint64_t m[Q];
            int cn[Q];
            int full = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int qr = q / QC, qc = q % QC;
                const float e = iq[q] - ip;
                d[q] = fmaf(e, e, fmaf(b[qc], b[qc], a2[qr]));
                m[q] = ballot(__float_as_uint(d[q]) <= th[q]);
                cn[q] = cnt[q] + 4 * __builtin_popcountll(m[q]);
                full |= cn[q];
            }
            uint32_t ovf = 0;  // queries whose buffer cannot take this step's survivors
            if (__builtin_expect((full & FULL) != 0, 0)) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (cn[q] & FULL) {
                        ovf |= 1u << q;
                        m[q] = 0;
                        cn[q] = cnt[q];
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < Q; q += 4) append4<NSLOT>(q, m + q, d + q, cnt + q, idx, slot0);
#pragma unroll
            for (int q = 0; q < Q; ++q) cnt[q] = cn[q];
            if (__builtin_expect(ovf != 0, 0)) {
                // rare: cut the full buffers down (which tightens the bounds) and
                // append this step's survivors
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (L == 0) S.cnt[q] = pend_count<NSLOT>(cnt[q]);
                wave_sync();
                while (ovf) {
                    const int q = __builtin_ctz(ovf);
                    ovf &= ovf - 1;
                    const int qr = q / QC, qc = q % QC;
                    const int r = r0 + qr;
                    const float a = feat(lam, r) - feat(lam, i);
                    const float bq = feat(lam, c0 + qc) - feat(lam, j);
                    const float e = S.iq[q] - ip;
                    const float d = fmaf(e, e, fmaf(bq, bq, a * a));
                    const bool rq = lc < SW && i <= bhi && i >= r - R && i <= r + R;
                    const int nb = uni(S.cnt[q]);
                    const uint32_t thq = uniu(S.tauhi[q]);
                    const uint32_t own = (uint32_t)r * (uint32_t)W + (uint32_t)(c0 + qc);
                    tighten(S, q, nb, jok && rq ? __float_as_uint(d) : ~0u, idx, thq, f.K, own, NSLOT,
                            cut_target<NSLOT>(f.K));
                    --cuts;
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    cnt[q] = pend_code<NSLOT>(uni(S.cnt[q]));
                    th[q] = S.tauhi[q];
                }
                if (cuts <= 0 && cr - jc > CROWDED_STEPS * SW) {
                    cr = hi = -1;  // ends both loops
                    given_up = true;
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) cnt[q] = pend_count<NSLOT>(cnt[q]);
    return given_up;
}

// The whole window: rows x 64-column chunks, nearest chunk first, four rows per group.
// Given up after `cuts` cuts of full buffers, as scan_pruned is.
template <int QR, int QC, int NSLOT>
__device__ __forceinline__ bool scan_all(TileLds<QR, QC, false, NSLOT>& S, const FrameDesc& f, int r0, int c0,
                                         int nqr, int nqc, int L, const float (&iq)[QR * QC],
                                         uint32_t (&th)[QR * QC], int (&cnt)[QR * QC],
                                         unsigned long long& pairs, int cuts) {
    constexpr int Q = QR * QC;
    const int H = f.H, W = f.W, R = f.R, K = f.K;
    const float lam = f.lambda;
    const float* __restrict__ pc1 = f.pc1;
    const float pinf = __int_as_float(0x7f800000), qnan = __int_as_float(0x7fc00000);
    const int rlo = max(0, r0 - R);
    const int rhi = min(H - 1, r0 + nqr - 1 + R);
    int nch = (W + WAVE - 1) / WAVE;
    const int cc = (c0 + (nqc - 1) / 2) / WAVE;
    int tab_base = -1;       // first row of the a2 table contents

    for (int t = 0; t < 2 * nch; ++t) {
        const int m = (t & 1) ? cc + (t + 1) / 2 : cc - t / 2;
        if (m < 0 || m >= nch) continue;
        const int J = m * WAVE;
        const int j = J + L;
        const bool valid = j < W;
        const uint64_t vm = ballot(valid);
        const int jl = valid ? j : W - 1;
        // lanes past the right edge get b = NaN, so no distance there is
        // within a bound
        float b[QC];
#pragma unroll
        for (int qc = 0; qc < QC; ++qc) b[qc] = valid ? feat(lam, c0 + qc) - feat(lam, j) : qnan;

        const int lo = rlo;
        int hi = rhi;

        // Table blocks are aligned to rlo: block k holds rows rlo + 64k ...
        // rlo + 64k + 63 (NaN past rhi and in the padding), so windows of up
        // to 64 rows fill it once per tile.
        for (int blk = rlo + ((lo - rlo) / A2ROWS) * A2ROWS; blk <= hi; blk += A2ROWS) {
            if (blk != tab_base) {
                wave_sync();
                for (int u = L; u < (A2ROWS + A2PAD) * QR; u += WAVE) {
                    const int rr = u / QR, qr = u % QR;
                    const int r = r0 + qr, i = blk + rr;
                    const bool act = rr < A2ROWS && qr < nqr && i <= rhi && i >= r - R && i <= r + R;
                    const float a = feat(lam, r) - feat(lam, i);
                    S.a2t[rr][qr] = act ? a * a : qnan;
                }
                wave_sync();
                tab_base = blk;
            }
            const int g0 = max(lo, blk) - blk;
            int g1 = min(hi, blk + A2ROWS - 1) - blk;  // last table row used
            const uint32_t joff = (uint32_t)jl;
            const float* __restrict__ rowp = pc1 + (size_t)(blk + g0) * W;
            float ipn[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                ipn[u] = rowp[(size_t)min(u, g1 - g0) * W + joff];
            for (int g = g0; g <= g1; g += 4) {
                float ip[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) ip[u] = ipn[u];
                if (g + 4 <= g1) {
                    const float* __restrict__ np = pc1 + (size_t)(blk + g + 4) * W;
#pragma unroll
                    for (int u = 0; u < 4; ++u) ipn[u] = np[(size_t)min(u, g1 - g - 4) * W + joff];
                }
                float a2[4][QR];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int qr = 0; qr < QR; ++qr) a2[u][qr] = S.a2t[g + u][qr];
                const int i0 = blk + g;
                if (f.stats) {
                    const int nvl = min(WAVE, W - J);
#pragma unroll
                    for (int qr = 0; qr < QR; ++qr) {
                        const int r = r0 + qr;
                        const int a = max(i0, max(lo, r - R)), z = min(i0 + 3, min(hi, r + R));
                        if (qr < nqr && z >= a) pairs += (unsigned long long)(z - a + 1) * nqc * nvl;
                    }
                }
                uint32_t ovf = 0;  // queries whose buffer cannot take this group's survivors
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int qr = q / QC, qc = q % QC;
                    float d[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float e = iq[q] - ip[u];
                        const float tt = fmaf(b[qc], b[qc], a2[u][qr]);
                        d[u] = fmaf(e, e, tt);
                    }
                    const uint32_t mn = min(min(__float_as_uint(d[0]), __float_as_uint(d[1])),
                                            min(__float_as_uint(d[2]), __float_as_uint(d[3])));
                    if (ballot(mn <= th[q])) {
                        // rare: some candidate of the group is within the
                        // bound; append the group's survivors if they fit
                        uint64_t mu[4];
                        int n = 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            mu[u] = ballot(__float_as_uint(d[u]) <= th[q]);
                            n += __builtin_popcountll(mu[u]);
                        }
                        if (cnt[q] + n <= NSLOT) {
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                if (__float_as_uint(d[u]) <= th[q]) {
                                    const int slot = cnt[q] + mbcnt(mu[u]);
                                    S.pend[q][0][slot] = __float_as_uint(d[u]);
                                    S.pend[q][1][slot] = (uint32_t)((i0 + u) * W + j);
                                }
                                cnt[q] += __builtin_popcountll(mu[u]);
                            }
                        } else {
                            ovf |= 1u << q;
                        }
                    }
                }
                if (ovf) {
                    // rare: cut the full buffers down (which tightens the
                    // bounds), appending the group row by row
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if (L == 0) S.cnt[q] = cnt[q];
                    wave_sync();
                    while (ovf) {
                        const int q = __builtin_ctz(ovf);
                        ovf &= ovf - 1;
                        const int qr = q / QC, qc = q % QC;
                        const int r = r0 + qr;
                        int cq = uni(S.cnt[q]);
                        uint32_t thq = uniu(S.tauhi[q]);
                        const float bq = valid ? feat(lam, c0 + qc) - feat(lam, j) : pinf;
                        const float iqq = S.iq[q];
                        for (int u = 0; u < 4; ++u) {
                            const int i = i0 + u;
                            if (qr >= nqr || i > hi || i < r - R || i > r + R) continue;
                            const float a2q = S.a2t[g + u][qr];
                            const float e = iqq - ip[u];
                            const float du = fmaf(e, e, fmaf(bq, bq, a2q));
                            uint64_t msk = ballot(__float_as_uint(du) <= thq) & vm;
                            if (!msk) continue;
                            if (cq + __builtin_popcountll(msk) > NSLOT) {
                                const uint32_t own = (uint32_t)r * (uint32_t)W + (uint32_t)(c0 + qc);
                                tighten(S, q, cq, valid ? __float_as_uint(du) : ~0u,
                                        (uint32_t)(i * W + j), thq, K, own, NSLOT,
                                        cut_target<NSLOT>(K));
                                --cuts;
                                cq = uni(S.cnt[q]);
                                thq = uniu(S.tauhi[q]);
                                continue;
                            }
                            if (valid && __float_as_uint(du) <= thq) {
                                S.pend[q][0][cq + mbcnt(msk)] = __float_as_uint(du);
                                S.pend[q][1][cq + mbcnt(msk)] = (uint32_t)(i * W + j);
                            }
                            cq += __builtin_popcountll(msk);
                        }
                        wave_sync();
                        if (L == 0) {
                            S.cnt[q] = cq;
                            S.tauhi[q] = thq;
                        }
                        wave_sync();
                    }
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        cnt[q] = uni(S.cnt[q]);
                        th[q] = S.tauhi[q];
                    }
                    if (cuts <= 0) nch = hi = g1 = -1;  // ends all loops
                }
            }
        }
    }
    return cuts <= 0;
}

// s + v[0] + v[1] + ... + v[N-1], left to right, where v[u] is the float at
// pb + lst[u] * rowb: all N gathers are issued before the first add.  lst is
// 16-byte aligned and N a multiple of 4.
template <int N>
__device__ __forceinline__ float gather_add(float s, const char* __restrict__ pb,
                                            const uint32_t* lst, uint32_t rowb) {
    float v[N];
#pragma unroll
    for (int u = 0; u < N; u += 4) {
        const uint4 id = *(const uint4*)(lst + u);
        v[u + 0] = *(const float*)(pb + (uint64_t)id.x * rowb);
        v[u + 1] = *(const float*)(pb + (uint64_t)id.y * rowb);
        v[u + 2] = *(const float*)(pb + (uint64_t)id.z * rowb);
        v[u + 3] = *(const float*)(pb + (uint64_t)id.w * rowb);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) s = s + v[u];
    return s;
}

// As gather_add, with 32-bit byte offsets from a wave-uniform base: v[u] is
// the float at base + lst[u] * rowb + cb, for frames whose linear indices fit
// 24 bits and whose probability array fits 2^32 bytes (one full-rate 24-bit
// multiply-add per gather instead of a 64-bit one).
template <int N>
__device__ __forceinline__ float gather_add24(float s, const char* __restrict__ base,
                                              const uint32_t* lst, uint32_t rowb, uint32_t cb) {
    float v[N];
#pragma unroll
    for (int u = 0; u < N; u += 4) {
        const uint4 id = *(const uint4*)(lst + u);
        v[u + 0] = *(const float*)(base + (__umul24(id.x, rowb) + cb));
        v[u + 1] = *(const float*)(base + (__umul24(id.y, rowb) + cb));
        v[u + 2] = *(const float*)(base + (__umul24(id.z, rowb) + cb));
        v[u + 3] = *(const float*)(base + (__umul24(id.w, rowb) + cb));
    }
#pragma unroll
    for (int u = 0; u < N; ++u) s = s + v[u];
    return s;
}

// Pass A.  Any set of block candidates of which at least K have a distance <= d
// bounds the query's final K-th key from above by (d, max index).  The block's
// NA candidates (128 or 64) are split into two groups of the same spatial
// spread; with m = ceil(K / 2), the larger of the groups' m-th smallest
// distances is such a d.  All Q blocks are evaluated and sorted together:
// segment q of the wavefront (P lanes) holds query q's block, the groups as the
// low and high halves of NR registers of 16-bit keys rounded down.
template <int QR, int QC, int NA>
__device__ __forceinline__ void tile_bound(TileState<QR, QC>& S, const FrameDesc& f, int r0, int c0,
                                           int nqr, int nqc, int L) {
    constexpr int Q = QR * QC, P = WAVE / Q, EA = NA / P, NR = EA / 2;
    constexpr int LNA = NA == 128 ? 7 : 6;
    static_assert((NA == 128 && Q == 8) || NA == 64, "pass-A block size");
    const int H = f.H, W = f.W, R = f.R, K = f.K;
    const float lam = f.lambda;
    const float* __restrict__ pc1 = f.pc1;
    const int sq = L / P, lp = L % P;  // this lane's query (segment) and slot in it
    const int sqr = sq / QC, sqc = sq % QC;
    const bool sok = sqr < nqr && sqc < nqc;
    const bool off32 = (uint64_t)H * (uint64_t)W <= (1u << 30);  // band byte offsets fit 32 bits
    const int r = r0 + sqr, c = c0 + sqc;
    const int i0w = max(0, r - R), i1w = min(H - 1, r + R);
    const int nr = i1w - i0w + 1;
    const int lbr = nr >= 8 ? 3 : (nr >= 4 ? 2 : (nr >= 2 ? 1 : 0));
    const int br = 1 << lbr;
    const int lbc = LNA - lbr;
    const int bc = 1 << lbc;
    const int rb = min(max(r - br / 2, i0w), i1w - br + 1);
    const int cb = max(0, min(c - bc / 2, W - bc));
    // I of the segment's query pixel (NaN for pixels off the frame)
    const float iqs = sok ? pc1[(uint32_t)r * (uint32_t)W + (uint32_t)c] : __int_as_float(0x7fc00000);
    const float frq = feat(lam, r), fcq = feat(lam, c);
    // Every lane loads (columns past the right edge clamped and given +inf;
    // rows rb .. rb+br-1 are inside the frame even for queries off its bottom
    // edge), so all EA loads are in flight together.
    uint32_t xp[NR];
    if (W >= NA / 8 && off32 && !ballot(lbr != 3)) {
        // every block is 8 rows x NA / 8 columns
        const char* __restrict__ pcb = (const char*)pc1;
        float pv[EA];
        if constexpr (NA == 128) {
            // lane lp takes columns cb + 2 lp (group 0) and cb + 2 lp + 1 (group
            // 1): both groups hold every row and alternate columns
            const int j = cb + 2 * lp;
            const uint32_t o4 = ((uint32_t)rb * (uint32_t)W + (uint32_t)j) * 4u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const char* row = pcb + (o4 + (uint32_t)u * (uint32_t)W * 4u);
                pv[2 * u] = *(const float*)row;
                pv[2 * u + 1] = *(const float*)(row + 4);
            }
            const float b0 = fcq - feat(lam, j), b1 = fcq - feat(lam, j + 1);
            // one query row: the eight row terms are the same in every segment,
            // lane u computes row u's
            const float al = frq - feat(lam, rb + lp);
            const float a2l = al * al;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float a2;
                if constexpr (QR == 1) {
                    a2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a2l), u));
                } else {
                    const float a = frq - feat(lam, rb + u);
                    a2 = a * a;
                }
                const float e0 = iqs - pv[2 * u], e1 = iqs - pv[2 * u + 1];
                // NaN bits for a query off the frame (segment unused)
                xp[u] = pack_hi(__float_as_uint(fmaf(e0, e0, fmaf(b0, b0, a2))),
                                __float_as_uint(fmaf(e1, e1, fmaf(b1, b1, a2))));
            }
        } else {
            // lane lp takes columns cb + lp (+ P for four lanes a segment), even
            // rows for group 0 and odd rows for group 1
            const int j = cb + lp;
            const uint32_t o4 = ((uint32_t)rb * (uint32_t)W + (uint32_t)j) * 4u;
#pragma unroll
            for (int h = 0; h < 8 / P; ++h)
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    pv[8 * h + u] = *(const float*)(pcb + (o4 + (uint32_t)u * (uint32_t)W * 4u) + 4 * P * h);
#pragma unroll
            for (int h = 0; h < 8 / P; ++h) {
                const float b = fcq - feat(lam, j + P * h);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float a0 = frq - feat(lam, rb + 2 * u), a1 = frq - feat(lam, rb + 2 * u + 1);
                    const float e0 = iqs - pv[8 * h + 2 * u], e1 = iqs - pv[8 * h + 2 * u + 1];
                    xp[4 * h + u] = pack_hi(__float_as_uint(fmaf(e0, e0, fmaf(b, b, a0 * a0))),
                                            __float_as_uint(fmaf(e1, e1, fmaf(b, b, a1 * a1))));
                }
            }
        }
    } else {
        // element e = u * P + lp of the block is row rb + (e >> lbc), column cb +
        // (e & (bc - 1)); group 0 the elements u < NR, group 1 the rest
        float pv[EA];
#pragma unroll
        for (int u = 0; u < EA; ++u) {
            const int e = u * P + lp;
            const int i = rb + (e >> lbc);
            const int j = min(cb + (e & (bc - 1)), W - 1);
            pv[u] = pc1[(uint32_t)i * (uint32_t)W + (uint32_t)j];
        }
        uint32_t x[EA];
#pragma unroll
        for (int u = 0; u < EA; ++u) {
            const int e = u * P + lp;
            const int i = rb + (e >> lbc);
            const int j = cb + (e & (bc - 1));
            const float a = frq - feat(lam, i);
            const float b = fcq - feat(lam, j);
            const float ee = iqs - pv[u];
            const uint32_t d = __float_as_uint(fmaf(ee, ee, fmaf(b, b, a * a)));
            x[u] = (sok && j < W) ? d : 0x7f800000u;  // +inf: no candidate
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) xp[u] = pack_hi(x[u], x[u + NR]);
    }
    if (lp == 0) S.iq[sq] = iqs;
    // prefill the query's buffer slots (see PAD)
    {
        const uint32_t own = (uint32_t)r * (uint32_t)W + (uint32_t)c;
        if constexpr (P >= 4) {
#pragma unroll
            for (int u = 0; u < WAVE / 4 / P; ++u) {
                const uint32_t d = PAD + 256u * (uint32_t)(lp + u * P);
                ((uint4*)S.pend[sq][0])[lp + u * P] = make_uint4(d, d + 64u, d + 128u, d + 192u);
                ((uint4*)S.pend[sq][1])[lp + u * P] = make_uint4(own, own, own, own);
            }
        }
    }
    // each group's element m - 1 (lane (m-1) / NR, register (m-1) % NR); at
    // least K candidates lie at or below the larger key
    const int m = (K + 1) / 2;
    const uint32_t v = pk_seg_rank<P>(xp, lp, uni((m - 1) % NR));
    const uint32_t kk = max(v & 0xffffu, v >> 16) + 1u;
    // (not above +inf: the scans give candidates outside the window NaN distances)
    if (lp == (m - 1) / NR) S.tauhi[sq] = sok ? min(kk << 16, 0x7f800000u) : 0u;
}

// Final selection and Eq. 2 of a tile; E: buffer slots per lane (all of them,
// or the first half where no buffer holds more).
template <int QR, int QC, int E, int NSLOT>
__device__ __forceinline__ void finish_tile(TileState<QR, QC, NSLOT>& S, const FrameDesc& f, int r0, int c0,
                                            int nqr, int nqc, int L) {
    constexpr int Q = QR * QC, P = WAVE / Q;
    const int H = f.H, W = f.W, K = f.K, C = f.C;
    const int sq = L / P, lp = L % P;
    const int sqr = sq / QC, sqc = sq % QC;
    const bool sok = sqr < nqr && sqc < nqc;
    const bool merged = S.tauhi[sq] > BIG;  // ordered by order_query, neighbours written
    const uint32_t pix = (uint32_t)(r0 + sqr) * (uint32_t)W + (uint32_t)(c0 + sqc);

    // One segmented sort of the candidate buffers.  The network sorts 32-bit
    // packed keys: the distance bits with their 6 low bits replaced by the
    // buffer slot.  Packed order is exact wherever the distance parts differ;
    // runs of equal distance parts are then put in (d, idx) order on the full
    // keys by odd-even transposition (rarely needed).
    uint32_t x[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        // slot blocks permuted by segment (u ^ sq: E is a power of two), so the
        // segments' reads of one u spread over the banks
        const int e = (u ^ (sq & (E - 1))) * P + lp;
        const uint32_t dh = S.pend[sq][0][e];
        x[u] = (dh & ~63u) | (uint32_t)e;
    }
    seg_sort<P>(x, lp);
    // two neighbours in sorted order share the distance part iff their keys
    // differ in the slot bits only: (a ^ b) <= 63 (keys are distinct)
    bool tie = false;
#pragma unroll
    for (int u = 0; u + 1 < E; ++u) tie |= (x[u] ^ x[u + 1]) < 64u;
    {
        uint32_t nx;  // the next lane's first
        asm("s_nop 1\n\tv_mov_b32_dpp %0, %1 row_shl:1 row_mask:0xf bank_mask:0xf" : "=v"(nx) : "v"(x[0]));
        tie |= lp < P - 1 && (x[E - 1] ^ nx) < 64u;
    }
    const bool ties = ballot(tie) != 0;
    uint32_t id[E];
    if (ties || f.out_nbr || f.out_dist) {
        uint64_t y[E];
#pragma unroll
        for (int u = 0; u < E; ++u)
            y[u] = make_key(__uint_as_float(S.pend[sq][0][x[u] & 63u]), (int)S.pend[sq][1][x[u] & 63u]);
        if (ties) {
            for (;;) {
                bool sw = false;
#pragma unroll
                for (int ph = 0; ph < 2; ++ph) {
#pragma unroll
                    for (int u = ph; u + 1 < E; u += 2) {
                        const uint64_t a = y[u], b = y[u + 1];
                        const bool t = b < a;
                        y[u] = t ? b : a;
                        y[u + 1] = t ? a : b;
                        sw |= t;
                    }
                    if (ph == 1) {
                        // pair (lane's last, next lane's first)
                        const uint64_t nx = (uint64_t)(uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)y[0], 0x101, 0xF, 0xF, false) |
                                            ((uint64_t)(uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(y[0] >> 32), 0x101, 0xF, 0xF, false) << 32);
                        const uint64_t pv = (uint64_t)(uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)y[E - 1], 0x111, 0xF, 0xF, false) |
                                            ((uint64_t)(uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(y[E - 1] >> 32), 0x111, 0xF, 0xF, false) << 32);
                        const bool tn = lp < P - 1 && nx < y[E - 1];  // this lane keeps the smaller
                        const bool tp = lp > 0 && y[0] < pv;          // this lane keeps the larger
                        y[E - 1] = tn ? nx : y[E - 1];
                        y[0] = tp ? pv : y[0];
                        sw |= tn;
                    }
                }
                if (!ballot(sw)) break;
            }
        }
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int e = lp * E + u;
            if (sok && !merged && e < K) {
                if (f.out_nbr) f.out_nbr[(size_t)pix * K + e] = (int32_t)(uint32_t)y[u];
                if (f.out_dist) f.out_dist[(size_t)pix * K + e] = __uint_as_float((uint32_t)(y[u] >> 32));
            }
            id[u] = (uint32_t)y[u];
        }
    } else {
#pragma unroll
        for (int u = 0; u < E; ++u) id[u] = S.pend[sq][1][x[u] & 63u];
    }

    // ---- Eq. 2: sums in neighbour order, one lane per (query, class)
    const uint32_t rowb = (uint32_t)C * 4u;  // bytes per probability row
    const uint64_t npix = (uint64_t)H * (uint64_t)W;
    const bool off24 = npix <= (1u << 24) && npix * rowb <= 0xFFFFFFFFull;
    if (C == 4 && off24 && ((uintptr_t)f.prob & 15) == 0) {
        // Four classes: every lane gathers its own ranks' rows (16 bytes, all in
        // flight together); the rows go through LDS, ROWS neighbours at a time,
        // to the lanes that sum them.  One load of a row serves four classes:
        // 8 loads and 8 shifts per lane where a gather per class took 40 of
        // each, in three trips to L2 instead of one.
        typedef float f4 __attribute__((ext_vector_type(4)));
        f4 row[E];
        if (sok && lp * E < K) {
#pragma unroll
            for (int u = 0; u < E; ++u) row[u] = *(const f4*)((const char*)f.prob + (id[u] << 4));
        }
        const int q = L >> 2, cl = L & 3;
        const float* col = (const float*)S.rows[q < Q ? q : 0] + cl;
        float s = 0.0f;
        auto put_rows = [&](int h) __attribute__((always_inline)) {
            wave_sync();  // the buffers, or the rows before, have been read
            if (sok && lp * E / ROWS == h && lp * E < K) {
#pragma unroll
                for (int u = 0; u < E; ++u) *(f4*)&S.rows[sq][row_at<E>(lp * E % ROWS + u)] = row[u];
            }
            wave_sync();
        };
        auto add_rows = [&](int n) __attribute__((always_inline)) {
            int k = 0;
            for (; k + 8 <= n; k += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = col[4 * (row_at<E>(k) + u)];
#pragma unroll
                for (int u = 0; u < 8; ++u) s = s + v[u];
            }
            for (; k < n; ++k) s = s + col[4 * row_at<E>(k)];
        };
        put_rows(0);
        add_rows(min(ROWS, K));
        if constexpr (P * E > ROWS) {
            if (K > ROWS) {
                put_rows(1);
                add_rows(K - ROWS);
            }
        }
        const int qr = q / QC, qc = q % QC;
        // class map: the lanes of a quad hold the query's four sums
        const float s0 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0x00, 0xF, 0xF, false));
        const float s1 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0x55, 0xF, 0xF, false));
        const float s2 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0xAA, 0xF, 0xF, false));
        const float s3 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0xFF, 0xF, 0xF, false));
        int best = 0;
        float bs = s0;
        if (s1 > bs) { bs = s1; best = 1; }
        if (s2 > bs) { bs = s2; best = 2; }
        if (s3 > bs) { bs = s3; best = 3; }
        if (q < Q && qr < nqr && qc < nqc) {
            const uint32_t px = (uint32_t)(r0 * W + c0) + __umul24((uint32_t)qr, (uint32_t)W) + (uint32_t)qc;
            *(float*)((char*)f.out_prob + ((px << 4) + (uint32_t)cl * 4u)) = s / (float)K;
            if (cl == 0) f.out_class[px] = best;
        }
        return;
    }
    // other class counts: the lists go through LDS, 16 bytes at a time (entries
    // from K on are never read)
    wave_sync();  // the buffers have been read
    if (sok && lp * E < K) {
#pragma unroll
        for (int u = 0; u < E; u += 4)
            *(uint4*)&S.list[sq][lp * E + u] = make_uint4(id[u], id[u + 1], id[u + 2], id[u + 3]);
    }
    wave_sync();
    // p / C by a reciprocal: (p + 0.5) / C sits at least 1/(2C) >= 1/32 from
    // an integer and p < 2^10, far beyond the reciprocal's rounding
    const float rc = __builtin_amdgcn_rcpf((float)C);
    for (int p = L; p < Q * C; p += WAVE) {
        const int q = (int)(uint32_t)(((float)p + 0.5f) * rc), cl = p - q * C;
        const int qr = (int)((uint32_t)q / QC), qc = (int)((uint32_t)q % QC);
        if (qr >= nqr || qc >= nqc) continue;
        const uint32_t* lst = S.list[q];
        float s = 0.0f;
        int k = 0;
        if (off24) {
            const char* __restrict__ base = (const char*)f.prob;
            const uint32_t cb = (uint32_t)cl * 4u;
            for (; k + 16 <= K; k += 16) s = gather_add24<16>(s, base, lst + k, rowb, cb);
            if (k + 8 <= K) {
                s = gather_add24<8>(s, base, lst + k, rowb, cb);
                k += 8;
            }
            for (; k < K; ++k) s = s + *(const float*)(base + (__umul24(lst[k], rowb) + cb));
        } else {
            const char* __restrict__ pb = (const char*)(f.prob + cl);
            for (; k + 16 <= K; k += 16) s = gather_add<16>(s, pb, lst + k, rowb);
            if (k + 8 <= K) {
                s = gather_add<8>(s, pb, lst + k, rowb);
                k += 8;
            }
            for (; k < K; ++k) s = s + *(const float*)(pb + (uint64_t)lst[k] * rowb);
        }
        S.sums[q][cl] = s;
        if (off24) {
            // the pixel's byte offset in the probability map fits 32 bits
            const uint32_t pix = (uint32_t)(r0 * W + c0) + __umul24((uint32_t)qr, (uint32_t)W) + (uint32_t)qc;
            *(float*)((char*)f.out_prob + (__umul24(pix, rowb) + (uint32_t)cl * 4u)) = s / (float)K;
        } else {
            const size_t pix = (size_t)(r0 + qr) * W + c0 + qc;
            f.out_prob[pix * C + cl] = s / (float)K;
        }
    }
    wave_sync();
    if (L < Q) {
        const int qr = L / QC, qc = L % QC;
        if (qr < nqr && qc < nqc) {
            int best = 0;
            float bs = S.sums[L][0];
            for (int cl = 1; cl < C; ++cl) {
                const float v = S.sums[L][cl];
                if (v > bs) { bs = v; best = cl; }
            }
            if (off24)
                f.out_class[(uint32_t)(r0 * W + c0) + __umul24((uint32_t)qr, (uint32_t)W) + (uint32_t)qc] = best;
            else
                f.out_class[(size_t)(r0 + qr) * W + c0 + qc] = best;
        }
    }
}

// Order the queries whose bound lies beyond the packed keys' range (rare), then select,
// average and write.  The buffers hold at most 64 candidates each.
template <int QR, int QC, int NSLOT>
__device__ __forceinline__ void select_tile(TileState<QR, QC, NSLOT>& S, const FrameDesc& f, int r0, int c0,
                                            int nqr, int nqc, int L, const int (&cnt)[QR * QC]) {
    constexpr int Q = QR * QC, E = Q;
    int most = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) most = max(most, uni(cnt[q]));
    wave_sync();
    {
        const bool one = L < Q && L / QC < nqr && L % QC < nqc;
        uint64_t need = ballot(one && S.tauhi[L % Q] > BIG);
        if (__builtin_expect(need != 0, 0)) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (L == 0) S.cnt[q] = cnt[q];
            wave_sync();
            while (need) {
                const int q = (int)__builtin_ctzll(need);
                need &= need - 1;
                order_query(S, f, r0, c0, q, uni(S.cnt[q]));
            }
        }
    }
    if constexpr (E >= 8) {
        if (most <= WAVE / 2 && f.K <= WAVE / 2) {
            finish_tile<QR, QC, E / 2>(S, f, r0, c0, nqr, nqc, L);
            return;
        }
    }
    finish_tile<QR, QC, E>(S, f, r0, c0, nqr, nqc, L);
}

// v, as a value that is not known before this point.
__device__ __forceinline__ uint32_t here(uint32_t v) {
    asm volatile("" : "+s"(v));
    return v;
}
// The same pointer, known to point to global memory.
template <class T>
__device__ __forceinline__ T* in_global(T* p) {
    typedef __attribute__((address_space(1))) T Global;
    return (T*)(Global*)(uintptr_t)p;
}

// A tile whose buffers overflow again and again, because a bound from 64 or 128 of its
// block's candidates lets far more than 64 through (small lambda, unstructured bands, K
// close to 64), is done over in parts of four queries, whose buffers have 128 slots in
// the same LDS, from the bounds that its scan has reached; and a tile of the pruned search
// whose bounds leave about half of the window (FrameDesc::wide) is done in this way from
// the start, by the whole-window scan.  380 x 480, with and without: lambda 0.0001, K = 40
// 670 and 1,380 us; lambda 0.001, K = 64 490 and 1,230; uniform noise, K = 56 400 and 700.
// It keeps no registers in the ordinary tiles: the frame is read again from where the
// kernel has it (`frame`), and nothing that it computes can be moved ahead (kept in a
// function of its own, its calls' stack cost every tile 4 %).
template <int QR, int QC, bool PRUNE>
__device__ __forceinline__ unsigned long long crowded_tile(
    uint32_t tile, const FrameDesc* frame, int r0, int c0, int lpr) {
    typedef __attribute__((address_space(3))) char Lds;
    typedef TileLds<1, 4, false, 2 * WAVE> Part;
    typedef TileState<QR, QC> Tile;
    static_assert(sizeof(Part) <= offsetof(Tile, tauhi), "a part fits below the tile's bounds");
    unsigned long long pairs = 0;
    for (int part = 0; part < QR * QC / 4; ++part) {
        // everything anew in each part: what the compiler moves out of the loop, or finds
        // in the ordinary tile's registers, costs registers there
        Tile& S = *(Tile*)(char*)(Lds*)here(tile);
        const uint64_t at = (uint64_t)here((uint32_t)((uint64_t)frame >> 32)) << 32 | here((uint32_t)(uint64_t)frame);
        FrameDesc f = *in_global((const FrameDesc*)at);
        f.pc1 = in_global(f.pc1);
        f.prob = in_global(f.prob);
        f.out_prob = in_global(f.out_prob);
        f.out_class = in_global(f.out_class);
        f.out_nbr = in_global(f.out_nbr);
        f.out_dist = in_global(f.out_dist);
        const int L = lane_id_here();
        const int r = (int)here((uint32_t)(r0 + 4 * part / QC)), c = (int)here((uint32_t)(c0 + 4 * part % QC));
        if (r >= f.H || c >= f.W) continue;
        Part& T = *(Part*)&S;
        const int nq = min(4, f.W - c);
        float iq[4];
        uint32_t th[4];
        int cnt[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            iq[q] = S.iq[4 * part + q];
            th[q] = S.tauhi[4 * part + q];
            cnt[q] = 0;
        }
        if (L < 4) {
            T.iq[L] = S.iq[4 * part + L];
            T.tauhi[L] = S.tauhi[4 * part + L];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                T.pend[q][0][WAVE * v + L] = PAD + 64u * (uint32_t)(WAVE * v + L);
                T.pend[q][1][WAVE * v + L] = (uint32_t)r * (uint32_t)f.W + (uint32_t)(c + q);
            }
        }
        wave_sync();
        if (PRUNE && !ballot(T.tauhi[L & 3] > f.wide))
            scan_pruned(T, f, r, c, 1, nq, lpr, L, iq, th, cnt, pairs, 0x7fffffff);
        else
            scan_all(T, f, r, c, 1, nq, L, iq, th, cnt, pairs, 0x7fffffff);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (L == 0) T.cnt[q] = cnt[q];
        wave_sync();
        for (int q = 0; q < 4; ++q) {
            const int nb = uni(T.cnt[q]);
            if (nb > WAVE)
                tighten(T, q, nb, ~0u, 0u, uniu(T.tauhi[q]), f.K,
                        (uint32_t)r * (uint32_t)f.W + (uint32_t)(c + q), WAVE, WAVE);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) cnt[q] = uni(T.cnt[q]);
        select_tile(T, f, r, c, 1, nq, L, cnt);
        wave_sync();
    }
    return pairs;
}

// Process one tile: query pixels (r0 + qr, c0 + qc), qr < QR, qc < QC.
// frame: f, as the kernel was given it in memory.
// NA: largest pass-A block (128 candidates per query; 64 for 16-query tiles).
template <int QR, int QC, bool PRUNE, int NA = (QR * QC == 8 ? 128 : WAVE)>
__device__ __forceinline__ void process_tile(TileLds<QR, QC, PRUNE>& S, const FrameDesc& f,
                                             const FrameDesc* frame, int r0, int c0, int lpr, int L) {
    constexpr int Q = QR * QC;
    const int H = f.H, W = f.W, R = f.R, K = f.K;
    const float lam = f.lambda;
    const int nqr = min(QR, H - r0), nqc = min(QC, W - c0);
    const float* __restrict__ pc1 = f.pc1;
    const float pinf = __int_as_float(0x7f800000), qnan = __int_as_float(0x7fc00000);

    // block size (see SMALL_K)
    bool big = NA == 128 && (K > SMALL_K || lam == 0.0f);
    if (!big) {
        tile_bound<QR, QC, 64>(S, f, r0, c0, nqr, nqc, L);
        if constexpr (NA == 128) {
            wave_sync();
            const float lim = lam * lam * WIDE2;
            big = ballot(S.tauhi[L % Q] > __float_as_uint(lim)) != 0;
        }
    }
    if constexpr (NA == 128)
        if (big) tile_bound<QR, QC, 128>(S, f, r0, c0, nqr, nqc, L);
    wave_sync();

    // Work counter (only reported when f.stats is set): candidate distances
    // evaluated for on-frame queries; pass A counts its block slots.
    unsigned long long pairs = (unsigned long long)(nqr * nqc) * (big ? 128 : WAVE);

    // Uniform per-query values live in VGPRs (read from LDS) to keep the
    // scalar register file free for loop state.  Queries off the frame have
    // iq = NaN and bound 0, so they never pass the test below.
    float iq[Q];
    uint32_t th[Q];
    int cnt[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        iq[q] = S.iq[q];
        th[q] = S.tauhi[q];
        cnt[q] = 0;
    }

    // ---- pass B
    bool crowded = false;
    if constexpr (PRUNE) {
        crowded = ballot(S.tauhi[L % Q] > f.wide) != 0;
        if (!crowded) crowded = scan_pruned(S, f, r0, c0, nqr, nqc, lpr, L, iq, th, cnt, pairs, crowded_cuts(Q, K));
    } else {
        crowded = scan_all(S, f, r0, c0, nqr, nqc, L, iq, th, cnt, pairs, crowded_cuts_all(Q, K));
        if (crowded) pairs = (unsigned long long)(nqr * nqc) * (big ? 128 : WAVE);  // all is evaluated again
    }

    // ---- final selection, Eq. 2, outputs
    if (__builtin_expect(crowded, 0)) pairs += crowded_tile<QR, QC, PRUNE>(
        (uint32_t)(uintptr_t)&S, frame, r0, c0, lpr);
    else select_tile(S, f, r0, c0, nqr, nqc, L, cnt);
    if (f.stats && L == 0) {
        atomicAdd(&f.stats[0], pairs);
        atomicAdd(&f.stats[1], 1ull);
    }
    wave_sync();
}

// Bijective remap of block ids so that each XCD (blocks are dealt round-robin
// to the 8 XCDs) works on a contiguous range of strips, which share window
// rows in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    const int full = nb & ~7;
    if (b >= full) return b;
    const int per = full >> 3;
    return (b & 7) * per + (b >> 3);
}

// 8-query tiles are held to 72 VGPRs, seven wavefronts per SIMD (those of the
// persistent kernels spill 18 to 35 of them around the claim loop).  The
// kernels of the time it was set, side by side: 380 x 480 K=40 52.3 us, 1000 x 1000
// 210, 1024 frames of 50 x 50 449; six wavefronts 53.6, 218 and 472; eight (64
// registers, some spilled) 54.4, 212 and 447.  Their 4,832
// bytes of LDS would allow eight.
#define KNNF_WAVES_PER_EU(QR, QC) __attribute__((amdgpu_waves_per_eu((QR) * (QC) == 8 ? 7 : 4)))

template <int QR, int QC, int WPB, bool PRUNE>
__global__ void __launch_bounds__(WPB * WAVE) KNNF_WAVES_PER_EU(QR, QC)
filter_frame_kernel(FrameDesc f, int lpr) {
    __shared__ TileLds<QR, QC, PRUNE> lds[WPB];
    const int w = uni((int)(threadIdx.x >> 6));
    const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    // tiles <= H * W < 2^31 (checked on the host): 32-bit index arithmetic
    const uint32_t ntc = (uint32_t)((f.W + QC - 1) / QC);
    const uint32_t ntiles = (uint32_t)((f.H + QR - 1) / QR) * ntc;
    const uint32_t s = (uint32_t)b * WPB + (uint32_t)w;
    if (s >= ntiles) return;
    const uint32_t band = s / ntc;
    const uint32_t tc = s - band * ntc;
    process_tile<QR, QC, PRUNE>(lds[w], f, (const FrameDesc*)__builtin_amdgcn_kernarg_segment_ptr(), (int)band * QR, (int)tc * QC, lpr, lane_id());
}

// Persistent batched kernel: each wavefront claims tile tasks from one global
// counter until all tasks of all work items are taken.  Work item k is a range
// of tiles of frames[k] starting at tile_base[k]; its tasks are the ids
// task_start[k] .. task_start[k+1]-1.  Claims go out in task order, so the
// whole device sweeps neighbouring tiles (which share window rows) at the same
// time.  Every wavefront leaves the loop after one failed claim, so the grid
// always drains.
template <int QR, int QC, int WPB, bool PRUNE>
__global__ void __launch_bounds__(WPB * WAVE) KNNF_WAVES_PER_EU(QR, QC)
filter_batch_kernel(const FrameDesc* __restrict__ frames, const uint32_t* __restrict__ task_start,
                    const uint32_t* __restrict__ tile_base, uint32_t nframes, uint32_t total_tasks,
                    uint32_t claim, uint32_t* counter, int lpr) {
    __shared__ TileLds<QR, QC, PRUNE> lds[WPB];
    const int w = uni((int)(threadIdx.x >> 6));
    const int L = lane_id();
    for (;;) {
        // claim `claim` consecutive tasks: fewer atomics on the counter
        uint32_t t0 = 0;
        if (L == 0) t0 = atomicAdd(counter, claim);
        t0 = uniu(t0);  // lane 0's claim
        if (t0 >= total_tasks) break;
        const uint32_t t1 = min(total_tasks, t0 + claim);
        uint32_t k = 0, next = 0;  // work item of the current task, its end
        for (uint32_t t = t0; t < t1; ++t) {
            if (t >= next || t == t0) {
                // work item k with task_start[k] <= t < task_start[k+1]
                uint32_t lo = 0, hi = nframes;
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (task_start[mid] <= t) lo = mid; else hi = mid;
                }
                k = lo;
                next = task_start[k + 1];
            }
            const FrameDesc f = frames[k];
            const uint32_t s = t - task_start[k] + tile_base[k];
            const uint32_t ntc = (uint32_t)((f.W + QC - 1) / QC);
            const int band = (int)(s / ntc);
            const int tc = (int)(s - (uint32_t)band * ntc);
            // the claim loop's registers leave no room for 128-candidate blocks
            process_tile<QR, QC, PRUNE, WAVE>(lds[w], f, frames + k, band * QR, tc * QC, lpr, lane_id_here());
        }
    }
}

// Non-persistent batched kernel over the same work table: one wavefront per
// task, the hardware dispatcher balances the load, XCD-aware block order.
template <int QR, int QC, int WPB, bool PRUNE>
__global__ void __launch_bounds__(WPB * WAVE) KNNF_WAVES_PER_EU(QR, QC)
filter_items_kernel(const FrameDesc* __restrict__ frames, const uint32_t* __restrict__ task_start,
                    const uint32_t* __restrict__ tile_base, uint32_t nframes,
                    uint32_t total_tasks, int lpr) {
    __shared__ TileLds<QR, QC, PRUNE> lds[WPB];
    const int w = uni((int)(threadIdx.x >> 6));
    const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
    const uint64_t t64 = (uint64_t)b * WPB + w;
    if (t64 >= total_tasks) return;
    const uint32_t t = (uint32_t)t64;
    uint32_t lo = 0, hi = nframes;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (task_start[mid] <= t) lo = mid; else hi = mid;
    }
    const FrameDesc f = frames[lo];
    const uint32_t s = t - task_start[lo] + tile_base[lo];
    const uint32_t ntc = (uint32_t)((f.W + QC - 1) / QC);
    const int band = (int)(s / ntc);
    const int tc = (int)(s - (uint32_t)band * ntc);
    process_tile<QR, QC, PRUNE>(lds[w], f, frames + lo, band * QR, tc * QC, lpr, lane_id());
}

template <int QR, int QC, int WPB, bool PRUNE>
int launch_items_t(const FrameDesc* fr, const uint32_t* ts, const uint32_t* tb, uint32_t n,
                   uint32_t tot, int lpr, hipStream_t st) {
    const uint64_t blocks = ((uint64_t)tot + WPB - 1) / WPB;
    hipLaunchKernelGGL((filter_items_kernel<QR, QC, WPB, PRUNE>), dim3((unsigned)blocks),
                       dim3(WPB * WAVE), 0, st, fr, ts, tb, n, tot, lpr);
    return (int)hipGetLastError();
}

template <int QR, int QC, int WPB, bool PRUNE>
int launch_frame_t(const FrameDesc& f, int lpr, hipStream_t st) {
    const long long tiles = (long long)((f.H + QR - 1) / QR) * ((f.W + QC - 1) / QC);
    const long long blocks = (tiles + WPB - 1) / WPB;
    hipLaunchKernelGGL((filter_frame_kernel<QR, QC, WPB, PRUNE>), dim3((unsigned)blocks),
                       dim3(WPB * WAVE), 0, st, f, lpr);
    return (int)hipGetLastError();
}

template <int QR, int QC, int WPB, bool PRUNE>
int launch_batch_t(const FrameDesc* fr, const uint32_t* ts, const uint32_t* tb, uint32_t n,
                   uint32_t tot, uint32_t* ctr, int grid, int lpr, hipStream_t st) {
    // at least four claims per resident wavefront, at most 8 tasks per claim; but no more
    // than 16,384 claims where 16 tasks each allow that: the counter takes one every 15 to
    // 20 ns (64 frames of 100 x 120, 1 x 16 tiles: 24,000 claims 355 us, 16,000 234)
    const uint64_t waves = (uint64_t)grid * WPB;
    const uint64_t few = std::min<uint64_t>(16, (tot + 16383) / 16384);
    const uint32_t claim = (uint32_t)std::max<uint64_t>({1, std::min<uint64_t>(8, tot / (waves * 4)), few});
    hipLaunchKernelGGL((filter_batch_kernel<QR, QC, WPB, PRUNE>), dim3((unsigned)grid),
                       dim3(WPB * WAVE), 0, st, fr, ts, tb, n, tot, claim, ctr, lpr);
    return (int)hipGetLastError();
}

template <int QR, int QC, int WPB, bool PRUNE>
int occupancy_t() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, filter_batch_kernel<QR, QC, WPB, PRUNE>, WPB * WAVE, 0) != hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

// Supported tile shapes (rows x columns) and workgroup sizes.
#define KNNF_SHAPE(FN, QR, QC, ...)                                                        \
    case (QR) * 10000 + (QC) * 100 + 1:                                                    \
        return pr ? FN<QR, QC, 1, true>(__VA_ARGS__) : FN<QR, QC, 1, false>(__VA_ARGS__);  \
    case (QR) * 10000 + (QC) * 100 + 2:                                                    \
        return pr ? FN<QR, QC, 2, true>(__VA_ARGS__) : FN<QR, QC, 2, false>(__VA_ARGS__);  \
    case (QR) * 10000 + (QC) * 100 + 4:                                                    \
        return pr ? FN<QR, QC, 4, true>(__VA_ARGS__) : FN<QR, QC, 4, false>(__VA_ARGS__);

#define KNNF_DISPATCH(FN, ...)                                                  \
    do {                                                                        \
        const bool pr = cfg.pruned != 0;                                        \
        switch (cfg.rows * 10000 + cfg.cols * 100 + cfg.waves) {                \
            KNNF_SHAPE(FN, 1, 8, __VA_ARGS__)                                   \
            KNNF_SHAPE(FN, 1, 16, __VA_ARGS__)                                  \
            KNNF_SHAPE(FN, 2, 4, __VA_ARGS__)                                   \
            KNNF_SHAPE(FN, 2, 8, __VA_ARGS__)                                   \
            KNNF_SHAPE(FN, 4, 4, __VA_ARGS__)                                   \
        default:                                                                \
            return (int)hipErrorInvalidValue;                                   \
        }                                                                       \
    } while (0)

}  // namespace

int launch_filter_frame(const FrameDesc& f, const LaunchCfg& cfg, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    KNNF_DISPATCH(launch_frame_t, f, cfg.chunk_log2, st);
}

int launch_filter_batch(const FrameDesc* d_frames, const uint32_t* d_task_start,
                        const uint32_t* d_tile_base, uint32_t nframes, uint32_t total_tasks,
                        uint32_t* d_counter, const LaunchCfg& cfg, int grid_blocks, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    KNNF_DISPATCH(launch_batch_t, d_frames, d_task_start, d_tile_base, nframes, total_tasks,
                  d_counter, grid_blocks, cfg.chunk_log2, st);
}

int persistent_blocks_per_cu(const LaunchCfg& cfg) { KNNF_DISPATCH(occupancy_t); }

int launch_filter_items(const FrameDesc* d_frames, const uint32_t* d_task_start,
                        const uint32_t* d_tile_base, uint32_t nframes, uint32_t total_tasks,
                        const LaunchCfg& cfg, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    KNNF_DISPATCH(launch_items_t, d_frames, d_task_start, d_tile_base, nframes, total_tasks,
                  cfg.chunk_log2, st);
}

// ---- Input check (validation before a launch): *flag = gen when any pc1 or
// prob value of the frames is NaN or infinite (exponent bits all ones).
__device__ __forceinline__ bool nonfinite(uint32_t u) { return (u & 0x7f800000u) == 0x7f800000u; }

// Any non-finite value among words t0, t0 + stride, ... of n words at p
// (16-byte loads where p is 16-byte aligned).
__device__ __forceinline__ bool scan_nonfinite(const float* p, size_t n, size_t t0, size_t stride) {
    bool bad = false;
    size_t k = t0;
    if (((uintptr_t)p & 15) == 0) {
        const uint4* __restrict__ q = (const uint4*)p;
        const size_t n4 = n >> 2;
        auto any = [](const uint4& v) {
            return nonfinite(v.x) | nonfinite(v.y) | nonfinite(v.z) | nonfinite(v.w);
        };
        for (; k + 3 * stride < n4; k += 4 * stride) {
            const uint4 a = q[k], b = q[k + stride], c = q[k + 2 * stride], d = q[k + 3 * stride];
            bad |= any(a) | any(b) | any(c) | any(d);
        }
        for (; k < n4; k += stride) bad |= any(q[k]);
        k = (n4 << 2) + t0;
    }
    const uint32_t* __restrict__ w = (const uint32_t*)p;
    for (; k < n; k += stride) bad |= nonfinite(w[k]);
    return bad;
}

__device__ __forceinline__ void check_frame(const FrameDesc& f, size_t t0, size_t stride,
                                            uint32_t* flag, uint32_t gen) {
    const size_t px = (size_t)f.H * (size_t)f.W;
    const bool bad = scan_nonfinite(f.pc1, px, t0, stride) |
                     scan_nonfinite(f.prob, px * (size_t)f.C, t0, stride);
    if (ballot(bad) && lane_id() == 0)
        __hip_atomic_store(flag, gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(256) check_frame_kernel(FrameDesc f, uint32_t* flag, uint32_t gen) {
    check_frame(f, (size_t)blockIdx.x * blockDim.x + threadIdx.x, (size_t)gridDim.x * blockDim.x,
                flag, gen);
}

// Frames of a batch table: blockIdx.y strides over the frames, blockIdx.x
// over each frame's values.
__global__ void __launch_bounds__(256)
check_items_kernel(const FrameDesc* __restrict__ frames, uint32_t n, uint32_t* flag, uint32_t gen) {
    for (uint32_t k = blockIdx.y; k < n; k += gridDim.y)
        check_frame(frames[k], (size_t)blockIdx.x * blockDim.x + threadIdx.x,
                    (size_t)gridDim.x * blockDim.x, flag, gen);
}

int launch_check_frame(const FrameDesc& f, uint32_t* flag, uint32_t gen, void* stream) {
    const size_t words = (size_t)f.H * (size_t)f.W * (size_t)(f.C + 1);
    // one 16-byte load per thread (the caller waits for the kernel), at most 1024
    // workgroups: a checked call on 50 x 50 takes 19.9 us, four loads one after
    // another 20.7; 375 x 493 71.5 against 72.8
    const size_t blocks = std::min<size_t>(1024, std::max<size_t>(1, words / (256 * 4)));
    hipLaunchKernelGGL(check_frame_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       (hipStream_t)stream, f, flag, gen);
    return (int)hipGetLastError();
}

int launch_check_items(const FrameDesc* d_frames, uint32_t n, uint32_t max_words, uint32_t* flag,
                       uint32_t gen, void* stream) {
    const unsigned bx = (unsigned)std::min<size_t>(64, std::max<size_t>(1, max_words / (256 * 16)));
    const unsigned by = std::min<unsigned>(n, 65535u);
    hipLaunchKernelGGL(check_items_kernel, dim3(bx, by), dim3(256), 0, (hipStream_t)stream,
                       d_frames, n, flag, gen);
    return (int)hipGetLastError();
}

__global__ void zero_counter_kernel(uint32_t* p) {
    __hip_atomic_store(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

int launch_zero_counter(uint32_t* d_counter, void* stream) {
    hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, d_counter);
    return (int)hipGetLastError();
}

__global__ void __launch_bounds__(256) put_table_kernel(TableWords t, uint32_t* __restrict__ base) {
    for (int r = 0; r < 3; ++r)
        for (uint32_t k = threadIdx.x; k < t.len[r]; k += blockDim.x) base[t.dst[r] + k] = t.w[t.src[r] + k];
}

int launch_put_table(const TableWords& t, uint32_t* d_base, void* stream) {
    hipLaunchKernelGGL(put_table_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, t, d_base);
    return (int)hipGetLastError();
}

// Four independent loads in flight per thread: reads of mapped host memory
// have long latency.
__device__ __forceinline__ uint32_t pair_word(const uint32_t* __restrict__ a, uint32_t na,
                                              const uint32_t* __restrict__ b, uint32_t k) {
    return k < na ? a[k] : b[k - na];
}
__device__ __forceinline__ void pair_put(uint32_t* __restrict__ da, uint32_t na,
                                         uint32_t* __restrict__ db, uint32_t k, uint32_t v) {
    if (k < na)
        da[k] = v;
    else
        db[k - na] = v;
}

__global__ void __launch_bounds__(256)
copy_pair_kernel(const uint32_t* __restrict__ a, uint32_t* __restrict__ da, uint32_t na,
                 const uint32_t* __restrict__ b, uint32_t* __restrict__ db, uint32_t nb) {
    const uint32_t n = na + nb;
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    for (; k + 3 * stride < n; k += 4 * stride) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = pair_word(a, na, b, k + u * stride);
#pragma unroll
        for (int u = 0; u < 4; ++u) pair_put(da, na, db, k + u * stride, v[u]);
    }
    for (; k < n; k += stride) pair_put(da, na, db, k, pair_word(a, na, b, k));
}

int launch_copy_pair(const uint32_t* a, uint32_t* da, uint32_t na, const uint32_t* b,
                     uint32_t* db, uint32_t nb, void* stream) {
    const uint32_t n = na + nb;
    // 64 workgroups already reach the host link's bandwidth (57 GB/s measured)
    const uint32_t blocks = std::max<uint32_t>(1, std::min<uint32_t>(64, (n + 1023) / 1024));
    hipLaunchKernelGGL(copy_pair_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, a, da,
                       na, b, db, nb);
    return (int)hipGetLastError();
}

}  // namespace knnf
