// Match search for gfx950: the first member of the query order without testing
// the order pattern by pattern.
//
// A pattern is a subset of ranks 1..8 and a set u of ranks above 8; it is a
// member iff s0 ^ h(u) is the sum of the subset's columns.  Gauss-Jordan steps
// on the columns h_1..h_8, applied to every rank's column and to s0, turn h_j
// into the unit vector of bit j - 1 (independent columns): s0 ^ h(u) is then
// such a sum iff its other bits are zero, and bits 0..7 are the subset's mask.
// One test per set u covers the 256 patterns that share it: the first 10^5
// patterns hold 2090 sets (33 steps of 64 lanes where testing the patterns
// takes 1563), the first 10^6 about 16 thousand, the first 5 x 10^6 80
// thousand.  The sets come by ascending logistic weight; a match of total
// weight W leaves only the sets of weight <= W to be tested, and the earliest
// match in the order wins.  Its query number comes from count tables
// (match_query), so the order itself is never read.
//
// Bound: the search is short (1 to 4 steps for most blocks), so a block's time
// is its ranking and the latency of a chain of a few table reads.  The ranking
// is therefore partial: patterns of logistic weight <= R flip ranks <= R only,
// so the 44 to 63 least reliable ranks, found with a threshold and sorted one
// key per lane (21 substeps), serve every weight up to their number (10^4
// patterns and more), and the whole block is sorted (28 substeps of two keys
// at n = 127, 45 of eight at n = 512) only when the search goes past it.
//
// Measured, the walk of the order (light and heavy pass) against this search:
// 2 x 10^5 blocks of BCH(127,113) at 4 dB, 10^5 queries, 443 -> 135 us (with the
// first pass); 5003 blocks of n = 512, m = 22, 10^6 queries, 1006 -> 73 us;
// three codes mixed, 10^6 blocks, 4.3 -> 0.90 ms; 10^4 blocks of n = 32, m = 6, 41 -> 13 us.
// About 345 vector and as many scalar instructions a block, 69 % of the issue
// rate of each.
#pragma once
#include "decode_impl.h"

namespace orbg {

// Check bits up to which a match's combinations of null masks (2^(8 - m) at least) are
// spread over the lanes.  In every kernel this costs the searches of other codes 2 to
// 4 % (scalar spills).  100 blocks of n = 128, us, one by one / by lanes / the walk of
// the order: m = 1 37.8 / 16.4 / 21.2, m = 2 22.0 / 16.4 / 21.2; from m = 4 on one by
// one is no slower.
#define ORBG_MATCH_FEW 3
#define ORBG_MATCH_SOME 44       // fewest ranks of a partial ranking (at most 63), where the limit needs as many

template <typename S>
struct MatchLds {
    S h[ORBG_MATCH_RANKS];              // h[r] = transformed column of rank r (h[0] = 0)
    uint32_t stage[ORBG_WAVE];          // keys of the partial ranking
    uint32_t null[ORBG_LOW_RANKS];      // null combinations of ranks 1..8 (masks)
    uint16_t pi[ORBG_MATCH_RANKS];      // pi[r] = received index of rank r
};

// Sum of a u32 over the wave, wave-uniform (all lanes active).
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}

// Largest and smallest u32 of the wave, wave-uniform (all lanes active).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#define ORBG_MAX_STEP(ctrl)                                                              \
    {                                                                                    \
        const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xF, 0xF, false); \
        v = o > v ? o : v;                                                               \
    }
    ORBG_MAX_STEP(0xB1)      // quad_perm [1,0,3,2]
    ORBG_MAX_STEP(0x4E)      // quad_perm [2,3,0,1]
    ORBG_MAX_STEP(0x141)     // row_half_mirror
    ORBG_MAX_STEP(0x140)     // row_mirror
#undef ORBG_MAX_STEP
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    const uint32_t e = a > b ? a : b, f = c > d ? c : d;
    return e > f ? e : f;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) { return ~wave_max_u32(~v); }

// A pattern by its place in the order: key = (logistic weight << 16) | (Hamming
// weight << 8) | (255 - mask of ranks 1..8 with its bits reversed), then the
// ranks above 8 as the big-endian bytes x, y of MatchTable::sets.  Patterns
// compare by (key, x, y): with both weights equal, the first rank that two
// patterns do not share decides, and the pattern that has it comes first, so a
// set bit 0 weighs most; equal masks leave the bytes.
struct Pattern {
    uint32_t key, x, y;
};

__device__ __forceinline__ uint32_t pattern_weight(const Pattern& p) { return p.key >> 16; }
__device__ __forceinline__ uint32_t pattern_mask(const Pattern& p)
{
    return __builtin_bitreverse32(255u - (p.key & 0xffu)) >> 24;
}

// Logistic weight of a mask of ranks 1..8, by the bits of the rank numbers
// (ranks 1, 3, 5, 7 have bit 0 set, and so on).
__device__ __forceinline__ uint32_t mask_weight(uint32_t m)
{
    return __popc(m & 0x55u) + 2u * __popc(m & 0x66u) + 4u * __popc(m & 0x78u) + 8u * (m >> 7);
}

// Ranks held by a set.
__device__ __forceinline__ uint32_t set_size(uint32_t x, uint32_t y)
{
    const uint32_t a = 4u - ((uint32_t)__builtin_ctz(x | 0x80000000u) >> 3);         // x != 0
    const uint32_t b = 7u - ((uint32_t)__builtin_ctz((y >> 8) | 0x80000000u) >> 3);  // y >> 8 != 0
    return (y >> 8) != 0 ? b : x != 0 ? a : 0u;
}

// Query number of a non-empty pattern in the basic order of length n: one more
// than the patterns of smaller logistic weight, those of equal weight and
// smaller Hamming weight, and those of its class before it.  Lane w takes the
// first two counts for Hamming weight w; the class count is the sum, over the
// ranks c outside the pattern, of the subsets that agree with it below c, hold
// c and fill up from above c (lane l takes c = l and l + 64): one round trip
// to the count tables.
__device__ __forceinline__ uint32_t match_query(const Pattern& p, const uint32_t* __restrict__ below,
                                                const uint32_t* __restrict__ above)
{
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t W = pattern_weight(p), w = (p.key >> 8) & 0xffu;
    uint64_t lo = (uint64_t)pattern_mask(p) << 1, hi = 0;  // ranks 0..63 and 64.. of the pattern
    for (uint64_t e = ((uint64_t)p.x << 32) | (p.y & 0xffffff00u); e != 0; e <<= 8) {
        const uint64_t bit = 1ull << ((e >> 56) & 63u);
        if ((e >> 62) != 0) hi |= bit; else lo |= bit;
    }
    // sum over the ranks c = base + lane outside the pattern
    uint32_t n = 0, s = 0;                               // wave-uniform: ranks below base, their sum
    auto count = [&](uint32_t base, uint64_t bits) -> uint32_t {
        const uint32_t c = base + lane;
        const uint32_t nc = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0u));
        uint32_t sc = s;
        for (uint64_t m = bits; m != 0; m &= m - 1) {
            const uint32_t r = base + (uint32_t)__builtin_ctzll(m);
            s += r;
            sc = c > r ? s : sc;
        }
        n += (uint32_t)__builtin_popcountll(bits);
        const bool ok = ((bits >> lane) & 1ull) == 0 && c != 0 && nc < w && sc + c <= W;   // then c <= W <= 100
        const uint32_t i = ok ? (c * 16u + (w - nc - 1u)) * ORBG_MATCH_WCOL + (W - sc - c) : 0u;
        const uint32_t v = above[i];
        return ok ? v : 0u;
    };
    const bool row = lane <= ORBG_WMAX_H;
    const uint32_t b = below[(row ? lane : 0u) * ORBG_MATCH_WCOL + W - (lane >= w ? 1u : 0u)];
    uint32_t v = (row ? b : 0u) + count(0u, lo);
    if (W >= 64u) v += count(64u, hi);
    return 1u + wave_sum(v);
}

// The least reliable ranks of a block: a threshold on |LLR| with want <=
// #(magnitudes below it) <= 63, moved from the caller's guess by steps of a
// quarter and then by halves; the keys below it are gathered through LDS and
// sorted one per lane.  Lane l < cnt then holds the received index of rank
// l + 1.  Returns cnt, or 0 when no threshold is found or two of the keys share
// a truncated magnitude (their order would need the full keys).
template <int NK>
__device__ __forceinline__ uint32_t rank_some(const float (&x)[NK], int n, uint32_t want, float& guess,
                                              uint32_t* stage, uint32_t& idx)
{
    constexpr int IB = IndexBits<NK>::value;
    constexpr uint32_t MOST = ORBG_WAVE - 1;
    const int lane = lane_id();
    float tau = guess, lo_t = 0.0f, hi_t = 0.0f;          // bracket (0: open)
    uint64_t mk[NK];
    uint32_t cnt = 0;
    bool ok = false;
#pragma unroll 1
    for (int it = 0; it < 10; ++it) {
        cnt = 0;
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            // lanes past n hold zeros and are no candidates
            mk[j] = ballot(fabsf(x[j]) < tau) & (n >= (j + 1) * ORBG_WAVE ? ~0ull
                                                 : n <= j * ORBG_WAVE    ? 0ull
                                                                         : (1ull << (n & 63)) - 1ull);
            cnt += (uint32_t)__builtin_popcountll(mk[j]);
        }
        if (cnt >= want && cnt <= MOST) { ok = true; break; }
        const bool up = cnt < want;
        lo_t = up ? tau : lo_t;
        hi_t = up ? hi_t : tau;
        const float open = tau * (up ? 1.25f : 0.8f);
        const float mid = 0.5f * (lo_t + hi_t);
        tau = __uint_as_float(uniform_u32(__float_as_uint(lo_t == 0.0f || hi_t == 0.0f ? open : mid)));
    }
    if (!ok) {
        guess = tau > 0.0f && tau < INFINITY ? tau : 1.0f;   // the next block goes on from here
        return 0;
    }
    uint32_t at = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        const uint32_t key = ((__float_as_uint(x[j]) & 0x7fffffffu) >> (IB - 1)) << IB | (uint32_t)(j * ORBG_WAVE + lane);
        const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk[j] >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)mk[j], at));
        if (__builtin_amdgcn_inverse_ballot_w64(mk[j])) stage[to] = key;
        at += (uint32_t)__builtin_popcountll(mk[j]);
    }
    wave_lds_sync();
    uint32_t k1[1] = {(uint32_t)lane < cnt ? stage[lane] : 0xffffffffu};
    wave_lds_sync();
    sort32<1>(k1);
    const uint32_t next = (uint32_t)__shfl_down((int)k1[0], 1, ORBG_WAVE);
    const bool tie = (uint32_t)lane + 1 < cnt && ((k1[0] ^ next) >> IB) == 0u;
    if (ballot(tie) != 0ull) return 0;
    idx = k1[0] & ((1u << IB) - 1u);
    // next block's guess: the middle of the window
    const uint32_t mid = (want + MOST) / 2;
    const uint32_t e = (mid < cnt ? mid : cnt) - 1;
    const uint32_t g = ((uint32_t)__builtin_amdgcn_readlane((int)k1[0], (int)e) >> IB) + 1u;
    guess = __uint_as_float(g << (IB - 1));
    return cnt;
}

// Gauss-Jordan steps on the columns of ranks 1..8 (rank r in lane r - 1 of
// g[0]), applied to g and to s0 (in a lane of g that holds no rank, or in *sv);
// returns the mask of independent ranks (bit r - 1), the combinations of the
// dependent ones in null[0 .. nulls - 1].
// Column k + 1 with a bit outside the pivots so far: bit k of every vector
// takes one of those bits too if the column's bit k is clear (a row operation;
// bits at or above n - k start as zero rows), and the column's other bits are
// cleared wherever bit k is set.
template <int NC, typename S>
__device__ __forceinline__ S match_reduce(S (&g)[NC], uint32_t* null, uint32_t& nulls, S* sv = nullptr)
{
    S piv = 0;
    nulls = 0;
#pragma unroll
    for (int k = 0; k < ORBG_LOW_RANKS; ++k) {
        const S p = readlane_s<S>(g[0], k);
        const S t = p & ~piv;
        if (t == 0) {                                     // the sum of the pivots in its low bits
            if (lane_id() == 0) null[nulls] = (uint32_t)p | (1u << k);
            ++nulls;
        } else {
            const S pm = p & ~((S)1 << k);
            if (((t >> k) & 1) == 0) {
                const int b = sizeof(S) == 4 ? __builtin_ctz((uint32_t)t) : __builtin_ctzll((uint64_t)t);
#pragma unroll
                for (int j = 0; j < NC; ++j) g[j] ^= ((g[j] >> b) & 1) << k;
                if (sv) *sv ^= ((*sv >> b) & 1) << k;
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) g[j] ^= ((S)0 - ((g[j] >> k) & 1)) & pm;
            if (sv) *sv ^= ((S)0 - ((*sv >> k) & 1)) & pm;
            piv |= (S)1 << k;
        }
    }
    return piv;
}

// Tests the sets from step t on, while their weight is at most min(limit(),
// reach): reach = the ranks whose columns are in L.h (every set of a weight up
// to it holds only those).  visit(pattern) is called for each match whose
// weight is at most limit().  Returns the step to go on from with more ranks.
// FEW (codes of at most ORBG_MATCH_FEW check bits, whose first eight columns have many
// null combinations): for the earliest match of each set only, which is enough where
// the earliest of all is looked for.
template <bool FEW, typename S, typename Limit, typename Visit>
__device__ __forceinline__ uint32_t match_scan(const uint2* __restrict__ sets, const MatchLds<S>& L, S sv, S piv,
                                               uint32_t nulls, uint32_t t, uint32_t reach, Limit&& limit,
                                               Visit&& visit)
{
    const int lane = lane_id();
    uint2 e0 = sets[t * ORBG_WAVE + lane], e1 = sets[(t + 1) * ORBG_WAVE + lane];
    for (;;) {
        const uint32_t first = uniform_u32(e0.y & 0xffu);
        if (first > limit() || first > reach) return t;
        const uint2 e2 = sets[(t + 2) * ORBG_WAVE + lane];
        const S h0 = L.h[e0.x >> 24], h1 = L.h[(e0.x >> 16) & 0xffu], h2 = L.h[(e0.x >> 8) & 0xffu],
                h3 = L.h[e0.x & 0xffu];
        S v = xor3<S>(xor3<S>(sv, h0, h1), h2, h3);
        if (ballot(e0.y > 0xffu) != 0ull) {
            const S i0 = L.h[e0.y >> 24], i1 = L.h[(e0.y >> 16) & 0xffu], i2 = L.h[(e0.y >> 8) & 0xffu];
            v = xor3<S>(v, i0, i1) ^ i2;
        }
        const uint32_t wu = e0.y & 0xffu;
        const bool match = (v & ~piv) == 0 && wu <= reach;
        if (ballot(match) != 0ull) {
            uint32_t m = (uint32_t)v & 0xffu;
            const uint32_t size = set_size(e0.x, e0.y);
            auto key_of = [&](uint32_t w, uint32_t sz, uint32_t mk) -> uint32_t {
                return ((w + mask_weight(mk)) << 16) | ((sz + __popc(mk)) << 8) | (255u - (__builtin_bitreverse32(mk) >> 24));
            };
            if constexpr (FEW) {
                // one match after the other, its combinations of the null masks one per
                // lane
                for (uint64_t left = ballot(match && wu <= limit()); left != 0;) {
                    const int l = __builtin_ctzll(left);
                    const uint32_t ml = (uint32_t)__builtin_amdgcn_readlane((int)m, l);
                    const uint32_t wl = (uint32_t)__builtin_amdgcn_readlane((int)wu, l);
                    const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)size, l);
                    uint32_t least = ~0u;
                    for (uint32_t k = (uint32_t)lane; k < (1u << nulls); k += ORBG_WAVE) {
                        uint32_t mk = ml;
                        for (uint32_t i = 0; i < nulls; ++i) mk ^= ((k >> i) & 1u) != 0 ? L.null[i] : 0u;
                        const uint32_t key = key_of(wl, sl, mk);
                        least = key < least ? key : least;
                    }
                    Pattern p;
                    p.key = wave_min_u32(least);
                    p.x = (uint32_t)__builtin_amdgcn_readlane((int)e0.x, l);
                    p.y = (uint32_t)__builtin_amdgcn_readlane((int)e0.y, l);
                    if (pattern_weight(p) <= limit()) visit(p);
                    left &= left - 1;
                    left &= ballot(wu <= limit());
                }
            }
            // every combination of the null masks (one after the other by Gray code)
            for (uint32_t k = 0; !FEW;) {
                const uint32_t key = key_of(wu, size, m);
                for (uint64_t left = ballot(match && (key >> 16) <= limit()); left != 0;) {
                    const int l = __builtin_ctzll(left);
                    Pattern p;
                    p.key = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
                    p.x = (uint32_t)__builtin_amdgcn_readlane((int)e0.x, l);
                    p.y = (uint32_t)__builtin_amdgcn_readlane((int)e0.y, l);
                    visit(p);
                    left &= left - 1;
                    left &= ballot((key >> 16) <= limit());
                }
                if (++k >= (1u << nulls)) break;
                m ^= uniform_u32(L.null[__builtin_ctz(k)]);
            }
        }
        if ((uint32_t)__builtin_amdgcn_readlane((int)(e0.y & 0xffu), ORBG_WAVE - 1) > reach) return t;
        e0 = e1;
        e1 = e2;
        ++t;
    }
}

// One block: its first member within the budget, written to its outputs.
template <int NK, bool ORDERED, bool FEW, typename S, class CD, class LO>
__device__ __forceinline__ void match_block(const float (&x)[NK], const uint64_t (&hrow)[NK], const CD& c,
                                            const S* __restrict__ cols, MatchLds<S>& L, uint32_t budget,
                                            uint32_t ordv, buf_t cw_row, uint64_t* q_out, uint8_t* ab_out,
                                            float& guess, const LO& lo)
{
    const int lane = lane_id();
    const int n = c.n;
    bool ybit[NK];
    const S s0 = hard_decision<NK, S>(x, n, hrow, ybit);
    constexpr uint32_t ALL = ORBG_MATCH_END - 1;          // reach of every set, not of the end marks
    constexpr uint32_t PREFIX = 64u * ORBG_WAVE;          // patterns a batch order covers
    const uint32_t lim = min(budget, c.slen);
    uint32_t q = 0;                                       // 0: not found
    Pattern best = {~0u, ~0u, ~0u};
    uint32_t empty = 1u;                                  // query 1 is the empty pattern, but not always where a
                                                          // batch order found it
    if (s0 == 0 && (!ORDERED || (uint32_t)__builtin_amdgcn_readfirstlane((int)ordv) == 0u)) {
        q = 1;
    } else {
        const uint32_t wlim = (uint32_t)c.wlim;
        uint32_t idx = 0, reach = 0;
        if (NK > 1)
            reach = rank_some<NK>(x, n, min(min(max(wlim, (uint32_t)ORBG_LOW_RANKS), (uint32_t)ORBG_MATCH_SOME),
                                            (uint32_t)n), guess, L.stage, idx);
        S sv = s0, piv = 0;
        uint32_t nulls = 0;
        if (lane == 0) L.h[0] = 0;
        if (reach != 0) {
            S g[1];
            const S col = cols[(uint32_t)lane < reach ? idx : 0u];
            g[0] = (uint32_t)lane < reach ? col : s0;
            piv = match_reduce<1, S>(g, L.null, nulls);
            sv = readlane_s<S>(g[0], ORBG_WAVE - 1);
            L.h[lane + 1] = g[0];
            L.pi[lane + 1] = (uint16_t)idx;
            wave_lds_sync();
            reach = reach == (uint32_t)n ? ALL : reach;
        }
        // Phase 0, with a batch order: of the matches among the first 4096
        // patterns, the one whose batch comes first in the block's order (a batch
        // that the order leaves out is not tested).  Phase 1: the earliest match
        // (in an ordered decode, past those 4096).
        uint32_t at = ~0u;
        int phase = ORDERED ? 0 : 1;
        const Pattern none = {(wlim << 16) | 0xffffu, ~0u, ~0u};   // after every pattern within the limit
        if (!ORDERED) best = none;
        auto limit = [&]() { return phase == 0 ? (uint32_t)c.wprefix : pattern_weight(best); };
        auto visit = [&](const Pattern& p) {
            if (phase == 0) {
                const uint32_t i = p.key >> 8 == 0u ? 0u : match_query(p, c.below, c.above) - 1u;
                if (i >= PREFIX) return;
                const uint64_t pos = ballot(ordv == i / ORBG_WAVE);
                if (pos == 0ull) return;
                const uint32_t k = (uint32_t)__builtin_ctzll(pos) * ORBG_WAVE + i % ORBG_WAVE;
                if (k < at) {
                    at = k;
                    best = p;
                }
            } else if (p.key < best.key || (p.key == best.key && (p.x < best.x || (p.x == best.x && p.y < best.y)))) {
                if (ORDERED && (p.key >> 8 == 0u || (pattern_weight(p) <= (uint32_t)c.wprefix &&
                                                     match_query(p, c.below, c.above) <= PREFIX)))
                    return;                               // in the reordered prefix
                best = p;
            }
        };
        // (one copy of the whole ranking and of the scan in the kernel: with two of
        // each, and two of the whole block for alternating row buffers, the code
        // came to 60 KB and the waves waited for instructions)
        uint32_t t = 0;
        for (;;) {
            if (reach == 0) {                             // the whole block's ranks
                uint32_t all[NK];
                rank_order<NK, NK == 1>(x, n, c.rdepth, 0, all);
#pragma unroll
                for (int j = 0; j < NK; ++j) {
                    const int e = lane * NK + j;
                    if (e < c.rdepth && e + 1 < ORBG_MATCH_RANKS) L.pi[e + 1] = (uint16_t)all[j];
                }
                wave_lds_sync();
                S g[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int r = lane + 1 + j * ORBG_WAVE;
                    const bool in = r <= c.rdepth && r < ORBG_MATCH_RANKS;
                    const S col = cols[in ? L.pi[r] : 0];
                    g[j] = in ? col : j == 1 && lane == ORBG_WAVE - 1 ? s0 : (S)0;
                }
                piv = match_reduce<2, S>(g, L.null, nulls);
                sv = readlane_s<S>(g[1], ORBG_WAVE - 1);
                L.h[lane + 1] = g[0];
                if (lane + 1 + ORBG_WAVE < ORBG_MATCH_RANKS) L.h[lane + 1 + ORBG_WAVE] = g[1];
                wave_lds_sync();
                reach = ALL;
            }
            t = match_scan<FEW>(c.sets, L, sv, piv, nulls, t, reach, limit, visit);
            if (reach < limit()) {                        // more ranks are needed
                reach = 0;
                continue;
            }
            if (ORDERED && phase == 0) {
                q = at + 1u;                              // 0: no match
                empty = 0u;
                if (q != 0 || lim <= PREFIX) break;
                phase = 1;
                best = none;
                t = 0;
                continue;
            }
            if (best.x != ~0u) q = match_query(best, c.below, c.above);
            break;
        }
        if (q > lim) q = 0;
    }
    uint32_t win_lo = 0, win_hi = 0;
    if (q > empty) {                                      // as a schedule entry: byte 0 the mask, then the ranks
        win_lo = pattern_mask(best) | ((best.x >> 16) & 0xff00u) | (best.x & 0xff0000u) | (best.x << 16 & 0xff000000u);
        win_hi = (best.x & 0xffu) | ((best.y >> 16) & 0xff00u) | (best.y & 0xff0000u) | (best.y << 16 & 0xff000000u);
    }
    write_codeword<NK>(ybit, L, win_lo, win_hi, cw_row, lo);
    write_result(q_out, ab_out, q != 0 ? q : budget, q == 0);
    wave_lds_sync();
}

// Blocks of a launch, one after the other (wave-uniform): every gridDim-th
// position from the workgroup's own, or (marks) the blocks marked ORBG_OPEN in
// every gridDim-th span of `span` (<= 64) abandon flags.  The flags of the next
// span are loaded a span ahead.
struct BlockCursor {
    const uint8_t* marks;
    int64_t nblocks, at;       // at: position, or the span's first block
    int64_t step;
    int span;
    uint64_t open;
    uint32_t ahead;            // per lane: flag of the next span
    __device__ __forceinline__ uint32_t flag(int64_t base) const
    {
        const int64_t b = base + lane_id();
        return lane_id() < span && b < nblocks ? marks[b] : 0u;
    }
    __device__ __forceinline__ BlockCursor(const uint8_t* m, int64_t n, int s) : marks(m), nblocks(n), span(s), open(0)
    {
        step = (int64_t)gridDim.x * (m ? s : 1);
        at = (int64_t)blockIdx.x * (m ? s : 1) - step;
        ahead = m ? flag(at + step) : 0u;
    }
    // next block, or -1
    __device__ __forceinline__ int64_t next()
    {
        if (marks == nullptr) {
            at = uniform_i64(at + step);
            return at < nblocks ? at : -1;
        }
        while (open == 0) {
            at = uniform_i64(at + step);
            if (at >= nblocks) {
                at -= step;                               // stays past the end on every later call
                return -1;
            }
            open = ballot(ahead == ORBG_OPEN);
            ahead = flag(at + step);
        }
        const int64_t b = at + __builtin_ctzll(open);
        open &= open - 1;
        return uniform_i64(b);
    }
};

// Waves per SIMD the registers are cut for: as many as the search fits without
// spilling vector registers (left alone it takes 79 at two keys per lane, six
// waves; at eight waves mixed codes go from 1082 to 990 us, BCH(127,113) 7
// points from 1999 to 1968; n = 512 loses, 73.8 instead of 72.8 us, and stays).
template <int NK, bool ORDERED, typename S>
constexpr int match_waves()
{
    const int less = ORDERED ? 1 : 0;
    return sizeof(S) == 8 ? 1 : NK == 2 ? 8 - less : NK == 4 ? 6 - less : 1;
}

// One wave per block.  marks (or nullptr): only the blocks marked ORBG_OPEN in
// the abandon flags.  ids (or nullptr): position i decodes the caller's block
// ids[i]; ORDERED: with the batch order of row i.  Every lookup uses NK keys
// per lane (the largest of the launch's codes; keys past a code's length are
// ranked last).
template <int NK, bool ORDERED, typename S, bool MIXED, bool FEW>
__global__ void __launch_bounds__(ORBG_WAVE, (match_waves<NK, ORDERED, S>()))
match_kernel(CodeTable codes, const uint8_t* __restrict__ block_code, const int64_t* __restrict__ row_off,
             const float* __restrict__ llr, int64_t nblocks, uint32_t budget, const uint8_t* __restrict__ order,
             uint8_t* __restrict__ cw, uint64_t* __restrict__ queries, uint8_t* abandoned, int span,
             const int64_t* __restrict__ ids, int64_t row_limit)
{
    extern __shared__ __align__(16) unsigned char orbg_dyn_lds[];
    uint64_t* s_rows = reinterpret_cast<uint64_t*>(orbg_dyn_lds);
    S* s_cols = reinterpret_cast<S*>(orbg_dyn_lds + (size_t)codes.rwords * sizeof(uint64_t));
    __shared__ MatchLds<S> L;
    BlockCursor cur(span > 0 ? abandoned : nullptr, nblocks, span);
    int64_t b = cur.next();
    if (b < 0) return;
    struct In {
        float x[NK];
        int64_t oid, row;
        uint32_t ordv;
        int ci;
    };
    auto fetch = [&](In& f, int64_t i) {
        const bool ok = i >= 0;
        int ci = 0;
        int64_t oid = 0, row = 0;
        if (ok) {
            oid = ids ? scalar_load_i64(ids, i) : i;
            if (MIXED) {
                ci = (int)scalar_load_u8(block_code, oid);
                ci = ci < codes.ncodes ? ci : 0;          // out-of-range indices read code 0
                row = scalar_load_i64(row_off, oid);
                row = uniform_i64((row >= 0 && row <= row_limit - codes.c[ci].n) ? row : -1);
            } else {
                row = oid * codes.c[0].n;
            }
        }
        f.ci = ci;
        f.oid = oid;
        f.row = row;
        const bool rv = ok && row >= 0;
        load_row_buf<NK>(make_buf(llr + (rv ? row : 0), rv ? (uint32_t)codes.c[ci].n * 4u : 0u), f.x);
        f.ordv = ORDERED ? load_order_buf(make_buf(order + (ok ? i : 0) * 64, ok ? 64u : 0u)) : 0u;
    };
    In cur_in, next_in;
    fetch(cur_in, b);
    for (int ci = 0; ci < (MIXED ? codes.ncodes : 1); ++ci) {
        const CodeDesc& c = codes.c[ci];
        for (int i = threadIdx.x; i < c.n; i += ORBG_WAVE) s_cols[c.col_base + i] = (S)c.cols[i];
        for (int i = threadIdx.x; i < c.m * c.nk; i += ORBG_WAVE) s_rows[c.row_base + i] = c.rows[i];
    }
    wave_lds_sync();
    constexpr bool HOIST = !MIXED && NK <= 4;
    uint64_t hrow0[NK];
    if (HOIST) load_hrows<NK>(s_rows, codes.c[0].m, hrow0);
    float guess = 4.0f;
    typedef const __attribute__((address_space(4))) CodeTable* const_table_ptr;
    const_table_ptr table = (const_table_ptr)__builtin_amdgcn_kernarg_segment_ptr();   // `codes`, the first argument
    // the next block's row loads while this one is decoded
    for (;;) {
        b = cur.next();
        fetch(next_in, b);
        // the code's fields are read where they are used (scalar loads): kept in
        // registers over the loop they spill, and come back by vector instructions
        asm volatile("" : "+s"(table));
        const auto& c = table->c[MIXED ? cur_in.ci : 0];
        uint64_t hr[NK];
        if (HOIST) {
#pragma unroll
            for (int j = 0; j < NK; ++j) hr[j] = hrow0[j];
        } else {
            load_hrows_pad<NK>(s_rows + c.row_base, c.m, c.nk, hr);
        }
        match_block<NK, ORDERED, FEW, S>(cur_in.x, hr, c, s_cols + c.col_base, L, budget, cur_in.ordv,
                                    make_buf(cw + (cur_in.row >= 0 ? cur_in.row : 0), cur_in.row >= 0 ? (uint32_t)c.n : 0u),
                                    queries + cur_in.oid, abandoned + cur_in.oid, guess, NoOffs{});
        if (b < 0) break;
        cur_in = next_in;
    }
}

template <int NK, bool ORDERED, typename S, bool MIXED, bool FEW = false>
static hipError_t launch_match_as(const DecodeArgs& a, bool marked, hipStream_t stream)
{
    uint32_t ncols = 0;
    for (int i = 0; i < (MIXED ? a.codes.ncodes : 1); ++i) {
        const uint32_t e = a.codes.c[i].col_base + (uint32_t)a.codes.c[i].n;
        ncols = e > ncols ? e : ncols;
    }
    const size_t lds = (size_t)a.codes.rwords * sizeof(uint64_t) + ncols * sizeof(S);
    const int64_t most = (int64_t)a.cus * 64;
    int span = 0;
    if (marked) {
        // short spans for small batches, so that no wave is left with many of the marked blocks
        span = 4;
        while (span < 64 && a.nblocks / span > 2 * most) span *= 2;
    }
    const int64_t units = marked ? (a.nblocks + span - 1) / span : a.nblocks;
    const int64_t grid = units < most ? units : most;
    match_kernel<NK, ORDERED, S, MIXED, FEW><<<(unsigned)grid, ORBG_WAVE, lds, stream>>>(
        a.codes, a.block_code, a.row_off, a.llr, a.nblocks, a.budget, a.order, a.cw, a.queries, a.abandoned, span,
        a.ids, a.row_limit);
    return hipGetLastError();
}

template <int NK>
hipError_t launch_match_nk(const DecodeArgs& a, bool s32, bool marked, hipStream_t stream)
{
    if (a.mixed) {
        if constexpr (NK <= 4)
            return s32 ? launch_match_as<NK, false, uint32_t, true>(a, marked, stream)
                       : launch_match_as<NK, false, uint64_t, true>(a, marked, stream);
        return hipErrorInvalidValue;                      // mixed launches take n <= 256
    }
    if (a.order)
        return s32 ? launch_match_as<NK, true, uint32_t, false>(a, marked, stream)
                   : launch_match_as<NK, true, uint64_t, false>(a, marked, stream);
    if (a.codes.c[0].m <= ORBG_MATCH_FEW) return launch_match_as<NK, false, uint32_t, false, true>(a, marked, stream);
    return s32 ? launch_match_as<NK, false, uint32_t, false>(a, marked, stream)
               : launch_match_as<NK, false, uint64_t, false>(a, marked, stream);
}

}  // namespace orbg
