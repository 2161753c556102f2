// Match search of full (m-line) ORBGRAND for gfx950 (order and fit as in
// mline_impl.h; Sec. III-D and III-E).
//
// A pattern's reliability weight is the sum of its ranks' weights (rank r of
// segment i weighs J_{i-1} + beta_i (r - I_{i-1})), so the match search of
// match_impl.h applies with other weights: Gauss-Jordan steps turn the columns
// of ranks 1..8 into unit vectors, one test per set u of higher ranks tells
// which subset of ranks 1..8 completes it to a member, and the member of least
// weight (the earliest in the order among equals) is the result.  The query
// number is a count: the patterns of smaller weight are, set by set, the subsets
// of ranks 1..8 that keep the total below it (a table of their weights), and
// those of equal weight are compared with the result one by one.
//
// The sets come from lists per size (MlineSets), each by ascending sum of ranks.
// Sets of weight <= L lie in a prefix of each list (a linear lower bound on the
// weights bounds their rank sum).  L grows level by level until the best match
// weighs no more than L, or the patterns up to L exceed the budget.
//
// Bound: vector issue; the full sort of a block (56 compare-exchanges of two
// keys at n = 127) and its fit are a third of the instructions, the search of
// most blocks takes one or two steps.  10^6 blocks of BCH(127,113) at 5 dB, two
// lines: 18.0 -> 1.54 ms (the walk of mline_kernel before); 10^5 blocks of n =
// 256, three lines, 5.5 dB: 38.7 -> 1.07 ms.  Not covered, and left marked in the
// abandon flag for mline_kernel: results of weight 511 and more (its wide variant
// takes them up to 2^18 - 2), sets of more than seven ranks above 8, sets of two and
// more with a rank above 254, or past the lists.
#pragma once
#include "match_impl.h"
#include "orbg_mline.h"

namespace orbg {

// Weights are cut at the cap; results below it are exact.  Narrow searches hold
// the subset weights as a table of 512 counts and a pattern's segment weights in
// 10 bits each; wide ones (the rare fits with a nearly flat first segment) as a
// sorted list and in words of their own.
#define ORBG_MM_HIST 512
template <bool WIDE>
constexpr uint32_t mm_cap() { return WIDE ? (1u << 18) - 1u : ORBG_MM_HIST - 1u; }

// A pattern's weights in segments 1..3 (narrow: all in a, segment 1 on top) and
// its flips per segment (8 bits each, segment 1 lowest).
struct MmSplit {
    uint32_t a, b, c, f;
};
__device__ __forceinline__ MmSplit operator+(const MmSplit& p, const MmSplit& q)
{
    return {p.a + q.a, p.b + q.b, p.c + q.c, p.f + q.f};
}
template <bool WIDE>
struct MmSplitLds { uint32_t a, f; };
template <>
struct MmSplitLds<true> { uint32_t a, b, c, f; };
template <bool WIDE>
__device__ __forceinline__ MmSplit get_split(const MmSplitLds<WIDE>& p)
{
    if constexpr (WIDE) return {p.a, p.b, p.c, p.f};
    else return {p.a, 0u, 0u, p.f};
}
template <bool WIDE>
__device__ __forceinline__ MmSplitLds<WIDE> put_split(const MmSplit& p)
{
    if constexpr (WIDE) return {p.a, p.b, p.c, p.f};
    else return {p.a, p.f};
}

// Ranks that the sets of two ranks and more can hold, by the code's width.  The
// slot after the last one is the end marks' rank.  Single ranks past it have the
// pattern bytes (255, then the rank - 255 in the last byte), ORBG_MM_SINGLE being
// the largest.  Those from 256 on lie in the last segment (its first rank is at
// most 256: anchors but the last are below floor(n / 2) <= 256) and share a
// split; rank 255 may end the segment before and has its own.
#define ORBG_MM_SINGLE 510
template <int NK>
constexpr int mm_ranks() { return NK <= 2 ? ORBG_MATCH_RANKS : ORBG_MM_RANKS; }

template <int NK, typename S, bool WIDE>
struct MmLds {
    struct Rank { S h; uint32_t v; };
    Rank r[mm_ranks<NK>() + 2];            // transformed column and weight of rank r (0: none)
    MmSplitLds<WIDE> split[mm_ranks<NK>() + 3];   // of rank r alone (single ranks: slots 255 and 256)
    struct { uint32_t v; MmSplitLds<WIDE> split; } nib[32];   // subsets of ranks 1..4 and 5..8
    union {
        uint32_t hist[ORBG_MM_HIST];    // narrow: hist[w] = subsets of ranks 1..8 of weight <= w;
                                        // wide: weight << 8 | subset, ascending
        float x[NK * ORBG_WAVE];        // |LLR| by received index, while the ranks are made
    };
    float L[NK <= 2 ? ORBG_WAVE + 1 : NK * 32 + 1];   // |LLR| of ranks 1..n/2
    uint32_t null[ORBG_LOW_RANKS];
    uint16_t pi[(NK <= 2 ? ORBG_MATCH_RANKS : NK * ORBG_WAVE) + 2];
    uint8_t sub[256];                   // narrow: the subsets by ascending weight
};

// The fitted model (wave-uniform): m segments, segment i of ranks I[i] + 1 ..
// I[i + 1], offsets J[i], slopes B[i].
struct MmModel {
    int m;
    int I[ORBG_ML_MSEG + 1];
    int J[ORBG_ML_MSEG], B[ORBG_ML_MSEG];
};

// Fit and quantization of fit_model (mline_impl.h), the anchors in scalars and
// one segment per lane in the quantization.  L[1 .. n / 2] in LDS.
template <int NK>
__device__ __forceinline__ MmModel fit_lines(const float* L, int n, int mreq, bool jdiv)
{
    const int lane = lane_id();
    MmModel md;
    md.m = 1;
    md.I[0] = 0;
#pragma unroll
    for (int i = 1; i <= ORBG_ML_MSEG; ++i) md.I[i] = n;
#pragma unroll
    for (int i = 0; i < ORBG_ML_MSEG; ++i) { md.J[i] = 0; md.B[i] = 1; }
    const int h = n / 2;
    if (h < 2) return md;
    constexpr int T = NK <= 2 ? 1 : NK / 2;               // ranks per lane: lane + 1 + 64 t <= h <= 32 NK
    float lj[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int j = lane + 1 + t * ORBG_WAVE;
        lj[t] = L[j <= h ? j : 1];
    }
    int anc[ORBG_ML_MSEG + 1] = {1, h, h, h, h};          // ascending, h past the last
    int na = 2;
    for (int it = 1; it < mreq; ++it) {
        uint32_t gap[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int j = lane + 1 + t * ORBG_WAVE;
            int a = anc[0], b = anc[1];
#pragma unroll
            for (int p = 1; p < ORBG_ML_MSEG; ++p) {
                const bool past = j >= anc[p];
                a = past ? anc[p] : a;
                b = past ? anc[p + 1] : b;
            }
            const bool in = j > a && j < b;               // strictly between two neighbours
            a = in ? a : 1;
            b = in ? b : 2;
            const float La = L[a], Lb = L[b];
            const float s = __fdiv_rn(__fsub_rn(Lb, La), (float)(b - a));
            const float line = __fadd_rn(La, __fmul_rn((float)(j - a), s));
            const float g = fabsf(__fsub_rn(lj[t], line));
            gap[t] = in && !__builtin_isnan(g) ? __float_as_uint(g) : 0u;
        }
        uint32_t top = gap[0];
#pragma unroll
        for (int t = 1; t < T; ++t) top = gap[t] > top ? gap[t] : top;
        top = wave_max_u32(top);
        if (top == 0u) break;                             // no rank between anchors, or the largest gap is 0
        int bj = 0;                                       // smallest rank at the largest gap
#pragma unroll
        for (int t = T - 1; t >= 0; --t) {
            const uint64_t at = ballot(gap[t] == top);
            bj = at != 0 ? t * ORBG_WAVE + (int)__builtin_ctzll(at) + 1 : bj;
        }
#pragma unroll
        for (int p = ORBG_ML_MSEG; p >= 1; --p) {         // insert
            const int prev = anc[p - 1];
            anc[p] = prev > bj ? prev : anc[p] > bj ? bj : anc[p];
        }
        ++na;
    }
    const int m = na - 1;
    // lane i: segment i between anchors i and i + 1
    int lo = anc[0], hi = anc[1];
#pragma unroll
    for (int p = 1; p < ORBG_ML_MSEG; ++p) {
        lo = lane == p ? anc[p] : lo;
        hi = lane == p ? anc[p + 1] : hi;
    }
    const bool seg = lane < m;
    const float Llo = L[lo], d = __fsub_rn(L[hi], Llo), len = (float)(seg ? hi - lo : 1);
    const float sl = __fdiv_rn(d, len);
    float Q = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sl), 0));
#pragma unroll
    for (int i = 1; i < ORBG_ML_MSEG; ++i) {
        const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sl), i));
        Q = i < m && s < Q ? s : Q;
    }
    if (!(Q > 0.0f) || !__builtin_isfinite(Q)) return md;
    const float bf = __fdiv_rn(d, __fmul_rn(len, Q)), jf = __fdiv_rn(Llo, Q);
    // [x] = floor(x + 1/2), capped at 2^20
    auto round_cap = [](float x) {
        const float r = floorf(__fadd_rn(x, 0.5f));
        return r > 1048576.0f ? 1048576.0f : r;
    };
    const bool fin = __builtin_isfinite(bf) && __builtin_isfinite(jf);
    const int B = fin ? (int)round_cap(bf) : 0;
    int J = fin ? (int)round_cap(jf) : 0;
    if (ballot(seg && (!fin || B < 1)) != 0ull) return md;
    if (lane == 0) J -= B;
    if (jdiv) {                                           // [J / B] B in exact arithmetic
        const int num = 2 * J + B, den = seg ? 2 * B : 1;
        int q = num / den;
        if (num % den != 0 && num < 0) --q;
        J = q * B;
    }
    md.m = m;
#pragma unroll
    for (int i = 0; i < ORBG_ML_MSEG; ++i) {
        if (i >= 1) md.I[i] = i < m ? anc[i] : n;
        if (i < m) {
            md.J[i] = __builtin_amdgcn_readlane(J, i);
            md.B[i] = __builtin_amdgcn_readlane(B, i);
        }
    }
    return md;
}

// A pattern: weight W, mask of ranks 1..8, ranks above 8 as big-endian bytes.
struct MmPattern {
    uint32_t W, mask, x, y;
};

// One block after its syndrome s0 != 0 is known and its ranks, weights and
// columns are in LDS.  Returns 0 (not covered), 1 (found) or 2 (no member
// within the budget).
template <int NK, typename S, bool WIDE, class TT>
struct MmSearch {
    static constexpr uint32_t CAP = mm_cap<WIDE>();
    MmLds<NK, S, WIDE>& L;
    const TT& T;
    S sv, piv;
    uint32_t nulls, budget;
    S g[NK];                       // columns and weights of ranks lane + 1 + 64 j
    uint32_t vr[NK];
    uint32_t lone;                 // lightest rank above 8
    uint32_t done;                 // lane c: entries of list c tested so far

    // Prefix of each list that holds all its sets of weight <= w (lane c: list c);
    // false where a list, or the lists together, do not reach that far.  A rank
    // of such a set of c weighs at most w - (c - 1) lone; over the ranks that do,
    // v_r >= (a r + g) / k (a: the slope from the lowest of them to the highest,
    // though any positive value is valid; g exact for it), so the set's rank sum
    // is at most (k w - c g) / a, and that of the c highest such ranks (on a nearly
    // flat stretch a is small and the first bound says little).
    __device__ __forceinline__ bool prefixes(uint32_t w, uint32_t& end) const
    {
        const uint32_t lane = (uint32_t)lane_id();
        end = 0;
        constexpr int NC = NK <= 4 ? NK : 4;               // the ranks of sets
        const int k = !WIDE || w < 4096u ? 64 : 1;         // (where the weights leave room)
        for (uint32_t c = 2; c <= ORBG_HIGH_SLOTS + 1 && c * lone <= w; ++c) {
            const uint32_t top = w - (c - 1) * lone;
            uint64_t some = 0;                            // (not empty: top is at least the lightest)
            uint32_t rlo = 0, rhi = 0;
            auto high = [&](int j) {
                const uint32_t r = lane + 1 + 64 * (uint32_t)j;
                return vr[j] <= top && (j > 0 || r > ORBG_LOW_RANKS) && (NK < 4 || j < 3 || r <= ORBG_MM_RANKS);
            };
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const uint64_t b = ballot(high(j));
                rhi = b != 0 ? 64u * (uint32_t)j + 64u - (uint32_t)__builtin_clzll(b) : rhi;
                rlo = some == 0 && b != 0 ? 64u * (uint32_t)j + (uint32_t)__builtin_ctzll(b) + 1u : rlo;
                some |= b;
            }
            if (some == 0) continue;                      // (the lightest rank lies past the sets')
            const int vlo = (int)uniform_u32(L.r[rlo].v), vhi = (int)uniform_u32(L.r[rhi].v);
            int a = k;
            if (rhi > rlo) a = (int)((float)k * (float)(vhi - vlo) * __builtin_amdgcn_rcpf((float)(rhi - rlo)));
            a = a < 4 ? (k == 1 ? (a < 1 ? 1 : a) : 4) : a;
            a = (int)uniform_u32((uint32_t)a);
            int gm = 0x3fffffff;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int gj = k * (int)vr[j] - a * (int)(lane + 1 + 64 * j);
                gm = high(j) && gj < gm ? gj : gm;
            }
            const int g = (int)(wave_min_u32((uint32_t)gm ^ 0x80000000u) ^ 0x80000000u);
            const int num = k * (int)w - (int)c * g;
            const float fs = (float)num * __builtin_amdgcn_rcpf((float)a) * 1.00001f + 0.01f;
            const int line = num < 0 ? 0 : (int)uniform_u32((uint32_t)(fs < 1e6f ? (int)fs : 1000000));
            const int tops = (int)(c * rhi) - (int)(c * (c - 1) / 2);   // (below 9 c and more: no such set)
            const int sum = line < tops ? line : tops < 0 ? 0 : tops;
            if (c > ORBG_HIGH_SLOTS) return sum < 100;    // 9 + ... + 16: a set of eight
            if (sum > T.limit[c]) return false;
            const uint32_t e = T.end[c * ORBG_MM_SUMS + (uint32_t)(sum < ORBG_MM_SUMS ? sum : ORBG_MM_SUMS - 1)];
            end = lane == c ? e : end;
        }
        return true;
    }

    // weight and packed values of a subset of ranks 1..8
    __device__ __forceinline__ uint32_t mask_weight_of(uint32_t m) const
    {
        return L.nib[m & 15u].v + L.nib[16u + (m >> 4)].v;
    }

    // Is pattern (m, x, y; split p) before `o` (split po), both of weight W?
    // Splits first; equal splits: in the first segment they differ in, fewer
    // flips, else the one that has the first rank not shared.
    __device__ __forceinline__ bool before(uint32_t m, uint32_t x, uint32_t y, const MmSplit& p, const MmPattern& o,
                                           const MmSplit& po) const
    {
        if (p.a != po.a) return p.a < po.a;
        if (p.b != po.b) return p.b < po.b;
        if (p.c != po.c) return p.c < po.c;
        uint32_t r, has;
        if (m != o.mask) {
            const uint32_t d = m ^ o.mask;
            r = (uint32_t)__builtin_ctz(d) + 1u;
            has = (m >> (r - 1u)) & 1u;
        } else {
            const uint32_t dx = x ^ o.x, dy = y ^ o.y;
            const bool inx = dx != 0;
            const uint32_t d = inx ? dx : dy;
            const uint32_t sh = d != 0 ? 24u - ((uint32_t)__builtin_clz(d) & 24u) : 0u;
            const uint32_t ra = ((inx ? x : y) >> sh) & 0xffu, rb = ((inx ? o.x : o.y) >> sh) & 0xffu;
            has = ra < rb;                                // both held: equal weights leave none shorter
            r = ra < rb ? ra : rb;
            if (d == 0) return false;                     // the pattern itself
        }
        const uint32_t field = L.split[r].f * 0xffu;      // flips of r's segment
        const uint32_t wa = p.f & field, wb = po.f & field;
        return wa != wb ? wa < wb : has != 0;
    }

    __device__ __forceinline__ MmSplit mask_split(uint32_t m) const
    {
        return get_split<WIDE>(L.nib[m & 15u].split) + get_split<WIDE>(L.nib[16u + (m >> 4)].split);
    }

    __device__ __forceinline__ MmSplit split_of(uint32_t m, uint32_t x, uint32_t y) const
    {
        MmSplit p = mask_split(m);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t r = (x >> (24 - 8 * k)) & 0xffu;
            p = p + get_split<WIDE>(L.split[NK >= 4 && k == 0 && (y & 0xffu) != 0 ? r + 1u : r]);
        }
        if (ballot(y != 0u) != 0ull) {
#pragma unroll
            for (int k = 0; k < 3; ++k) p = p + get_split<WIDE>(L.split[(y >> (24 - 8 * k)) & 0xffu]);
        }
        return p;
    }

    // Table of the subsets of ranks 1..8 by weight: hist (cumulative) and sub.
    __device__ __forceinline__ void sort_subsets() const
    {
        const uint32_t lane = (uint32_t)lane_id();
        if constexpr (WIDE) {
            uint32_t key[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t m = k * ORBG_WAVE + lane;
                key[k] = mask_weight_of(m) << 8 | m;      // at most 8 x 2^18, below 2^21
            }
            sort32<4>(key);
#pragma unroll
            for (int k = 0; k < 4; ++k) L.hist[lane * 4 + k] = key[k];
            wave_lds_sync();
            return;
        }
#pragma unroll
        for (int k = 0; k < ORBG_MM_HIST / ORBG_WAVE; ++k) L.hist[k * ORBG_WAVE + lane] = 0u;
        wave_lds_sync();
        uint32_t w[4], at[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            w[k] = mask_weight_of(k * ORBG_WAVE + lane);
            w[k] = w[k] < CAP ? w[k] : CAP;
            at[k] = atomicAdd(&L.hist[w[k]], 1u);         // place inside its weight
        }
        wave_lds_sync();
        // inclusive sums, eight weights per lane
        uint32_t c[8], s = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s += L.hist[lane * 8 + k];
            c[k] = s;
        }
        uint32_t sum = s;
#pragma unroll
        for (int d = 1; d < ORBG_WAVE; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)sum, d, ORBG_WAVE);
            sum += lane >= (uint32_t)d ? o : 0u;
        }
        const uint32_t base = sum - s;
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 8; ++k) L.hist[lane * 8 + k] = base + c[k];
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t start = w[k] != 0 ? L.hist[w[k] - 1] : 0u;
            L.sub[start + at[k]] = (uint8_t)(k * ORBG_WAVE + lane);
        }
        wave_lds_sync();
    }

    // Subsets of ranks 1..8 of weight <= w.
    __device__ __forceinline__ uint32_t subsets_upto(uint32_t w) const
    {
        if constexpr (!WIDE) return L.hist[w];
        uint32_t n = 0;                                   // entries known to be <= w
        const uint32_t top = w << 8 | 0xffu;
#pragma unroll
        for (uint32_t d = 128; d != 0; d >>= 1) n += L.hist[n + d - 1] <= top ? d : 0u;
        return n + (n == 255u && L.hist[255] <= top ? 1u : 0u);
    }

    // f(x, y) for the entries [from_c, end_c) of every list, in whole steps.
    template <typename F>
    __device__ __forceinline__ void each_step(uint32_t from, uint32_t end, F&& f) const
    {
        const uint32_t lane = (uint32_t)lane_id();
        for (uint32_t c = 2; c <= ORBG_HIGH_SLOTS; ++c) {
            const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)end, (int)c);
            uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)from, (int)c);
            if (p >= e) continue;
            const uint2* s = T.sets + T.start[c];
            uint2 nx = s[p + lane];
            for (; p < e; p += ORBG_WAVE) {
                const uint2 cur = nx;
                nx = s[p + ORBG_WAVE + lane];             // the lists end in two steps of end marks
                f(cur.x, cur.y);
            }
        }
    }

    // f(x, y, weight, column, slot of its split) for the empty set (lane 0 of the
    // first step) and the single ranks above 8; weight ~0 where a lane holds neither.
    template <typename F>
    __device__ __forceinline__ void each_single(F&& f) const
    {
        const uint32_t lane = (uint32_t)lane_id();
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            const uint32_t r = lane + 1 + 64 * (uint32_t)j;
            const bool low = j == 0 && r <= ORBG_LOW_RANKS, far = NK >= 4 && r > ORBG_MM_RANKS;
            const uint32_t wu = low ? (lane == 0 ? 0u : ~0u) : (NK < 8 || r <= ORBG_MM_SINGLE) ? vr[j] : ~0u;
            f(low ? 0u : far ? (uint32_t)(ORBG_MM_RANKS + 1) << 24 : r << 24,
              far ? r - (ORBG_MM_RANKS + 1) : 0u, wu, low ? (S)0 : g[j],
              low ? 0u : r < ORBG_MM_RANKS + 2u || !far ? r : ORBG_MM_RANKS + 2u);
        }
    }

    // One more than the patterns before o when every rank above 8 weighs more:
    // the 256 subsets of ranks 1..8, four per lane.
    __device__ __forceinline__ uint32_t count_low(const MmPattern& o) const
    {
        const uint32_t lane = (uint32_t)lane_id();
        const MmSplit po = mask_split(o.mask);
        const uint32_t vl = L.nib[lane & 15u].v;
        const MmSplit pl = get_split<WIDE>(L.nib[lane & 15u].split);
        uint32_t n = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const auto& hi = L.nib[16u + 4u * (uint32_t)k + (lane >> 4)];
            const uint32_t w = vl + hi.v;
            const bool bf = before((lane & 15u) | (4u * (uint32_t)k + (lane >> 4)) << 4, 0u, 0u,
                                   pl + get_split<WIDE>(hi.split), o, po);
            n += w < o.W || (w == o.W && bf) ? 1u : 0u;
        }
        return 1u + wave_sum(n);
    }

    // Patterns of weight < w, and (with o) those of weight w before o, plus one.
    __device__ __forceinline__ uint64_t count(uint32_t w, uint32_t end, bool with, const MmPattern& o) const
    {
        MmSplit po = {0u, 0u, 0u, 0u};
        if (with) po = split_of(o.mask, o.x, o.y);
        uint32_t total = 0;                               // per lane: at most 256 per set
        const uint32_t second = WIDE ? uniform_u32(L.hist[1] >> 8) : 0u;
        auto add = [&](uint32_t x, uint32_t y, uint32_t wu, auto&& split) {
            const bool some = wu <= w;
            const uint32_t left = some ? w - wu : 0u;
            uint32_t upto = 1u, under = left != 0 ? 1u : 0u;
            // (wide: most steps leave room for the empty subset alone)
            if (!WIDE || ballot(left >= second) != 0ull) {
                upto = subsets_upto(left);
                under = left != 0 ? subsets_upto(left - 1u) : 0u;
            }
            uint32_t n = some ? under : 0u;
            if (with) {
                MmSplit p = {0u, 0u, 0u, 0u};
                const uint32_t k = some ? upto - under : 0u;
                if (ballot(k != 0u) != 0ull) p = split();
                for (uint32_t i = 0; ballot(i < k) != 0ull; ++i) {
                    const uint32_t at = i < k ? under + i : 0u;
                    const uint32_t m = WIDE ? L.hist[at] & 0xffu : L.sub[at];
                    const bool bf = before(m, x, y, p + mask_split(m), o, po);
                    n += i < k && bf ? 1u : 0u;
                }
            }
            total += n;
        };
        each_single([&](uint32_t x, uint32_t y, uint32_t wu, S, uint32_t r) {
            add(x, y, wu, [&]() { return get_split<WIDE>(L.split[r]); });
        });
        each_step(0u, end, [&](uint32_t x, uint32_t y) {
            add(x, y, weight(x, y), [&]() { return split_of(0u, x, y); });
        });
        return (uint64_t)wave_sum(total) + (with ? 1u : 0u);
    }

    __device__ __forceinline__ uint32_t weight(uint32_t x, uint32_t y) const
    {
        uint32_t w = L.r[x >> 24].v + L.r[(x >> 16) & 0xffu].v + L.r[(x >> 8) & 0xffu].v + L.r[x & 0xffu].v;
        if (ballot(y != 0u) != 0ull) w += L.r[y >> 24].v + L.r[(y >> 16) & 0xffu].v + L.r[(y >> 8) & 0xffu].v;
        return w;
    }

    // Completes the sets of a step to members and keeps the earliest.
    __device__ __forceinline__ void test(S v, uint32_t x, uint32_t y, uint32_t wu, MmPattern& best) const
    {
        auto limit = [&]() { return best.W < CAP ? best.W : CAP - 1u; };
        const bool match = (v & ~piv) == 0 && wu <= limit();
        if (ballot(match) == 0ull) return;
        uint32_t m = (uint32_t)v & 0xffu;
        for (uint32_t k = 0;;) {
            const uint32_t W = wu + mask_weight_of(m);
            for (uint64_t left = ballot(match && W <= limit()); left != 0;) {
                const int l = __builtin_ctzll(left);
                MmPattern p;
                p.W = (uint32_t)__builtin_amdgcn_readlane((int)W, l);
                p.mask = (uint32_t)__builtin_amdgcn_readlane((int)m, l);
                p.x = (uint32_t)__builtin_amdgcn_readlane((int)x, l);
                p.y = (uint32_t)__builtin_amdgcn_readlane((int)y, l);
                bool take = p.W < best.W;
                if (!take) {
                    take = uniform_u32(before(p.mask, p.x, p.y, split_of(p.mask, p.x, p.y), best,
                                              split_of(best.mask, best.x, best.y)) ? 1u : 0u) != 0u;
                }
                if (take) best = p;
                left &= left - 1;
                left &= ballot(W <= limit());
            }
            if (++k >= (1u << nulls)) break;
            m ^= uniform_u32(L.null[__builtin_ctz(k)]);
        }
    }

    // far: lightest rank past those that the sets hold; none: past the single ones.
    __device__ __forceinline__ int run(uint32_t far, uint32_t none, MmPattern& best, uint32_t& q)
    {
        const uint32_t lane = (uint32_t)lane_id();
        best = {CAP, 0u, 0u, 0u};                         // none yet
        each_single([&](uint32_t x, uint32_t y, uint32_t wu, S col, uint32_t) { test(sv ^ col, x, y, wu, best); });
        // sets of two weigh twice the lightest rank at least
        lone = lane + 1 > ORBG_LOW_RANKS ? vr[0] : CAP;
#pragma unroll
        for (int j = 1; j < NK; ++j) lone = vr[j] < lone ? vr[j] : lone;
        lone = wave_min_u32(lone);
        // as far as the weights, the ranks and the lists reach
        uint32_t most = CAP < none ? CAP : none;
        most = (far < CAP && far + lone < most ? far + lone : most) - 1u;
        uint32_t last = 0, level = 2u * lone - (lone != 0u ? 1u : 0u), tested = NK, end = 0;
        done = 0;
        bool counted = false;
        if (best.W <= level && best.W <= most) {
            if (best.W < lone) {
                q = count_low(best);
                return q > budget ? 2 : 1;
            }
            level = best.W;
        }
        for (;;) {
            level = level < most ? level : most;
            while (level > last && !prefixes(level, end)) level = last + (level - last) / 2u;
            if (level <= last) return 0;
            last = level;
            each_step(done, end, [&](uint32_t x, uint32_t y) {
                const auto a = L.r[x >> 24], b = L.r[(x >> 16) & 0xffu], c = L.r[(x >> 8) & 0xffu], d = L.r[x & 0xffu];
                S v = xor3<S>(xor3<S>(sv, a.h, b.h), c.h, d.h);
                uint32_t wu = a.v + b.v + c.v + d.v;
                if (ballot(y != 0u) != 0ull) {
                    const auto e = L.r[y >> 24], f = L.r[(y >> 16) & 0xffu], g = L.r[(y >> 8) & 0xffu];
                    v = xor3<S>(v, e.h, f.h) ^ g.h;
                    wu += e.v + f.v + g.v;
                }
                test(v, x, y, wu, best);
                ++tested;
            });
            if (best.W <= level) break;
            // whole steps were taken
            const uint32_t up = done + (end > done ? (end - done + ORBG_WAVE - 1) / ORBG_WAVE * ORBG_WAVE : 0u);
            done = up;
            // out of budget?  (at most 256 patterns per set)
            if ((uint64_t)(tested * ORBG_WAVE + 1u) * 256u > budget) {
                if (!counted) sort_subsets();
                counted = true;
                if (count(level + 1u, end, false, best) >= budget) return 2;
            }
            const uint32_t next = level + level / 4u + 1u;
            level = next < best.W ? next : best.W;        // (above the last: the search ends at best.W)
        }
        if (!counted) sort_subsets();
        if (!prefixes(best.W, end)) return 0;
        const uint64_t n = count(best.W, end, true, best);
        if (n > budget) return 2;
        q = (uint32_t)n;
        return 1;
    }
};

// One block: ranks, fit, search, outputs.  Returns 0 if the search does not cover
// it (no output but the mark then).
template <int NK, typename S, bool WIDE, class AA, class TT>
__device__ __forceinline__ int mline_match_block(const AA& a, const TT& T, MmLds<NK, S, WIDE>& L,
                                                 const float (&x)[NK], const uint64_t (&hrow)[NK], int64_t b)
{
    constexpr uint32_t CAP = mm_cap<WIDE>();
    const int lane = lane_id();
    const int n = a.n;
    const int h = n / 2;
    bool ybit[NK];
    const S s0 = hard_decision<NK, S>(x, n, hrow, ybit);
    int found = 1;
    uint32_t q = 1;
    MmPattern best = {0u, 0u, 0u, 0u};
    int m_used = 1;
    int32_t j0v = 0;
    if (s0 != 0 || a.mfit != nullptr || a.j0 != nullptr) {
        // ranks, all of them: single ones can be flipped
        uint32_t idx[NK];
        constexpr int RANKS = mm_ranks<NK>();
        rank_order<NK>(x, n, n, 0, idx);
#pragma unroll
        for (int j = 0; j < NK; ++j) L.x[j * ORBG_WAVE + lane] = fabsf(x[j]);
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            const int r = lane * NK + j + 1;
            if (r <= h) L.L[r] = L.x[idx[j]];
            if (r <= n) L.pi[r] = (uint16_t)idx[j];
        }
        wave_lds_sync();
        const MmModel md = fit_lines<NK>(L.L, n, a.mseg, a.jdiv);
        m_used = md.m;
        j0v = md.J[0];
        if (s0 != 0) {
            const uint32_t limit = (n < 32 && a.budget > (1u << n)) ? (1u << n) : a.budget;
            MmSearch<NK, S, WIDE, TT> F{L, T, s0, 0, 0u, limit, {}, {}, 0u, 0u};
            // weight of rank r, cut at the cap (ranks past n weigh that much)
            auto weigh = [&](int r, MmSplit& sp) -> uint32_t {
                int J = md.J[0], B = md.B[0], I = 0, s = 0;
#pragma unroll
                for (int i = 1; i < ORBG_ML_MSEG; ++i) {
                    const bool past = i < md.m && r > md.I[i];
                    J = past ? md.J[i] : J;
                    B = past ? md.B[i] : B;
                    I = past ? md.I[i] : I;
                    s = past ? i : s;
                }
                const uint32_t v = (uint32_t)(J + B * (r - I));   // at most 2^20 + 512 x 2^20
                const uint32_t w = r <= n && v < CAP ? v : CAP;
                const uint32_t f = 1u << (8 * s);
                s = s == md.m - 1 ? 3 : s;                // (the others' weights fix the last segment's)
                if (WIDE) sp = {s == 0 ? w : 0u, s == 1 ? w : 0u, s == 2 ? w : 0u, 0u};
                else sp = {s == 0 ? w << 20 : s == 1 ? w << 10 : s == 2 ? w : 0u, 0u, 0u, 0u};
                sp.f = f;
                return w;
            };
            MmSplit sp[NK] = {};
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                const int r = lane + 1 + j * ORBG_WAVE;
                F.vr[j] = r <= n ? weigh(r, sp[j]) : CAP;
                F.g[j] = r <= n ? (S)a.cols[L.pi[r]] : (S)0;
            }
            F.piv = match_reduce<NK, S>(F.g, L.null, F.nulls, &F.sv);
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                const int r = lane + 1 + j * ORBG_WAVE;
                if (r <= RANKS) {
                    L.r[r] = {F.g[j], F.vr[j]};
                    L.split[r] = put_split<WIDE>(sp[j]);
                } else if (NK >= 4 && r == RANKS + 1) {
                    L.split[r] = put_split<WIDE>(sp[j]);
                }
            }
            if (lane == 0) {
                L.r[0] = {0, 0u};
                L.split[0] = {};
                L.r[RANKS + 1] = {0, CAP};
                if (NK >= 4) L.split[RANKS + 2] = put_split<WIDE>({0u, 0u, 0u, 1u << (8 * (md.m - 1))});
            }
            // subsets of ranks 1..4 (lanes 0..15) and 5..8 (lanes 16..31)
            uint32_t nv = 0;
            MmSplit ns = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool on = ((lane >> k) & 1) != 0;
                const int from = ((lane >> 2) & 4) + k;   // lane of rank k + 1 or k + 5
                auto pick = [&](uint32_t v) -> uint32_t {
                    const uint32_t o = (uint32_t)__shfl((int)v, from, ORBG_WAVE);
                    return on ? o : 0u;
                };
                nv += pick(F.vr[0]);
                ns.a += pick(sp[0].a);
                if (WIDE) {
                    ns.b += pick(sp[0].b);
                    ns.c += pick(sp[0].c);
                }
                ns.f += pick(sp[0].f);
            }
            if (lane < 32) {
                L.nib[lane].v = nv;
                L.nib[lane].split = put_split<WIDE>(ns);
            }
            wave_lds_sync();
            // lightest rank past `top`
            auto lightest_past = [&](int top) -> uint32_t {
                uint32_t least = ~0u;
#pragma unroll
                for (int i = 0; i < ORBG_ML_MSEG; ++i) {
                    const int lo = md.I[i] > top ? md.I[i] + 1 : top + 1;
                    const int hi = i + 1 < md.m ? md.I[i + 1] : n;
                    if (i < md.m && lo <= hi) {
                        const uint32_t v = (uint32_t)(md.J[i] + md.B[i] * (lo - md.I[i]));
                        least = v < least ? v : least;
                    }
                }
                return least;
            };
            const uint32_t far = NK >= 4 && n > RANKS ? lightest_past(RANKS) : ~0u;
            const uint32_t none = NK >= 8 && n > ORBG_MM_SINGLE ? lightest_past(ORBG_MM_SINGLE) : ~0u;
            found = F.run(far, none, best, q);
        }
    }
    if (found == 0) {                                 // left for mline_kernel
        if (lane == 0) a.abandoned[b] = ORBG_OPEN;
    } else {
        uint32_t lo = 0, hi = 0;
        if (found == 1 && q > 1) {
            if (NK >= 4 && (best.x >> 24) > ORBG_MM_RANKS) {  // a single rank past the sets'
                if (lane == 0) L.pi[ORBG_MM_RANKS + 1] = L.pi[ORBG_MM_RANKS + 1 + best.y];
                best.y = 0;
                wave_lds_sync();
            }
            lo = best.mask | ((best.x >> 16) & 0xff00u) | (best.x & 0xff0000u) | (best.x << 16 & 0xff000000u);
            hi = (best.x & 0xffu) | ((best.y >> 16) & 0xff00u) | (best.y & 0xff0000u) | (best.y << 16 & 0xff000000u);
        }
        write_codeword<NK>(ybit, L, lo, hi, make_buf(a.cw + b * (int64_t)n, (uint32_t)n), NoOffs{});
        write_result(a.queries + b, a.abandoned + b, found == 1 ? q : a.budget, found != 1);
        if (lane == 0) {
            if (a.mfit != nullptr) a.mfit[b] = m_used;
            if (a.j0 != nullptr) a.j0[b] = j0v;
        }
    }
    wave_lds_sync();
    return found;
}

template <int NK, typename S>
__global__ void __launch_bounds__(ORBG_WAVE, NK <= 2 ? 4 : 1) mline_match_kernel(MlineArgs a)
{
    __shared__ MmLds<NK, S, false> L;
    const int lane = lane_id();
    const int n = a.n;
    uint64_t hrow[NK];
#pragma unroll
    for (int j = 0; j < NK; ++j) hrow[j] = lane < a.m ? a.rows[lane * NK + j] : 0ull;
    auto fetch = [&](float (&x)[NK], int64_t b) {
        load_row_buf<NK>(make_buf(a.llr + (b < a.nblocks ? b * (int64_t)n : 0), b < a.nblocks ? (uint32_t)n * 4u : 0u), x);
    };
    typedef const __attribute__((address_space(4))) MlineArgs* const_args_ptr;
    const_args_ptr args = (const_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    float x[NK], next[NK];
    int64_t b = blockIdx.x;
    fetch(x, b);
    while (b < a.nblocks) {
        fetch(next, b + gridDim.x);                       // loads while this block is decoded
        // the arguments are read where they are used (scalar loads): kept in
        // registers over the loop they spill, and come back by vector instructions
        asm volatile("" : "+s"(args));
        mline_match_block<NK, S, false>(*args, args->sets, L, x, hrow, b);
        b += gridDim.x;
#pragma unroll
        for (int j = 0; j < NK; ++j) x[j] = next[j];
    }
}

template <int NK>
hipError_t launch_mline_match_nk(const MlineArgs& a, int grid, hipStream_t stream)
{
    if (a.m <= 32) mline_match_kernel<NK, uint32_t><<<grid, ORBG_WAVE, 0, stream>>>(a);
    else mline_match_kernel<NK, uint64_t><<<grid, ORBG_WAVE, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace orbg
