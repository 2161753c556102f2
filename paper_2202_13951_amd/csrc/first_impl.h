// First pass of a large batch for gfx950: query 1 for every block, the first
// batch of 64 patterns for the others; a block that neither decides is marked
// for the match search (match_impl.h).
//
// One wave takes groups of K rows (all K loads in flight together) and works on
// them from registers: base syndrome by row parities; s0 = 0 is query 1 and is
// written out.  For the others a threshold on |LLR| picks the 9 to 16 least
// reliable bits; their keys go to a 16-key slot in LDS.  Four slots are sorted
// at a time, one per row of 16 lanes (10 substeps for four blocks, lane
// exchanges inside DPP rows), and each block's patterns are tested one per
// lane: the ranks a lane's pattern flips are the same for every block, so its
// LDS addresses are made once per kernel and a test is four reads and an XOR.
// With c ranks known, the patterns of logistic weight <= c are tested.
//
// Bound: vector and scalar issue (each wave instruction holds a SIMD for four
// cycles) beside the one read of every row: 49 vector and 44 scalar instructions
// a block.  7 x 10^6 blocks of BCH(127,113), 4 to 7 dB: 1.21 ms, 3.9 TB/s (a
// large copy reaches 4.75); with the match search of the 14 % it leaves 1.97 ms,
// where one pass that ranked and walked block by block took 2.80.
#pragma once
#include "match_impl.h"

namespace orbg {

#define ORBG_FIRST_MIN 9         // fewest ranks a block goes on with
#define ORBG_FIRST_N 12          // shorter codes go to the match search
#define ORBG_FIRST_ROW 20        // ranks 0..16 of a sorted block, padded

// Staged blocks: at most 3 left over and the K (<= 16) of one group; a power of two.
constexpr uint32_t first_slots(int k) { return k <= 4 ? 8u : k <= 8 ? 16u : 32u; }

// Words of a staged block: its hard decision (2 NK), syndrome (2), index and
// (ranks | code << 8), mixed codes also the row's offset (2) and length; one per
// lane of the store, so a power of two.
template <int NK, bool MIXED>
struct FirstWords {
    static constexpr int SYN = 2 * NK, ID = 2 * NK + 2, INFO = 2 * NK + 3, ROW = 2 * NK + 4, LEN = 2 * NK + 6;
    static constexpr int W = NK <= 2 && !MIXED ? 8 : NK <= 4 ? 16 : NK == 8 ? 32 : 64;
};

template <int NK, typename S, bool MIXED, int K>
struct FirstLds {
    static constexpr uint32_t SLOTS = first_slots(K);
    uint32_t key[SLOTS * 16];
    uint32_t word[SLOTS * FirstWords<NK, MIXED>::W + ORBG_WAVE];   // (the last 64: lanes past W)
    S h[4 * ORBG_FIRST_ROW];             // columns by rank of four sorted blocks (rank 0: zero)
    uint32_t pi[4 * ORBG_FIRST_ROW];     // their received indices (rank 0: none)
    uint4 code[MIXED ? ORBG_MAX_CODES : 1];   // mixed codes: n, m | nk << 8, row_base, col_base
};

// Lane l of `reg` <- v (both wave-uniform).  (clang has no builtin for it; the
// name is the intrinsic's.)
__device__ int32_t writelane_i32(int32_t v, int32_t l, int32_t old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ void writelane(uint32_t& reg, uint32_t v, uint32_t l)
{
    reg = (uint32_t)writelane_i32((int32_t)v, (int32_t)l, (int32_t)reg);
}

// K: rows per group (at most 16).
template <int NK, typename S, bool MIXED, int K>
__global__ void __launch_bounds__(ORBG_WAVE)
first_kernel(CodeTable codes, const uint8_t* __restrict__ block_code, const int64_t* __restrict__ row_off,
             const float* __restrict__ llr, int64_t nblocks, uint32_t budget, uint8_t* __restrict__ cw,
             uint64_t* __restrict__ queries, uint8_t* __restrict__ abandoned, int64_t row_limit)
{
    extern __shared__ __align__(16) unsigned char orbg_dyn_lds[];
    uint64_t* s_rows = reinterpret_cast<uint64_t*>(orbg_dyn_lds);
    S* s_cols = reinterpret_cast<S*>(orbg_dyn_lds + (size_t)codes.rwords * sizeof(uint64_t));
    __shared__ FirstLds<NK, S, MIXED, K> L;
    constexpr uint32_t SLOTS = first_slots(K);
    constexpr int IB = IndexBits<NK>::value;
    constexpr bool HOIST = !MIXED && NK <= 4;
    const int lane = lane_id();
    for (int ci = 0; ci < (MIXED ? codes.ncodes : 1); ++ci) {
        const CodeDesc& c = codes.c[ci];
        for (int i = threadIdx.x; i < c.n; i += ORBG_WAVE) s_cols[c.col_base + i] = (S)c.cols[i];
        for (int i = threadIdx.x; i < c.m * c.nk; i += ORBG_WAVE) s_rows[c.row_base + i] = c.rows[i];
        if (MIXED && lane == 0) L.code[ci] = make_uint4((uint32_t)c.n, (uint32_t)(c.m | c.nk << 8), c.row_base, c.col_base);
    }
    if (lane < 4) {
        L.h[lane * ORBG_FIRST_ROW] = 0;
        L.pi[lane * ORBG_FIRST_ROW] = ~0u;
    }
    // this lane's pattern of the first batch (at most four ranks), its weight
    uint32_t a[4] = {0, 0, 0, 0}, wpat = 0;
    {
        // (the same for every length from 12 up: the batch reaches rank 12)
        int cp = 0;
        while (MIXED && cp + 1 < codes.ncodes && codes.c[cp].n < ORBG_FIRST_N) ++cp;
        const uint2 e = load_entry(codes.c[cp].sched, (uint32_t)lane);
        uint32_t m = e.x & 0xffu, high = e.x >> 8;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t r = m != 0 ? (uint32_t)__builtin_ctz(m) + 1u : (high & 0xffu);
            high = m != 0 ? high : high >> 8;
            m &= m - 1;
            a[k] = r;
            wpat += r;
        }
    }
    wave_lds_sync();
    uint64_t hrow0[NK];
    if (HOIST) load_hrows<NK>(s_rows, codes.c[0].m, hrow0);
    LaneOffs<NK> lo = lane_offsets<NK>(MIXED ? NK * ORBG_WAVE : codes.c[0].n);

    using Q = FirstWords<NK, MIXED>;
    // this lane's word of slot 0; lanes past W write beside the slots
    uint32_t* const my_word = &L.word[lane < Q::W ? lane : SLOTS * Q::W + lane];
    const uint32_t word_step = lane < Q::W ? Q::W : 0u;
    // one code: codewords, query counts and flags of all blocks (the host keeps
    // the batch's codewords within ORBG_PAST bytes); a block is a scalar offset
    const uint32_t n0 = (uint32_t)codes.c[0].n;
    const buf_t cw_all = make_buf(cw, MIXED ? 0u : (uint32_t)nblocks * n0);
    const buf_t q_all = make_buf(queries, MIXED ? 0u : (uint32_t)nblocks * 8u);
    const buf_t ab_all = make_buf(abandoned, MIXED ? 0u : (uint32_t)nblocks);
    uint32_t head = 0, staged = 0;
    float tau = 2.0f;                                     // threshold, carried from block to block

    // codeword y, query count and flag of block b
    // (mixed codes: its row's offset, or -1, and length)
    auto write = [&](uint32_t b, int64_t row, uint32_t n, const uint64_t (&y)[NK], uint32_t q) {
        const u32x2_t qv = {q, 0u};
        if constexpr (!MIXED) {
#pragma unroll
            for (int j = 0; j < NK; ++j)
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(__builtin_amdgcn_inverse_ballot_w64(y[j]) ? 1 : 0), cw_all,
                                                     lo.c[j], b * n0, 0);
            __builtin_amdgcn_raw_buffer_store_b64(qv, q_all, lo.r, b * 8u, 0);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)0, ab_all, lo.r, b, 0);
        } else {
            const buf_t cb = make_buf(cw + (row >= 0 ? row : 0), row >= 0 ? n : 0u);
#pragma unroll
            for (int j = 0; j < NK; ++j)
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(__builtin_amdgcn_inverse_ballot_w64(y[j]) ? 1 : 0), cb,
                                                     lo.c[j], 0, 0);
            write_result(queries + b, abandoned + b, q, false, lo.r);
        }
    };
    auto mark = [&](uint32_t b) {
        if constexpr (!MIXED) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)ORBG_OPEN, ab_all, lo.r, b, 0);
        else __builtin_amdgcn_raw_buffer_store_b8((uint8_t)ORBG_OPEN, make_buf(abandoned + b, 1), lo.r, 0, 0);
    };

    // Sorts the `cnt` (1..4) oldest staged blocks and tests their patterns.
    auto flush = [&](uint32_t cnt) {
        const uint32_t sub = (uint32_t)lane >> 4, in = (uint32_t)lane & 15u;
        const uint32_t slot = (head + sub) & (SLOTS - 1);
        wave_lds_sync();
        const uint32_t mt = L.word[slot * Q::W + Q::INFO];
        uint32_t words[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            words[j] = L.word[((head + (uint32_t)j) & (SLOTS - 1)) * Q::W + ((uint32_t)lane & (Q::W - 1))];
        const uint32_t known = sub < cnt ? mt & 0xffu : 0u;
        uint32_t k1[1] = {in < known ? L.key[slot * 16u + in] : 0xffffffffu};
        sort32<1, 16>(k1);
        const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)k1[0], 0x101, 0xF, 0xF, false);   // row_shl:1
        uint64_t ties = ballot(in + 1u < known && ((k1[0] ^ next) >> IB) == 0u);
        if (ties != 0ull) {
            // rows on a coarse grid are ranked by their keys all the same (read again:
            // ties are rare, or all rows are coarse).  3 x 10^5 blocks of LLRs rounded
            // to whole numbers, us, before the passes / left to the search / so: n = 32
            // 140 / 133 / 45, n = 127 240 / 256 / 101.
#pragma unroll 1
            for (uint32_t j = 0; j < cnt; ++j) {
                if (((ties >> (16u * j)) & 0xffffull) == 0ull) continue;
                const uint32_t* w = L.word + ((head + j) & (SLOTS - 1)) * Q::W;
                const uint32_t n = MIXED ? uniform_u32(w[Q::LEN]) : n0;
                int64_t row = MIXED ? uniform_i64((int64_t)(((uint64_t)w[Q::ROW + 1] << 32) | w[Q::ROW]))
                                    : (int64_t)uniform_u32(w[Q::ID]) * n0;
                float xt[NK];
                load_row_buf<NK>(make_buf(llr + (row >= 0 ? row : 0), row >= 0 ? n * 4u : 0u), xt, lo);
                if (coarse_row<NK>(xt)) ties &= ~(0xffffull << (16u * j));
            }
        }
        const uint32_t idx = k1[0] & ((1u << IB) - 1u);
        const uint32_t cb = MIXED ? (sub < cnt ? L.code[mt >> 8].w : 0u) : 0u;
        const S col = s_cols[in < known ? cb + idx : 0u];
        L.h[sub * ORBG_FIRST_ROW + 1 + in] = in < known ? col : (S)0;
        L.pi[sub * ORBG_FIRST_ROW + 1 + in] = in < known ? idx : ~0u;
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if ((uint32_t)j >= cnt) break;
            auto get = [&](int k) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)words[j], k); };
            const uint32_t info = get(Q::INFO);
            const S s0 = sizeof(S) == 4 ? (S)get(Q::SYN) : (S)(((uint64_t)get(Q::SYN + 1) << 32) | get(Q::SYN));
            const uint32_t b = get(Q::ID);
            const S* h = L.h + j * ORBG_FIRST_ROW;
            const S v = xor3<S>(xor3<S>(s0, h[a[0]], h[a[1]]), h[a[2]], h[a[3]]);
            const uint64_t hits = ballot(v == 0 && wpat <= (info & 0xffu));
            const uint32_t wl = hits != 0 ? (uint32_t)__builtin_ctzll(hits) : 0u;
            if (hits != 0 && ((ties >> (16 * j)) & 0xffffull) == 0ull && wl < budget) {
                uint64_t y[NK];
#pragma unroll
                for (int k = 0; k < NK; ++k) y[k] = ((uint64_t)get(2 * k + 1) << 32) | get(2 * k);
                // flips as lane masks (compares are vector work: the scalar unit is
                // the busier one)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t p =
                        (uint32_t)__builtin_amdgcn_readlane((int)L.pi[j * ORBG_FIRST_ROW + a[u]], (int)wl);
#pragma unroll
                    for (int k = 0; k < NK; ++k) y[k] ^= ballot((uint32_t)(k * ORBG_WAVE + lane) == p);
                }
                if constexpr (MIXED)
                    write(b, (int64_t)(((uint64_t)get(Q::ROW + 1) << 32) | get(Q::ROW)), get(Q::LEN), y, wl + 1u);
                else
                    write(b, 0, 0u, y, wl + 1u);
            } else {
                mark(b);
            }
        }
        wave_lds_sync();
        head = (head + cnt) & (SLOTS - 1);
        staged -= cnt;
    };

    const int64_t step = (int64_t)gridDim.x * K;
    // mixed codes: lane l loads the code and row offset of the group's block l, one
    // group early (scalar loads, three round trips in a row for each block, took
    // three codes' 10^6 blocks from 901 to 991 us a decode)
    uint32_t code_in = 0;
    int64_t row_in = -1;
    auto ahead = [&](int64_t g) {
        const bool in = MIXED && lane < K && g + lane < nblocks;
        code_in = in ? block_code[g + lane] : 0u;
        row_in = in ? row_off[g + lane] : -1;
    };
    if (MIXED) ahead((int64_t)blockIdx.x * K);
    for (int64_t g = (int64_t)blockIdx.x * K; g < nblocks; g += step) {
        float xs[K][NK];
        uint4 code = {0u, 0u, 0u, 0u};                    // lane l: block l's
        uint32_t code_id = 0;
        int64_t row_id = -1;
        auto of = [&](uint32_t v, int kk) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)v, kk); };
        auto row_at = [&](int kk) -> int64_t {
            return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)row_id >> 32), kk) << 32) | of((uint32_t)row_id, kk));
        };
        const uint32_t cnt = uniform_u32((uint32_t)(nblocks - g < K ? nblocks - g : K));
        if constexpr (!MIXED) {
            // the group's rows lie back to back: one descriptor, a scalar offset per row
            const uint32_t n4 = (uint32_t)codes.c[0].n * 4u;
            const buf_t lb = make_buf(llr + g * codes.c[0].n, cnt * n4);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) load_row_buf<NK>(lb, xs[kk], lo, (uint32_t)kk < cnt ? (uint32_t)kk * n4 : 0u);
        } else {
            code_id = code_in < (uint32_t)codes.ncodes ? code_in : 0u;   // out-of-range indices read code 0
            code = L.code[code_id];
            row_id = row_in >= 0 && row_in <= row_limit - (int64_t)code.x ? row_in : -1;
            ahead(g + step);
#pragma unroll
            for (int kk = 0; kk < K; ++kk) {
                const int64_t row = row_at(kk);
                load_row_buf<NK>(make_buf(llr + (row >= 0 ? row : 0), row >= 0 ? of(code.x, kk) * 4u : 0u), xs[kk], lo);
            }
        }
        int64_t g2 = g;
        uint32_t cnt2 = cnt;
        asm volatile("" : "+s"(g2), "+s"(cnt2));          // (row values are made again after the loads)
#pragma unroll
        for (int kk = 0; kk < K; ++kk) {
            if ((uint32_t)kk >= cnt2) break;
            const uint32_t n = MIXED ? of(code.x, kk) : (uint32_t)codes.c[0].n;
            uint64_t hr[NK];
            if (HOIST) {
#pragma unroll
                for (int j = 0; j < NK; ++j) hr[j] = hrow0[j];
            } else {
                const uint32_t mk = MIXED ? of(code.y, kk) : (uint32_t)(codes.c[0].m | codes.c[0].nk << 8);
                load_hrows_pad<NK>(s_rows + (MIXED ? of(code.z, kk) : 0u), (int)(mk & 0xffu), (int)(mk >> 8), hr);
            }
            bool yb[NK];
            const S s0 = hard_decision<NK, S>(xs[kk], (int)n, hr, yb);
            uint64_t y[NK];
#pragma unroll
            for (int j = 0; j < NK; ++j) y[j] = ballot(yb[j]);
            if (s0 == 0) {
                write((uint32_t)g2 + kk, MIXED ? row_at(kk) : 0, n, y, 1u);
                continue;
            }
            // threshold: 9 to 16 magnitudes below it, by steps of a quarter and
            // then by halves
            uint32_t below = 0;
            uint64_t mk[NK];
            auto pick = [&]() {
                below = 0;
#pragma unroll
                for (int j = 0; j < NK; ++j) {
                    // lanes past n read 0 and are no candidates
                    mk[j] = ballot(fabsf(xs[kk][j]) < tau) &
                            ((int)n >= (j + 1) * ORBG_WAVE ? ~0ull : (int)n <= j * ORBG_WAVE ? 0ull
                                                                                     : (1ull << (n & 63u)) - 1ull);
                    below += (uint32_t)__builtin_popcountll(mk[j]);
                }
            };
            float lo_t = 0.0f, hi_t = 0.0f;               // bracket (0: open)
#pragma unroll 1
            for (int it = 0; it < 8; ++it) {
                pick();
                if (below >= ORBG_FIRST_MIN && below <= 16u) break;
                const bool up = below < ORBG_FIRST_MIN;
                lo_t = up ? tau : lo_t;
                hi_t = up ? hi_t : tau;
                const float open = tau * (up ? 1.25f : 0.8f);
                const float mid = 0.5f * (lo_t + hi_t);
                tau = __uint_as_float(uniform_u32(__float_as_uint(lo_t == 0.0f || hi_t == 0.0f ? open : mid)));
            }
            if (below < ORBG_FIRST_MIN || below > 16u || n < ORBG_FIRST_N) {
                tau = tau > 0.0f && tau < INFINITY ? tau : 2.0f;   // (rows of zeros or infinities)
                mark((uint32_t)g2 + kk);
                continue;
            }
            const uint32_t slot = (head + staged) & (SLOTS - 1);
            uint32_t at = slot * 16u;
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                const uint32_t i = (uint32_t)(j * ORBG_WAVE + lane);
                // truncated magnitude above the index, as in rank_order
                const uint32_t key = ((__float_as_uint(xs[kk][j]) & 0x7fffffffu) >> (IB - 1)) << IB | i;
                const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk[j] >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)mk[j], at));
                if (__builtin_amdgcn_inverse_ballot_w64(mk[j])) L.key[to] = key;
                at += (uint32_t)__builtin_popcountll(mk[j]);
            }
            uint32_t wv = 0;
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                writelane(wv, (uint32_t)y[j], 2 * j);
                writelane(wv, (uint32_t)(y[j] >> 32), 2 * j + 1);
            }
            writelane(wv, (uint32_t)s0, Q::SYN);
            if (sizeof(S) == 8) writelane(wv, (uint32_t)((uint64_t)s0 >> 32), Q::SYN + 1);
            writelane(wv, (uint32_t)g2 + kk, Q::ID);
            writelane(wv, below | (MIXED ? of(code_id, kk) << 8 : 0u), Q::INFO);
            if (MIXED) {
                const int64_t row = row_at(kk);
                writelane(wv, (uint32_t)row, Q::ROW);
                writelane(wv, (uint32_t)((uint64_t)row >> 32), Q::ROW + 1);
                writelane(wv, n, Q::LEN);
            }
            my_word[slot * word_step] = wv;
            ++staged;
        }
        while (staged >= 4u) flush(4u);
    }
    if (staged != 0) flush(staged);
}

template <int NK, typename S, bool MIXED>
static hipError_t launch_first_as(const DecodeArgs& a, hipStream_t stream)
{
    uint32_t ncols = 0;
    for (int i = 0; i < (MIXED ? a.codes.ncodes : 1); ++i) {
        const uint32_t e = a.codes.c[i].col_base + (uint32_t)a.codes.c[i].n;
        ncols = e > ncols ? e : ncols;
    }
    const size_t lds = (size_t)a.codes.rwords * sizeof(uint64_t) + ncols * sizeof(S);
    // small batches: short groups, so that more waves share the rows
    constexpr int KS = ScreenDepth<NK>::value < 4 ? ScreenDepth<NK>::value : 4;
    const int64_t most = (int64_t)a.cus * 32;
    auto go = [&](auto kernel, int k) {
        const int64_t units = (a.nblocks + k - 1) / k;
        kernel<<<(unsigned)(units < most ? units : most), ORBG_WAVE, lds, stream>>>(
            a.codes, a.block_code, a.row_off, a.llr, a.nblocks, a.budget, a.cw, a.queries, a.abandoned, a.row_limit);
        return hipGetLastError();
    };
    if (a.nblocks < most * ScreenDepth<NK>::value) return go(first_kernel<NK, S, MIXED, KS>, KS);
    return go(first_kernel<NK, S, MIXED, ScreenDepth<NK>::value>, ScreenDepth<NK>::value);
}

template <int NK>
hipError_t launch_first_nk(const DecodeArgs& a, bool s32, hipStream_t stream)
{
    if (a.mixed) {
        if constexpr (NK <= 4)
            return s32 ? launch_first_as<NK, uint32_t, true>(a, stream) : launch_first_as<NK, uint64_t, true>(a, stream);
        return hipErrorInvalidValue;                      // mixed launches take n <= 256
    }
    return s32 ? launch_first_as<NK, uint32_t, false>(a, stream) : launch_first_as<NK, uint64_t, false>(a, stream);
}

}  // namespace orbg
