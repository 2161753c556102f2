// Device-side helpers shared by the ORBGRAND kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define ORBG_WAVE 64
#define ORBG_RANK_SLOTS 256   // LDS slots per wave for permuted columns: rank 0 is the zero column
#define ORBG_ENTRY_RANKS 16   // ranks held by one 16-byte schedule entry (u8 each, 0 = unused)

namespace orbg {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Orders this wave's LDS traffic: every lane's earlier LDS writes are visible to
// every lane's later LDS reads (waits for the LDS queue, keeps the compiler
// from moving accesses across).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// XOR of one 32-bit value over the 16 lanes of each DPP row (every lane of the
// row receives it): quad swaps, half-row mirror, row mirror.  All lanes active.
__device__ __forceinline__ uint32_t row_xor16(uint32_t v)
{
    v ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    v ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    v ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    v ^= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    return v;
}

// XOR of a u64 over the whole wave, returned wave-uniform.  All lanes active.
__device__ __forceinline__ uint64_t wave_xor_reduce(uint64_t v)
{
    const uint32_t lo = row_xor16((uint32_t)v), hi = row_xor16((uint32_t)(v >> 32));
    const uint32_t l = __builtin_amdgcn_readlane(lo, 0) ^ __builtin_amdgcn_readlane(lo, 16) ^
                       __builtin_amdgcn_readlane(lo, 32) ^ __builtin_amdgcn_readlane(lo, 48);
    const uint32_t h = __builtin_amdgcn_readlane(hi, 0) ^ __builtin_amdgcn_readlane(hi, 16) ^
                       __builtin_amdgcn_readlane(hi, 32) ^ __builtin_amdgcn_readlane(hi, 48);
    return ((uint64_t)h << 32) | l;
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Ascending bitonic sort of 64*NK u64 keys held NK per lane.  Element e lives
// in lane e / NK, register e % NK, so distances below NK are exchanged inside a
// lane and larger ones across lanes (lane distance d / NK).  Keys must be
// distinct except for padding.  A compare-exchange is one 64-bit compare, a
// lane-mask XOR with the stage's direction and two selects.
template <int NK, typename KEY = uint64_t>
__device__ __forceinline__ void bitonic_sort(KEY (&key)[NK])
{
    // the direction masks are made where they are used: hoisted out of a block
    // loop they take 2 scalar registers each and spill
    int lane = lane_id();
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int size = 2; size <= ORBG_WAVE * NK; size <<= 1) {
#pragma unroll
        for (int d = size >> 1; d > 0; d >>= 1) {
            if (d < NK) {
#pragma unroll
                for (int j = 0; j < NK; ++j) {
                    if ((j & d) == 0) {
                        // ascending iff bit `size` of e = lane * NK + j is clear
                        const bool desc = ((lane * NK + j) & size) != 0;
                        const KEY a = key[j], b = key[j | d];
                        const bool sw = (a > b) != desc;
                        key[j] = sw ? b : a;
                        key[j | d] = sw ? a : b;
                    }
                }
            } else {
                const int ld = d / NK;
                // the lower lane of a pair keeps the minimum in ascending runs
                const bool keep_min = ((lane & ld) == 0) == (((lane * NK) & size) == 0);
#pragma unroll
                for (int j = 0; j < NK; ++j) {
                    const KEY p = __shfl_xor(key[j], ld, ORBG_WAVE);
                    const bool take_p = (p < key[j]) == keep_min;
                    key[j] = take_p ? p : key[j];
                }
            }
        }
    }
}

// Value of lane (lane XOR LD) for a wave-constant distance LD, all lanes active:
// quad permutes for 1 and 2, a half-row mirror composed with a quad reversal for
// 4 (7 - (i ^ 3) = i ^ 4 inside each group of 8), a half-row rotation for 8.
template <int LD>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    static_assert(LD == 1 || LD == 2 || LD == 4 || LD == 8, "lane distance");
    if constexpr (LD == 1) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    } else if constexpr (LD == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    } else if constexpr (LD == 4) {
        const int m = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);     // row_half_mirror
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, false);        // quad_perm [3,2,1,0]
    } else {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false);  // row_ror:8
    }
}

// Value of lane (lane XOR M), all lanes active.
template <int M>
__device__ __forceinline__ uint32_t lane_xor_mask(uint32_t v)
{
    if constexpr (M == 3) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x1B, 0xF, 0xF, false);     // quad_perm [3,2,1,0]
    else if constexpr (M == 7) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    else if constexpr (M == 15) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    else return lane_xor<M>(v);
}

// Per-lane bit of a constant lane mask.  The two scalar moves are written out
// so that the constant is made where it is used: the compiler would otherwise
// hoist it out of the block loop, spill it and reload it with vector
// instructions.
template <uint64_t M>
__device__ __forceinline__ bool lane_bit()
{
    uint32_t lo, hi;
    asm volatile("s_mov_b32 %0, %2\n\ts_mov_b32 %1, %3"
                 : "=s"(lo), "=s"(hi)
                 : "i"((int32_t)(uint32_t)M), "i"((int32_t)(uint32_t)(M >> 32)));
    return __builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo);
}

// All ones in the lanes whose bit BIT is set, zero in the others.
template <int BIT>
__device__ __forceinline__ uint32_t lane_fill()
{
    return (uint32_t)((int32_t)((uint32_t)lane_id() << (31 - BIT)) >> 31);
}

// Median of three: with c = 0 the smaller, with c = ~0 the larger of a and b
// (one instruction, so a lane's side of an exchange is an operand, not a select).
__device__ __forceinline__ uint32_t med3(uint32_t a, uint32_t b, uint32_t c)
{
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    const uint32_t m = hi < c ? hi : c;
    return lo < m ? m : lo;
}

constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }

// Substeps D, D / 2, ..., 1, the smaller key to the lower index.
template <int NK, int D>
__device__ __forceinline__ void sort_halves(uint32_t (&key)[NK])
{
    if constexpr (D >= NK) {
        constexpr int LD = D / NK;
        const uint32_t up = lane_fill<log2_of(LD)>();
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            if constexpr (LD == 16) {
                const auto r = __builtin_amdgcn_permlane16_swap(key[j], key[j], false, false);
                key[j] = med3(r[0], r[1], up);
            } else if constexpr (LD == 32) {
                const auto r = __builtin_amdgcn_permlane32_swap(key[j], key[j], false, false);
                key[j] = med3(r[0], r[1], up);
            } else {
                key[j] = med3(lane_xor<LD>(key[j]), key[j], up);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < NK; ++j)
            if ((j & D) == 0) {
                const uint32_t a = key[j], b = key[j | D];
                key[j] = a < b ? a : b;
                key[j | D] = a < b ? b : a;
            }
    }
    if constexpr (D > 1) sort_halves<NK, D / 2>(key);
}

// Stages SIZE .. MAX (up to one row of 16 lanes) with mirrored first substeps.
template <int NK, int SIZE, int MAX>
__device__ __forceinline__ void sort_stages(uint32_t (&key)[NK])
{
    if constexpr (SIZE <= NK) {
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            const int o = j ^ (SIZE - 1);
            if (j < o) {
                const uint32_t a = key[j], b = key[o];
                key[j] = a < b ? a : b;
                key[o] = a < b ? b : a;
            }
        }
    } else {
        constexpr int M = SIZE / NK - 1;                  // 1, 3, 7 or 15
        const uint32_t up = lane_fill<log2_of(M + 1) - 1>();
        uint32_t p[NK];
#pragma unroll
        for (int j = 0; j < NK; ++j) p[j] = lane_xor_mask<M>(key[NK - 1 - j]);
#pragma unroll
        for (int j = 0; j < NK; ++j) key[j] = med3(p[j], key[j], up);
    }
    if constexpr (SIZE > 2) sort_halves<NK, SIZE / 4>(key);
    if constexpr (SIZE < MAX) sort_stages<NK, SIZE * 2, MAX>(key);
}

// Ascending sort of every GROUP (16, 32 or 64) lanes' GROUP * NK u32 keys,
// element e = lane * NK + j in register j of its lane.  Bitonic network in
// which every exchange puts the smaller key at the lower index: mirrored first
// substeps inside a row of 16 lanes, keys complemented in the rows (halves)
// that have to run down for the stages over 32 and 64 lanes.  Across lanes an
// exchange is a lane move and a median with the lane's side (distances 16 and
// 32 by row and half swaps: no LDS traffic), inside a lane a minimum and a
// maximum: 51 vector instructions for 64 keys, where compares with scalar
// direction masks and selects took 78 and 63 scalar ones.
template <int NK, int GROUP = ORBG_WAVE>
__device__ __forceinline__ void sort32(uint32_t (&key)[NK])
{
    static_assert(GROUP == 16 || GROUP == 32 || GROUP == 64, "lanes of a group");
    const uint32_t c16 = lane_fill<4>(), c32 = lane_fill<5>();
    if constexpr (GROUP > 16) {
#pragma unroll
        for (int j = 0; j < NK; ++j) key[j] ^= c16;
    }
    sort_stages<NK, 2, 16 * NK>(key);
    if constexpr (GROUP > 16) {
#pragma unroll
        for (int j = 0; j < NK; ++j) key[j] ^= GROUP == 64 ? c16 ^ c32 : c16;
        sort_halves<NK, 16 * NK>(key);
    }
    if constexpr (GROUP == 64) {
#pragma unroll
        for (int j = 0; j < NK; ++j) key[j] ^= c32;
        sort_halves<NK, 32 * NK>(key);
    }
}

// Ascending sorts of several short sequences at once: groups of LG consecutive
// lanes (8 or 16) hold one sequence of LG R keys each, element e of it in
// register e % R of its lane e / R.  Bitonic network with mirrored first
// substeps, so every compare-exchange puts the smaller key at the lower index:
// inside a lane it is a minimum and a maximum without a select.  OP: MIN and MAX
// of two registers (32-bit keys, or two independent 16-bit keys per register).
struct KeyU32 {
    static __device__ __forceinline__ uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
    static __device__ __forceinline__ uint32_t max(uint32_t a, uint32_t b) { return a < b ? b : a; }
};
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
struct KeyPairU16 {
    static __device__ __forceinline__ uint32_t min(uint32_t a, uint32_t b)
    {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a),
                                                                      __builtin_bit_cast(u16x2_t, b)));
    }
    static __device__ __forceinline__ uint32_t max(uint32_t a, uint32_t b)
    {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a),
                                                                      __builtin_bit_cast(u16x2_t, b)));
    }
};

// Lanes that hold the lower index of an exchange over lane mask M.
template <int M>
constexpr uint64_t lower_lanes()
{
    const int top = M >= 8 ? 8 : M >= 4 ? 4 : M >= 2 ? 2 : 1;
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l)
        if ((l & top) == 0) m |= 1ull << l;
    return m;
}

template <class OP, int R, int D>
__device__ __forceinline__ void group_halves(uint32_t (&k)[R])
{
    if constexpr (D >= R) {
        constexpr int M = D / R;
        const bool low = lane_bit<lower_lanes<M>()>();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t p = lane_xor_mask<M>(k[j]);
            const uint32_t a = OP::min(p, k[j]), b = OP::max(p, k[j]);
            k[j] = low ? a : b;
        }
    } else {
#pragma unroll
        for (int j = 0; j < R; ++j)
            if ((j & D) == 0) {
                const uint32_t a = OP::min(k[j], k[j | D]), b = OP::max(k[j], k[j | D]);
                k[j] = a;
                k[j | D] = b;
            }
    }
    if constexpr (D > 1) group_halves<OP, R, D / 2>(k);
}

template <class OP, int LG, int R, int SIZE = 2>
__device__ __forceinline__ void group_sort(uint32_t (&k)[R])
{
    if constexpr (SIZE <= R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int o = j ^ (SIZE - 1);
            if (j < o) {
                const uint32_t a = OP::min(k[j], k[o]), b = OP::max(k[j], k[o]);
                k[j] = a;
                k[o] = b;
            }
        }
    } else {
        constexpr int M = SIZE / R - 1;
        const bool low = lane_bit<lower_lanes<M>()>();
#pragma unroll
        for (int j = 0; j < R / 2; ++j) {
            const uint32_t p = lane_xor_mask<M>(k[R - 1 - j]), q = lane_xor_mask<M>(k[j]);
            const uint32_t a = OP::min(p, k[j]), b = OP::max(p, k[j]);
            const uint32_t c = OP::min(q, k[R - 1 - j]), d = OP::max(q, k[R - 1 - j]);
            k[j] = low ? a : b;
            k[R - 1 - j] = low ? c : d;
        }
    }
    if constexpr (SIZE > 2) group_halves<OP, R, SIZE / 4>(k);
    if constexpr (SIZE < LG * R) group_sort<OP, LG, R, SIZE * 2>(k);
}

}  // namespace orbg
