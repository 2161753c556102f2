// Learned batch-order proposal: a 128 -> 256 -> 256 -> 64 ReLU network in BF16
// with FP32 accumulation on the matrix cores, its backward pass and Adam.
//
// Input of the network: a block's reliabilities |LLR_i| sorted ascending (the
// ordered reliability curve of Sec. III-A), scaled by 1/8 and rounded to BF16.
// Output: 64 logits, one per batch of 64 consecutive patterns of the basic
// ORBGRAND order; the decoder tests batches by decreasing logit
// (orbg_decode_ordered) and falls back to the plain order after them.
//
// Parameters (FP32 masters, flat): W1 [256 x 128], b1 [256], W2 [256 x 256],
// b2 [256], W3 [64 x 256], b3 [64] (output x input, row-major).  The forward
// uses BF16 copies of the weights (same layout); the backward also uses BF16
// transposed copies W1t [128 x 256], W2t [256 x 256], W3t [256 x 64].
//
// Products: gfx950's v_mfma_f32_16x16x32_bf16 tiles.  Weight gradients reduce over
// the batch: partials of row chunks in FP32 and a deterministic reduction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "orbg_device.h"
#include "orbg_mlp.h"

namespace orbg {

typedef short s8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
// (a caller's rows need no more than their elements' alignment)
typedef float f4row __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u2row __attribute__((ext_vector_type(2), aligned(1)));

__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);   // NaN stays NaN
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);                 // nearest, ties to even
}

// Two values at once (the instruction gives the same bits for every input).
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32x2_to_bf16(float a, float b)
{
    const f2v v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2v));
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ---------------------------------------------------------------------------
// Features: sorted |LLR| / 8 in BF16, one wave per block (n = 128).  ids (or
// nullptr): row ids[b] of llr gives feature row b.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) features_kernel(const float* __restrict__ llr, int64_t batch,
                                                       uint16_t* __restrict__ x, const int64_t* __restrict__ ids)
{
    const int lane = lane_id();
    const int64_t b = (int64_t)blockIdx.x * 4 + threadIdx.x / ORBG_WAVE;
    if (b >= batch) return;
    const int64_t src = ids ? ids[b] : b;
    uint32_t key[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) key[j] = __float_as_uint(llr[src * MLP_IN + j * ORBG_WAVE + lane]) & 0x7fffffffu;
    bitonic_sort<2, uint32_t>(key);
#pragma unroll
    for (int j = 0; j < 2; ++j) x[b * MLP_IN + lane * 2 + j] = f32_to_bf16(__uint_as_float(key[j]) * 0.125f);
}

// BF16 copies (and transposed copies of the weight matrices) of FP32 masters.
__device__ __forceinline__ void write_copies(int64_t p, float w, uint16_t* __restrict__ wb, uint16_t* __restrict__ wt)
{
    const uint16_t h = f32_to_bf16(w);
    wb[p] = h;
    if (p < MLP_OFF_B1) {                                           // W1 [256 x 128]
        const int64_t rr = p / MLP_IN, cc = p % MLP_IN;
        wt[MLP_T_W1 + cc * MLP_HID + rr] = h;
    } else if (p >= MLP_OFF_W2 && p < MLP_OFF_B2) {                 // W2 [256 x 256]
        const int64_t qq = p - MLP_OFF_W2, rr = qq / MLP_HID, cc = qq % MLP_HID;
        wt[MLP_T_W2 + cc * MLP_HID + rr] = h;
    } else if (p >= MLP_OFF_W3 && p < MLP_OFF_B3) {                 // W3 [64 x 256]
        const int64_t qq = p - MLP_OFF_W3, rr = qq / MLP_HID, cc = qq % MLP_HID;
        wt[MLP_T_W3 + cc * MLP_OUT + rr] = h;
    }
}

__global__ void prepare_kernel(const float* __restrict__ w, uint16_t* __restrict__ wb, uint16_t* __restrict__ wt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < MLP_NPARAM) write_copies(p, w[p], wb, wt);
}

__global__ void adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, float lr, float beta1, float beta2, float eps, float c1,
                            float c2, uint16_t* __restrict__ wb, uint16_t* __restrict__ wt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    const float gg = g[p];
    const float mm = beta1 * m[p] + (1.f - beta1) * gg;
    const float vv = beta2 * v[p] + (1.f - beta2) * gg * gg;
    m[p] = mm;
    v[p] = vv;
    const float ww = w[p] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    w[p] = ww;
    write_copies(p, ww, wb, wt);
}

// Order-preserving bits of a logit (increasing with f, -0 as +0, NaN lowest).
__device__ __forceinline__ uint32_t order_bits(float logit)
{
    const float f = logit + 0.0f;                               // -0 -> +0
    const uint32_t u = __float_as_uint(f);
    const bool nan = (u & 0x7fffffffu) > 0x7f800000u;
    return nan ? 0u : ((u >> 31) ? ~u : (u | 0x80000000u));
}

// One row's batch order (one logit per lane, all lanes active): lane e
// returns the e-th batch to test.
__device__ __forceinline__ uint8_t order_of_row(float logit, int pin0)
{
    const int lane = lane_id();
    uint64_t key[1] = {((uint64_t)(~order_bits(logit)) << 32) | (uint32_t)lane};   // ascending = decreasing f
    if (pin0 && lane == 0) key[0] = 0ull;
    bitonic_sort<1, uint64_t>(key);
    return (uint8_t)(key[0] & 63u);
}

// Eight rows' batch orders (lg: their logits, row stride MLP_OUT), eight lanes a
// row: 32-bit keys of the top 26 order bits above the batch index; a row in
// which two neighbours share those bits is sorted by its full keys.  About 45
// instructions a row (one key per lane and 64-bit keys: 170).  Rows past
// `rows` are not written.
__device__ __forceinline__ void order_of_rows(const float* lg, int rows, int pin0, uint8_t* __restrict__ out)
{
    const int lane = lane_id(), row = lane >> 3, sub = lane & 7;
    uint32_t k[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float4 v = *reinterpret_cast<const float4*>(lg + row * MLP_OUT + sub * 8 + h * 4);
        const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            k[h * 4 + t] = (~order_bits(f[t]) & ~63u) | (uint32_t)(sub * 8 + h * 4 + t);
    }
    if (pin0 && sub == 0) k[0] = 0u;                            // before every key (no logit's order bits are all set)
    group_sort<KeyU32, 8, 8>(k);
    uint32_t same = 0;
#pragma unroll
    for (int j = 0; j + 1 < 8; ++j) same |= ((k[j] ^ k[j + 1]) >> 6) == 0u ? 1u : 0u;
    const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)k[0], 0x101, 0xF, 0xF, false);   // row_shl:1
    same |= sub < 7 && ((k[7] ^ next) >> 6) == 0u ? 1u : 0u;
    uint64_t ties = ballot(same != 0u);
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        lo |= (k[j] & 63u) << (8 * j);
        hi |= (k[4 + j] & 63u) << (8 * j);
    }
    if (row < rows) *reinterpret_cast<u2row*>(out + row * MLP_OUT + sub * 8) = (u2row){lo, hi};
    if (ties == 0ull) return;
    // (each such row's store follows the one above in program order, both made by this wave)
    __builtin_amdgcn_s_waitcnt(0);
    for (int r = 0; r < 8; ++r) {
        if (((ties >> (8 * r)) & 0xffull) == 0ull || r >= rows) continue;
        const uint8_t o = order_of_row(lg[r * MLP_OUT + lane], pin0);
        out[r * MLP_OUT + lane] = o;
    }
}

// Batch order: decreasing logit, ties (and +-0) to the lower index, NaN last;
// pin0: batch 0 first whatever its logit, the others as before.  One wave per
// row: key = (order-preserving bits of -logit) << 32 | index, sorted ascending
// by the register bitonic network; lane e then holds the e-th batch to test.
__global__ void __launch_bounds__(256) order_kernel(const float* __restrict__ logits, int64_t batch,
                                                    uint8_t* __restrict__ order, int pin0)
{
    const int lane = lane_id();
    const int64_t b = (int64_t)blockIdx.x * 4 + threadIdx.x / ORBG_WAVE;
    if (b >= batch) return;
    order[b * MLP_OUT + lane] = order_of_row(logits[b * MLP_OUT + lane], pin0);
}

// Order table of a gated decode: row b = identity for blocks decided by batch 0,
// the learned order for listed blocks (row ids[i] = rows[i]).
__global__ void order_identity_kernel(uint8_t* __restrict__ order, int64_t batch)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < batch * MLP_OUT) order[e] = (uint8_t)(e % MLP_OUT);
}

__global__ void order_scatter_kernel(const uint8_t* __restrict__ rows, const int64_t* __restrict__ ids, int64_t count,
                                     uint8_t* __restrict__ order)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < count * MLP_OUT) order[ids[e / MLP_OUT] * MLP_OUT + e % MLP_OUT] = rows[e];
}

hipError_t mlp_order_table(const uint8_t* rows, const int64_t* ids, int64_t count, int64_t batch, uint8_t* order,
                           hipStream_t st)
{
    if (batch > 0)
        order_identity_kernel<<<(unsigned)((batch * MLP_OUT + 255) / 256), 256, 0, st>>>(order, batch);
    if (count > 0)
        order_scatter_kernel<<<(unsigned)((count * MLP_OUT + 255) / 256), 256, 0, st>>>(rows, ids, count, order);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused inference: (features,) the three layers and (the batch order) of
// FT = 32 rows per 256-thread workgroup.  The rows' features and hidden
// activations stay in LDS as BF16 [row][k], the 16-byte groups of a row
// XOR-swizzled by the row index so that the 16 rows an MFMA fragment reads
// fall in different banks; each wave computes a quarter of a layer's outputs
// for all FT rows, its weight fragments read straight from global memory (the
// BF16 weights, 224 KB, stay in L2).
// ---------------------------------------------------------------------------
constexpr int FT = 32;

// Element offset of (row, k) in a swizzled [FT][kdim] activation tile.
__device__ __forceinline__ int swz(int row, int k, int kdim)
{
    return row * kdim + ((((k >> 3) ^ (row & 15))) << 3) + (k & 7);
}

// One layer: out(i, j) = sum_k in(i, k) W[j][k] for the FT rows and this
// wave's N / 4 outputs.  HIDDEN: BF16(ReLU(. + bias)) to the swizzled LDS tile
// `oh`; else . + bias as FP32 to `of` (row stride MLP_OUT).
template <int K, int N, bool HIDDEN>
__device__ __forceinline__ void fused_layer(const uint16_t* in, const uint16_t* __restrict__ W,
                                            const float* __restrict__ bias, uint16_t* oh, float* of)
{
    const int lane = lane_id();
    const int wave = threadIdx.x / ORBG_WAVE;
    const int r = lane & 15, q = lane >> 4;
    constexpr int NW = N / 4, CT = NW / 16, RT = FT / 16;
    f4v acc[RT][CT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[a][c] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int k = 0; k < K; k += 32) {
        const int kk = k + 8 * q;
        s8v fa[RT], fb[CT];
#pragma unroll
        for (int a = 0; a < RT; ++a) fa[a] = *reinterpret_cast<const s8v*>(in + swz(a * 16 + r, kk, K));
#pragma unroll
        for (int c = 0; c < CT; ++c)
            fb[c] = *reinterpret_cast<const s8v*>(W + (int64_t)(wave * NW + c * 16 + r) * K + kk);
#pragma unroll
        for (int a = 0; a < RT; ++a)
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, fa[a]),
                                                                    __builtin_bit_cast(bf8v, fb[c]), acc[a][c], 0, 0, 0);
    }
    // lane holds D[4q + t][r] of each 16 x 16 tile, t = 0..3
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int i = a * 16 + 4 * q + t;
                const int j = wave * NW + c * 16 + r;
                const float v = acc[a][c][t];
                if (!HIDDEN) {
                    of[i * MLP_OUT + j] = v + bias[j];
                } else if ((t & 1) == 0) {                // two rows of one output at a time
                    const uint32_t p = f32x2_to_bf16(fmaxf(v + bias[j], 0.f), fmaxf(acc[a][c][t | 1] + bias[j], 0.f));
                    oh[swz(i, j, N)] = (uint16_t)p;
                    oh[swz(i + 1, j, N)] = (uint16_t)(p >> 16);
                }
            }
}

// Features of 128 / LG rows of a tile (rows rr ..), LG lanes for two rows: the
// lanes of a group hold row `a` in the low and row `a + 64 / LG` in the high
// halves of 128 / LG packed keys each.  Rounding to BF16 keeps the order, so the
// rounded values are sorted (about 50 instructions a row for LG = 8, where
// sorting 32-bit magnitudes one row at a time took 200).  A row with a NaN sorts
// its 32-bit magnitudes instead (payloads need not keep their order).
template <int LG>
struct FeatureRows {
    static constexpr int R = MLP_IN / LG, ROWS = 2 * ORBG_WAVE / LG, HALF = ORBG_WAVE / LG;
    f4v v[2][R / 4];

    // row r of the tile: row ids[row0 + r] (or row0 + r) of llr, zeros where there is none
    __device__ __forceinline__ void load(const float* __restrict__ llr, int64_t llr_rows, const int64_t* __restrict__ ids,
                                         int64_t row0, int64_t batch, int rr)
    {
        const int g = lane_id() / LG, sub = lane_id() % LG;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t b = row0 + rr + g + t * HALF;
            const int64_t src = b < batch ? (ids ? ids[b] : b) : -1;
#pragma unroll
            for (int q = 0; q < R / 4; ++q) {
                v[t][q] = (f4v){0.f, 0.f, 0.f, 0.f};
                if (src >= 0 && src < llr_rows)
                    v[t][q] = *reinterpret_cast<const f4row*>(llr + src * MLP_IN + (q * LG + sub) * 4);
            }
        }
    }

    __device__ __forceinline__ void sort_to(uint16_t* sa, int rr) const
    {
        const int lane = lane_id(), g = lane / LG, sub = lane % LG;
        uint32_t k[R];
        bool nan = false;
#pragma unroll
        for (int q = 0; q < R / 4; ++q) {
            const float a[4] = {v[0][q].x, v[0][q].y, v[0][q].z, v[0][q].w};
            const float b[4] = {v[1][q].x, v[1][q].y, v[1][q].z, v[1][q].w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                k[q * 4 + t] = f32x2_to_bf16(fabsf(a[t]) * 0.125f, fabsf(b[t]) * 0.125f);
                nan |= __builtin_isnan(a[t]) || __builtin_isnan(b[t]);
            }
        }
        if (ballot(nan) != 0ull) {                        // every row of the wave, one after the other
            for (int r = 0; r < ROWS; ++r) {
                // elements 2 lane and 2 lane + 1 of the row, through the tile's own place
                uint32_t* tmp = reinterpret_cast<uint32_t*>(sa + (rr + r) * MLP_IN);   // 64 words: half a row's magnitudes
                uint32_t m[2];
                for (int h = 0; h < 2; ++h) {
                    if (g == r % HALF) {
#pragma unroll
                        for (int q = 0; q < R / 4; ++q) {
                            const f4v w = r < HALF ? v[0][q] : v[1][q];
                            const float f[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                if ((q * 4 + t) / (R / 2) == h)
                                    tmp[(q * 4 + t) % (R / 2) * LG + sub] = __float_as_uint(f[t]) & 0x7fffffffu;
                        }
                    }
                    wave_lds_sync();
                    m[h] = tmp[lane];
                    wave_lds_sync();
                }
                bitonic_sort<2, uint32_t>(m);
                const uint32_t pair = (uint32_t)f32_to_bf16(__uint_as_float(m[0]) * 0.125f) |
                                      ((uint32_t)f32_to_bf16(__uint_as_float(m[1]) * 0.125f) << 16);
                *reinterpret_cast<uint32_t*>(sa + swz(rr + r, 2 * lane, MLP_IN)) = pair;
            }
            return;
        }
        group_sort<KeyPairU16, LG, R>(k);
        // element sub R + j of both rows; 8 values are one swizzled group
#pragma unroll
        for (int q = 0; q < R / 8; ++q) {
            uint4 a, b;
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                lo[t] = __builtin_amdgcn_perm(k[q * 8 + 2 * t + 1], k[q * 8 + 2 * t], 0x05040100u);
                hi[t] = __builtin_amdgcn_perm(k[q * 8 + 2 * t + 1], k[q * 8 + 2 * t], 0x07060302u);
            }
            a = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            b = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(sa + swz(rr + g, sub * R + q * 8, MLP_IN)) = a;
            *reinterpret_cast<uint4*>(sa + swz(rr + g + HALF, sub * R + q * 8, MLP_IN)) = b;
        }
    }
};

// FEAT: features of llr rows (ids[b], or b) made here, a row outside
// [0, llr_rows) giving zero features; else read from x.  logits (or nullptr)
// and order (or nullptr, ORDER false) receive the results.
template <bool FEAT, bool ORDER>
__global__ void __launch_bounds__(256)
mlp_infer_kernel(const float* __restrict__ llr, int64_t llr_rows, const int64_t* __restrict__ ids,
                 const uint16_t* __restrict__ x, int64_t batch, const float* __restrict__ w,
                 const uint16_t* __restrict__ wb, float* __restrict__ logits, uint8_t* __restrict__ order, int pin0)
{
    __shared__ __align__(16) uint16_t sa[FT * MLP_HID];     // features (FT x 128), then h2
    __shared__ __align__(16) uint16_t sb[FT * MLP_HID];     // h1, then the logits (FT x 64 FP32)
    const int wave = threadIdx.x / ORBG_WAVE;
    const int64_t row0 = (int64_t)blockIdx.x * FT;
    const int rows = (int)(batch - row0 < FT ? batch - row0 : FT);
    if (FEAT) {
        // sorted |LLR| / 8 in BF16 (as features_kernel); rows past the batch are zero
        FeatureRows<16> f;
        static_assert(4 * FeatureRows<16>::ROWS == FT, "eight rows a wave");
        f.load(llr, llr_rows, ids, row0, batch, wave * 8);
        f.sort_to(sa, wave * 8);
    } else {
        for (int g = threadIdx.x; g < FT * (MLP_IN / 8); g += 256) {
            const int rr = g / (MLP_IN / 8), kg = g % (MLP_IN / 8);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (rr < rows) v = *reinterpret_cast<const uint4*>(x + (row0 + rr) * MLP_IN + kg * 8);
            *reinterpret_cast<uint4*>(sa + swz(rr, kg * 8, MLP_IN)) = v;
        }
    }
    __syncthreads();
    fused_layer<MLP_IN, MLP_HID, true>(sa, wb + MLP_OFF_W1, w + MLP_OFF_B1, sb, nullptr);
    __syncthreads();
    fused_layer<MLP_HID, MLP_HID, true>(sb, wb + MLP_OFF_W2, w + MLP_OFF_B2, sa, nullptr);
    __syncthreads();
    float* lg = reinterpret_cast<float*>(sb);
    fused_layer<MLP_HID, MLP_OUT, false>(sa, wb + MLP_OFF_W3, w + MLP_OFF_B3, nullptr, lg);
    __syncthreads();
    if (logits != nullptr)
        for (int e = threadIdx.x; e < rows * MLP_OUT; e += 256) logits[row0 * MLP_OUT + e] = lg[e];
    if (ORDER && wave * 8 < rows)
        order_of_rows(lg + wave * 8 * MLP_OUT, rows - wave * 8, pin0, order + (row0 + wave * 8) * MLP_OUT);
}

// Large batches: one workgroup of eight waves per CU keeps all weights in
// registers (128 a lane: each wave an eighth of the outputs of layers 1 and 2, a
// quarter of layer 3's for half of the rows) and works through tiles of PT rows,
// so the weights are read once per CU instead of once per 32 rows (8192 times
// 224 KB from L2 at 2.6 x 10^5 rows).  Activations and logits as in
// mlp_infer_kernel; the next tile's LLR rows load during the batch orders.  Same
// products in the same order: the same bits.  2^18 rows with features and
// orders: 247 us with the weights from L2, 147 us so (492 us before the group
// sorts).
constexpr int PT = 128;
constexpr int RT = 2;            // row tiles of 16 at a time (four: registers go to scratch)

template <int K, int T, int CT>
__device__ __forceinline__ void reg_products(const uint16_t* in, int row0, const s8v (&W)[CT][K / 32], f4v (&acc)[T][CT])
{
    const int lane = lane_id(), r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[a][c] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < K / 32; ++k) {
        s8v fa[T];
#pragma unroll
        for (int a = 0; a < T; ++a)
            fa[a] = *reinterpret_cast<const s8v*>(in + swz(row0 + a * 16 + r, k * 32 + 8 * q, K));
#pragma unroll
        for (int a = 0; a < T; ++a)
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, fa[a]),
                                                                    __builtin_bit_cast(bf8v, W[c][k]), acc[a][c], 0, 0, 0);
    }
}

template <int K, int CT>
__device__ __forceinline__ void load_weights(const uint16_t* __restrict__ w, int col0, s8v (&W)[CT][K / 32])
{
    const int lane = lane_id(), r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int k = 0; k < K / 32; ++k)
            W[c][k] = *reinterpret_cast<const s8v*>(w + (int64_t)(col0 + c * 16 + r) * K + k * 32 + 8 * q);
}

// BF16(ReLU(. + bias)) of 16 RT rows x 32 outputs into the tile.
__device__ __forceinline__ void store_hidden(const f4v (&acc)[RT][2], int row0, int col0, const float (&bias)[2], uint16_t* oh)
{
    const int lane = lane_id(), r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int t = 0; t < 4; t += 2) {
                const int i = row0 + a * 16 + 4 * q + t, j = col0 + c * 16 + r;
                const uint32_t p = f32x2_to_bf16(fmaxf(acc[a][c][t] + bias[c], 0.f), fmaxf(acc[a][c][t + 1] + bias[c], 0.f));
                oh[swz(i, j, MLP_HID)] = (uint16_t)p;
                oh[swz(i + 1, j, MLP_HID)] = (uint16_t)(p >> 16);
            }
}

template <bool FEAT, bool ORDER>
__global__ void __launch_bounds__(512)
mlp_infer_persistent(const float* __restrict__ llr, int64_t llr_rows, const int64_t* __restrict__ ids,
                     const uint16_t* __restrict__ x, int64_t batch, const float* __restrict__ w,
                     const uint16_t* __restrict__ wb, float* __restrict__ logits, uint8_t* __restrict__ order, int pin0)
{
    extern __shared__ __align__(16) unsigned char orbg_mlp_lds[];
    uint16_t* sa = reinterpret_cast<uint16_t*>(orbg_mlp_lds);   // features (PT x 128), then h2 (PT x 256)
    uint16_t* sb = sa + PT * MLP_HID;                           // h1, then the logits (PT x 64 FP32)
    float* lg = reinterpret_cast<float*>(sb);
    const int lane = lane_id();
    const int wave = threadIdx.x / ORBG_WAVE;
    s8v W1[2][MLP_IN / 32], W2[2][MLP_HID / 32], W3[1][MLP_HID / 32];
    const int c12 = wave * 32, c3 = (wave & 3) * 16, r3 = (wave >> 2) * 64;
    load_weights<MLP_IN, 2>(wb + MLP_OFF_W1, c12, W1);
    load_weights<MLP_HID, 2>(wb + MLP_OFF_W2, c12, W2);
    load_weights<MLP_HID, 1>(wb + MLP_OFF_W3, c3, W3);
    const int r = lane & 15, q = lane >> 4;
    const float b1[2] = {w[MLP_OFF_B1 + c12 + r], w[MLP_OFF_B1 + c12 + 16 + r]};
    const float b2[2] = {w[MLP_OFF_B2 + c12 + r], w[MLP_OFF_B2 + c12 + 16 + r]};
    const float b3 = w[MLP_OFF_B3 + c3 + r];
    const int64_t tiles = (batch + PT - 1) / PT;
    FeatureRows<8> f;
    static_assert(8 * FeatureRows<8>::ROWS == PT, "sixteen rows a wave");
    if (FEAT) f.load(llr, llr_rows, ids, (int64_t)blockIdx.x * PT, batch, wave * 16);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t row0 = t * PT;
        const int rows = (int)(batch - row0 < PT ? batch - row0 : PT);
        if (FEAT) {
            f.sort_to(sa, wave * 16);
        } else {
            for (int g = threadIdx.x; g < PT * (MLP_IN / 8); g += 512) {
                const int rr = g / (MLP_IN / 8), kg = g % (MLP_IN / 8);
                uint4 v = make_uint4(0u, 0u, 0u, 0u);
                if (rr < rows) v = *reinterpret_cast<const uint4*>(x + (row0 + rr) * MLP_IN + kg * 8);
                *reinterpret_cast<uint4*>(sa + swz(rr, kg * 8, MLP_IN)) = v;
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int h = 0; h < PT; h += 16 * RT) {
            f4v acc[RT][2];
            reg_products<MLP_IN, RT, 2>(sa, h, W1, acc);
            store_hidden(acc, h, c12, b1, sb);
        }
        __syncthreads();
#pragma unroll 1
        for (int h = 0; h < PT; h += 16 * RT) {
            f4v acc[RT][2];
            reg_products<MLP_HID, RT, 2>(sb, h, W2, acc);
            store_hidden(acc, h, c12, b2, sa);
        }
        __syncthreads();
#pragma unroll 1
        for (int h = r3; h < r3 + 64; h += 16 * RT) {
            f4v acc[RT][1];
            reg_products<MLP_HID, RT, 1>(sa, h, W3, acc);
#pragma unroll
            for (int a = 0; a < RT; ++a)
#pragma unroll
                for (int u = 0; u < 4; ++u) lg[(h + a * 16 + 4 * q + u) * MLP_OUT + c3 + r] = acc[a][0][u] + b3;
        }
        if (FEAT && t + gridDim.x < tiles)
            f.load(llr, llr_rows, ids, (t + gridDim.x) * PT, batch, wave * 16);
        __syncthreads();
        if (logits != nullptr)
            for (int e = threadIdx.x; e < rows * MLP_OUT; e += 512) logits[row0 * MLP_OUT + e] = lg[e];
        if (ORDER) {
#pragma unroll 1
            for (int rr = wave * 16; rr < wave * 16 + 16 && rr < rows; rr += 8)
                order_of_rows(lg + rr * MLP_OUT, rows - rr, pin0, order + (row0 + rr) * MLP_OUT);
        }
        // (the next tile's features go to sa, which layer 3 has read; lg is
        // written again two barriers on)
    }
}

// Rows from which the persistent kernel is the quicker one (20000 rows 29.0 us
// against 27.2 of the other, 32768 rows 27.9 against 32).
#define MLP_PERSIST_ROWS 24576
hipError_t mlp_infer(const float* w, const uint16_t* wb, const float* llr, int64_t llr_rows, const int64_t* ids,
                     const uint16_t* x, int64_t batch, float* logits, uint8_t* order, bool pin0, hipStream_t st)
{
    if (batch <= 0) return hipSuccess;
    // from about two tiles per CU on, the weights stay in registers
    int dev = 0, cus = 256;
    if (batch >= MLP_PERSIST_ROWS && hipGetDevice(&dev) == hipSuccess) {
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        const int64_t tiles = (batch + PT - 1) / PT;
        const unsigned pg = (unsigned)(tiles < cus ? tiles : cus);
        const size_t lds = (size_t)2 * PT * MLP_HID * sizeof(uint16_t);
        auto go = [&](auto kernel) -> hipError_t {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            kernel<<<pg, 512, lds, st>>>(llr, llr_rows, ids, x, batch, w, wb, logits, order, pin0);
            return hipGetLastError();
        };
        if (llr) return order ? go(mlp_infer_persistent<true, true>) : go(mlp_infer_persistent<true, false>);
        return order ? go(mlp_infer_persistent<false, true>) : go(mlp_infer_persistent<false, false>);
    }
    const unsigned grid = (unsigned)((batch + FT - 1) / FT);
    if (llr) {
        if (order)
            mlp_infer_kernel<true, true><<<grid, 256, 0, st>>>(llr, llr_rows, ids, x, batch, w, wb, logits, order, pin0);
        else
            mlp_infer_kernel<true, false><<<grid, 256, 0, st>>>(llr, llr_rows, ids, x, batch, w, wb, logits, order, pin0);
    } else {
        if (order)
            mlp_infer_kernel<false, true><<<grid, 256, 0, st>>>(llr, llr_rows, ids, x, batch, w, wb, logits, order, pin0);
        else
            mlp_infer_kernel<false, false><<<grid, 256, 0, st>>>(llr, llr_rows, ids, x, batch, w, wb, logits, order,
                                                                pin0);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Training: three launches.
//   1. train_rows_kernel, FT rows per workgroup: forward, softmax cross-entropy
//      and the gradients dl, dz2, dz1 of the layers' outputs, all from LDS; the
//      activations and gradients go out transposed ([feature][row]), as the
//      weight gradients reduce over the rows.
//   2. train_weights_kernel: dW = dz^T h and db = the row sums of dz^T as 64 x 64
//      tiles over chunks of rows, fragments read straight from the transposed
//      copies (8 consecutive rows are one 16-byte load; from the row-major copies
//      each was eight 2-byte loads).
//   3. train_reduce_kernel: the chunks' partials in a fixed order, and the loss.
// One minibatch of 8192: 38 us (24, 14 and 4 on the device's clock,
// overlapping); 453 us as
// 19 launches of separate products, column sums (181 us of them, one thread per
// column) and reductions.
// Bound: latency and launches (5 GFLOP, 20 MB written and read once).
// ---------------------------------------------------------------------------

// Element offset in a [FT][64] tile (as swz, eight 16-byte groups a row).
__device__ __forceinline__ int swz64(int row, int k) { return row * MLP_OUT + ((((k >> 3) ^ (row & 7))) << 3) + (k & 7); }

constexpr int TRAIN_THREADS = 512;

// out(i, j) = sum_k in(i, k) W[j][k] for the FT rows and this wave's eighth of
// the 256 outputs, in the order of fused_layer.  SWZ64: `in` is a [FT][64] tile.
template <int K, bool SWZ64>
__device__ __forceinline__ void train_products(const uint16_t* in, const uint16_t* __restrict__ W, f4v (&acc)[FT / 16][2])
{
    const int lane = lane_id(), wave = threadIdx.x / ORBG_WAVE, r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int a = 0; a < FT / 16; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[a][c] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k = 0; k < K; k += 32) {
        const int kk = k + 8 * q;
        s8v fa[FT / 16], fb[2];
#pragma unroll
        for (int a = 0; a < FT / 16; ++a)
            fa[a] = *reinterpret_cast<const s8v*>(in + (SWZ64 ? swz64(a * 16 + r, kk) : swz(a * 16 + r, kk, K)));
#pragma unroll
        for (int c = 0; c < 2; ++c) fb[c] = *reinterpret_cast<const s8v*>(W + (int64_t)(wave * 32 + c * 16 + r) * K + kk);
#pragma unroll
        for (int a = 0; a < FT / 16; ++a)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, fa[a]),
                                                                    __builtin_bit_cast(bf8v, fb[c]), acc[a][c], 0, 0, 0);
    }
}

// This wave's outputs f(i, j, value) in BF16, to the [FT][256] tile (or nullptr)
// and to the transposed copy (column row0 of [256][ldb]).
template <typename F>
__device__ __forceinline__ void train_store(const f4v (&acc)[FT / 16][2], uint16_t* tile, uint16_t* __restrict__ t,
                                            int64_t ldb, int64_t row0, F&& f)
{
    const int lane = lane_id(), wave = threadIdx.x / ORBG_WAVE, r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int a = 0; a < FT / 16; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int i = a * 16 + 4 * q, j = wave * 32 + c * 16 + r;
            const uint32_t lo = f32x2_to_bf16(f(i, j, acc[a][c][0]), f(i + 1, j, acc[a][c][1]));
            const uint32_t hi = f32x2_to_bf16(f(i + 2, j, acc[a][c][2]), f(i + 3, j, acc[a][c][3]));
            if (tile) {
                tile[swz(i, j, MLP_HID)] = (uint16_t)lo;
                tile[swz(i + 1, j, MLP_HID)] = (uint16_t)(lo >> 16);
                tile[swz(i + 2, j, MLP_HID)] = (uint16_t)hi;
                tile[swz(i + 3, j, MLP_HID)] = (uint16_t)(hi >> 16);
            }
            *reinterpret_cast<uint2*>(t + (int64_t)j * ldb + row0 + i) = make_uint2(lo, hi);
        }
}

// wloss: per wave, the loss summed over its rows.  Rows past the batch: zero
// gradients.
__global__ void __launch_bounds__(TRAIN_THREADS)
train_rows_kernel(const uint16_t* __restrict__ x, const int32_t* __restrict__ labels, int64_t batch,
                  const float* __restrict__ w, const uint16_t* __restrict__ wb, const uint16_t* __restrict__ wt,
                  MlpWorkspace ws)
{
    __shared__ __align__(16) uint16_t s0[FT * MLP_HID];     // x (FT x 128), then dz2
    __shared__ __align__(16) uint16_t s1[FT * MLP_HID];     // h1
    __shared__ __align__(16) uint16_t s2[FT * MLP_HID];     // h2
    __shared__ __align__(16) float lg[FT * MLP_OUT];        // logits
    __shared__ __align__(16) uint16_t sd[FT * MLP_OUT];     // dl
    const int lane = lane_id();
    const int wave = threadIdx.x / ORBG_WAVE;
    const int64_t row0 = (int64_t)blockIdx.x * FT, ldb = ws.ldb;
    const int rows = (int)(batch - row0 < FT ? batch - row0 : FT);
    for (int g = threadIdx.x; g < FT * (MLP_IN / 8); g += TRAIN_THREADS) {
        const int rr = g / (MLP_IN / 8), kg = g % (MLP_IN / 8);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (rr < rows) v = *reinterpret_cast<const uint4*>(x + (row0 + rr) * MLP_IN + kg * 8);
        *reinterpret_cast<uint4*>(s0 + swz(rr, kg * 8, MLP_IN)) = v;
    }
    __syncthreads();
    // eight rows of one feature from a tile
    auto column = [&](const uint16_t* tile, int i, auto&& at) -> uint4 {
        uint32_t p[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) p[t] = (uint32_t)tile[at(i + 2 * t)] | ((uint32_t)tile[at(i + 2 * t + 1)] << 16);
        return make_uint4(p[0], p[1], p[2], p[3]);
    };
    for (int g = threadIdx.x; g < MLP_IN * (FT / 8); g += TRAIN_THREADS) {
        const int j = g / (FT / 8), i = g % (FT / 8) * 8;
        *reinterpret_cast<uint4*>(ws.xt + (int64_t)j * ldb + row0 + i) =
            column(s0, i, [&](int k) { return swz(k, j, MLP_IN); });
    }
    f4v acc[FT / 16][2];
    train_products<MLP_IN, false>(s0, wb + MLP_OFF_W1, acc);
    train_store(acc, s1, ws.h1t, ldb, row0, [&](int, int j, float v) { return fmaxf(v + w[MLP_OFF_B1 + j], 0.f); });
    __syncthreads();
    train_products<MLP_HID, false>(s1, wb + MLP_OFF_W2, acc);
    train_store(acc, s2, ws.h2t, ldb, row0, [&](int, int j, float v) { return fmaxf(v + w[MLP_OFF_B2 + j], 0.f); });
    __syncthreads();
    {
        // logits: wave = (row tile, column tile)
        static_assert(FT / 16 * (MLP_OUT / 16) == TRAIN_THREADS / ORBG_WAVE, "one tile a wave");
        const int r = lane & 15, q = lane >> 4, i0 = (wave >> 2) * 16, j = (wave & 3) * 16 + r;
        f4v l = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < MLP_HID; k += 32)
            l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf8v, *reinterpret_cast<const s8v*>(s2 + swz(i0 + r, k + 8 * q, MLP_HID))),
                __builtin_bit_cast(bf8v, *reinterpret_cast<const s8v*>(wb + MLP_OFF_W3 + j * MLP_HID + k + 8 * q)), l, 0,
                0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) lg[(i0 + 4 * q + u) * MLP_OUT + j] = l[u] + w[MLP_OFF_B3 + j];
    }
    __syncthreads();
    // softmax cross-entropy, a row per wave at a time (lane = class):
    // dl = (softmax - onehot) / batch in BF16
    float loss = 0.f;
    for (int rr = wave * (FT / 8); rr < (wave + 1) * (FT / 8); ++rr) {
        uint16_t d = 0;
        if (rr < rows) {
            const float v = lg[rr * MLP_OUT + lane];
            float mx = v;
#pragma unroll
            for (int k = 1; k < 64; k <<= 1) mx = fmaxf(mx, __shfl_xor(mx, k, ORBG_WAVE));
            const float e = __expf(v - mx);
            float s = e;
#pragma unroll
            for (int k = 1; k < 64; k <<= 1) s += __shfl_xor(s, k, ORBG_WAVE);
            const int lab = labels[row0 + rr];
            const float p = e / s;
            d = f32_to_bf16((p - (lane == lab ? 1.f : 0.f)) / (float)batch);
            loss += __logf(s) + mx - __shfl(v, lab & 63, ORBG_WAVE);
        }
        sd[swz64(rr, lane)] = d;
    }
    if (lane == 0) ws.wloss[(int64_t)blockIdx.x * 8 + wave] = loss;
    __syncthreads();
    if (threadIdx.x < MLP_OUT * (FT / 8)) {
        const int j = threadIdx.x / (FT / 8), i = threadIdx.x % (FT / 8) * 8;
        *reinterpret_cast<uint4*>(ws.dlt + (int64_t)j * ldb + row0 + i) = column(sd, i, [&](int k) { return swz64(k, j); });
    }
    // dz2 = (dl W3) * [h2 > 0], dz1 = (dz2 W2) * [h1 > 0]
    train_products<MLP_OUT, true>(sd, wt + MLP_T_W3, acc);
    train_store(acc, s0, ws.dz2t, ldb, row0, [&](int i, int j, float v) { return s2[swz(i, j, MLP_HID)] != 0 ? v : 0.f; });
    __syncthreads();
    train_products<MLP_HID, false>(s0, wt + MLP_T_W2, acc);
    train_store(acc, nullptr, ws.dz1t, ldb, row0, [&](int i, int j, float v) { return s1[swz(i, j, MLP_HID)] != 0 ? v : 0.f; });
}

// blockIdx.x: 64 x 64 tile of dW1 (0..7), dW2 (8..23) or dW3 (24..27);
// blockIdx.y: chunk of rows.  Tiles of the first column block make the bias
// gradient of their rows too (a product with ones).
__global__ void __launch_bounds__(256) train_weights_kernel(MlpWorkspace ws)
{
    const int lane = lane_id(), wave = threadIdx.x / ORBG_WAVE, r = lane & 15, q = lane >> 4;
    const int t = blockIdx.x;
    const uint16_t* A = t < 8 ? ws.dz1t : t < 24 ? ws.dz2t : ws.dlt;
    const uint16_t* B = t < 8 ? ws.xt : t < 24 ? ws.h1t : ws.h2t;
    const int N = t < 8 ? MLP_IN : MLP_HID;
    const int tl = t < 8 ? t : t < 24 ? t - 8 : t - 24, nj = N / 64;
    const int i0 = tl / nj * 64 + (wave >> 1) * 32, j0 = tl % nj * 64 + (wave & 1) * 32;
    const int off = t < 8 ? MLP_OFF_W1 : t < 24 ? MLP_OFF_W2 : MLP_OFF_W3;
    const int boff = t < 8 ? MLP_OFF_B1 : t < 24 ? MLP_OFF_B2 : MLP_OFF_B3;
    const bool bias = j0 == 0;                              // (wave-uniform)
    const int64_t kb = (int64_t)blockIdx.y * ws.kchunk, ke = kb + ws.kchunk < ws.rows ? kb + ws.kchunk : ws.rows;
    f4v acc[2][2], sum[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        sum[a] = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[a][c] = (f4v){0.f, 0.f, 0.f, 0.f};
    }
    const uint16_t* pa = A + (int64_t)(i0 + r) * ws.ldb + 8 * q;
    const uint16_t* pb = B + (int64_t)(j0 + r) * ws.ldb + 8 * q;
    const s8v ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
#pragma unroll 4
    for (int64_t k = kb; k < ke; k += 32) {
        s8v fa[2], fb[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) fa[a] = *reinterpret_cast<const s8v*>(pa + a * 16 * ws.ldb + k);
#pragma unroll
        for (int c = 0; c < 2; ++c) fb[c] = *reinterpret_cast<const s8v*>(pb + c * 16 * ws.ldb + k);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, fa[a]),
                                                                    __builtin_bit_cast(bf8v, fb[c]), acc[a][c], 0, 0, 0);
            if (bias)
                sum[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, fa[a]),
                                                                 __builtin_bit_cast(bf8v, ones), sum[a], 0, 0, 0);
        }
    }
    // lane holds D[4q + u][r] of each 16 x 16 tile, u = 0..3
    float* part = ws.part + (int64_t)blockIdx.y * MLP_NPARAM;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + a * 16 + 4 * q + u;
#pragma unroll
            for (int c = 0; c < 2; ++c) part[off + i * N + j0 + c * 16 + r] = acc[a][c][u];
            if (bias && r == 0) part[boff + i] = sum[a][u];
        }
}

// grads = the chunks' partials in ascending order; the last workgroup sums the
// loss (nloss values).
__global__ void __launch_bounds__(256) train_reduce_kernel(const float* __restrict__ part, int splits,
                                                           float* __restrict__ grads, const float* __restrict__ wloss,
                                                           int64_t nloss, float scale, float* __restrict__ loss)
{
    if (blockIdx.x + 1 < gridDim.x) {
        const int e = (int)blockIdx.x * 256 + threadIdx.x;
        if (e >= MLP_NPARAM) return;
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < splits; ++z) s += part[(int64_t)z * MLP_NPARAM + e];
        grads[e] = s;
        return;
    }
    __shared__ float red[256];
    float s = 0.f;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < nloss; i += 256) s += wloss[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if (threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] * scale;
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
static int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

MlpWorkspace mlp_carve(void* base, int64_t batch)
{
    MlpWorkspace w;
    unsigned char* p = reinterpret_cast<unsigned char*>(base);
    int64_t o = 0;
    auto take = [&](int64_t bytes) { void* r = p ? p + o : nullptr; o += align256(bytes); return r; };
    // rows padded to whole MFMA steps (the tail holds zero gradients); weight
    // gradients reduce over chunks of at least MLP_KCHUNK_MIN rows, at most
    // MLP_SPLITS_MAX of them (each writes and reads back all gradients once)
    w.rows = (batch + 31) / 32 * 32;
    // (the copies' row length is kept off multiples of 128 elements: a fragment's
    // 16 rows would otherwise fall on the same memory channels)
    w.ldb = w.rows + (w.rows % 64 == 0 ? 32 : 0);
    int64_t kchunk = (batch + MLP_SPLITS_MAX - 1) / MLP_SPLITS_MAX;
    kchunk = kchunk < MLP_KCHUNK_MIN ? MLP_KCHUNK_MIN : (kchunk + 31) / 32 * 32;
    w.splits = (int)((batch + kchunk - 1) / kchunk);
    w.kchunk = (int)kchunk;
    w.xt = (uint16_t*)take(w.ldb * MLP_IN * 2);
    w.h1t = (uint16_t*)take(w.ldb * MLP_HID * 2);
    w.h2t = (uint16_t*)take(w.ldb * MLP_HID * 2);
    w.dlt = (uint16_t*)take(w.ldb * MLP_OUT * 2);
    w.dz2t = (uint16_t*)take(w.ldb * MLP_HID * 2);
    w.dz1t = (uint16_t*)take(w.ldb * MLP_HID * 2);
    // (room for the most splits any batch of this size or smaller uses, so the
    // work space grows with the batch)
    const int64_t room = (batch + MLP_KCHUNK_MIN - 1) / MLP_KCHUNK_MIN;
    w.part = (float*)take((room < MLP_SPLITS_MAX ? room : MLP_SPLITS_MAX) * MLP_NPARAM * 4);
    w.wloss = (float*)take((batch + FT - 1) / FT * 8 * 4);
    w.bytes = o;
    return w;
}

hipError_t mlp_features(const float* llr, int64_t batch, uint16_t* x, hipStream_t st, const int64_t* ids)
{
    if (batch > 0) features_kernel<<<(unsigned)((batch + 3) / 4), 256, 0, st>>>(llr, batch, x, ids);
    return hipGetLastError();
}

hipError_t mlp_prepare(const float* w, uint16_t* wb, uint16_t* wt, hipStream_t st)
{
    prepare_kernel<<<(MLP_NPARAM + 255) / 256, 256, 0, st>>>(w, wb, wt);
    return hipGetLastError();
}

hipError_t mlp_forward(const float* w, const uint16_t* wb, const uint16_t* x, int64_t batch, float* logits,
                       const MlpWorkspace&, hipStream_t st)
{
    return mlp_infer(w, wb, nullptr, 0, nullptr, x, batch, logits, nullptr, false, st);
}

// Backward: forward, softmax cross-entropy, gradients of all parameters, mean loss.
hipError_t mlp_backward(const float* w, const uint16_t* wb, const uint16_t* wt, const uint16_t* x,
                        const int32_t* labels, int64_t batch, float* grads, float* loss, const MlpWorkspace& ws,
                        hipStream_t st)
{
    if (batch <= 0) return hipSuccess;
    const unsigned tiles = (unsigned)((batch + FT - 1) / FT);
    train_rows_kernel<<<tiles, TRAIN_THREADS, 0, st>>>(x, labels, batch, w, wb, wt, ws);
    train_weights_kernel<<<dim3(28, ws.splits), 256, 0, st>>>(ws);
    train_reduce_kernel<<<(MLP_NPARAM + 255) / 256 + 1, 256, 0, st>>>(ws.part, ws.splits, grads, ws.wloss,
                                                                      (int64_t)tiles * 8, 1.0f / (float)batch, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(float* w, float* m, float* v, const float* g, float lr, int step, uint16_t* wb, uint16_t* wt,
                    hipStream_t st)
{
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    adam_kernel<<<(MLP_NPARAM + 255) / 256, 256, 0, st>>>(w, m, v, g, lr, b1, b2, eps, c1, c2, wb, wt);
    return hipGetLastError();
}

hipError_t mlp_order(const float* logits, int64_t batch, uint8_t* order, hipStream_t st, bool pin0)
{
    if (batch > 0) order_kernel<<<(unsigned)((batch + 3) / 4), 256, 0, st>>>(logits, batch, order, pin0 ? 1 : 0);
    return hipGetLastError();
}

}  // namespace orbg
