// Dispatch of a decode to the kernels of its keys per lane (decode_nk*.hip);
// the kernels themselves are in decode_impl.h.
#include "orbg_kernels.h"
#include "orbg_internal.h"

namespace orbg {

template <int NKMAX>
hipError_t launch_decode_nk(const DecodeArgs& a, bool s32, hipStream_t stream);
extern template hipError_t launch_decode_nk<1>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_decode_nk<2>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_decode_nk<4>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_decode_nk<8>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_decode_nk<16>(const DecodeArgs&, bool, hipStream_t);
template <int NK>
hipError_t launch_match_nk(const DecodeArgs& a, bool s32, bool marked, hipStream_t stream);
extern template hipError_t launch_match_nk<1>(const DecodeArgs&, bool, bool, hipStream_t);
extern template hipError_t launch_match_nk<2>(const DecodeArgs&, bool, bool, hipStream_t);
extern template hipError_t launch_match_nk<4>(const DecodeArgs&, bool, bool, hipStream_t);
extern template hipError_t launch_match_nk<8>(const DecodeArgs&, bool, bool, hipStream_t);
extern template hipError_t launch_match_nk<16>(const DecodeArgs&, bool, bool, hipStream_t);
template <int NK>
hipError_t launch_first_nk(const DecodeArgs& a, bool s32, hipStream_t stream);
extern template hipError_t launch_first_nk<1>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_first_nk<2>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_first_nk<4>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_first_nk<8>(const DecodeArgs&, bool, hipStream_t);
extern template hipError_t launch_first_nk<16>(const DecodeArgs&, bool, hipStream_t);

static hipError_t launch_light(const DecodeArgs& a, int nk, bool s32, hipStream_t stream)
{
    if (nk <= 1) return launch_decode_nk<1>(a, s32, stream);
    if (nk <= 2) return launch_decode_nk<2>(a, s32, stream);
    if (nk <= 4) return launch_decode_nk<4>(a, s32, stream);
    if (nk <= 8) return launch_decode_nk<8>(a, s32, stream);
    return launch_decode_nk<16>(a, s32, stream);
}

static hipError_t launch_first(const DecodeArgs& a, int nk, bool s32, hipStream_t stream)
{
    if (nk <= 1) return launch_first_nk<1>(a, s32, stream);
    if (nk <= 2) return launch_first_nk<2>(a, s32, stream);
    if (nk <= 4) return launch_first_nk<4>(a, s32, stream);
    if (nk <= 8) return launch_first_nk<8>(a, s32, stream);
    return launch_first_nk<16>(a, s32, stream);
}

static hipError_t launch_match(const DecodeArgs& a, int nk, bool s32, bool marked, hipStream_t stream)
{
    if (nk <= 1) return launch_match_nk<1>(a, s32, marked, stream);
    if (nk <= 2) return launch_match_nk<2>(a, s32, marked, stream);
    if (nk <= 4) return launch_match_nk<4>(a, s32, marked, stream);
    if (nk <= 8) return launch_match_nk<8>(a, s32, marked, stream);
    return launch_match_nk<16>(a, s32, marked, stream);
}

// Lists the blocks marked ORBG_OPEN in the abandon flags and counts them.  One
// workgroup per LIST_SPAN flags: its marked blocks are counted, take their
// place with one increment, and are written in ascending order.
#define LIST_SPAN 4096
__global__ void __launch_bounds__(256) list_open_kernel(const uint8_t* __restrict__ flags, int64_t nblocks,
                                                        int64_t* __restrict__ list,
                                                        unsigned long long* __restrict__ count)
{
    __shared__ uint32_t waves[LIST_SPAN / 64];
    __shared__ unsigned long long at;
    const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const int64_t base = (int64_t)blockIdx.x * LIST_SPAN;
    uint64_t open[LIST_SPAN / 256];
#pragma unroll
    for (int k = 0; k < LIST_SPAN / 256; ++k) {
        const int64_t b = base + k * 256 + threadIdx.x;
        open[k] = __ballot(b < nblocks && flags[b] == ORBG_OPEN);
        if (lane == 0) waves[k * 4 + wave] = (uint32_t)__popcll(open[k]);
    }
    __syncthreads();
    if (wave == 0) {                                      // exclusive sums of the 64 counts
        const uint32_t v = waves[lane];
        uint32_t s = v;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(s, d, 64);
            s += lane >= d ? o : 0u;
        }
        waves[lane] = s - v;
        if (lane == 63) at = s != 0 ? atomicAdd(count, (unsigned long long)s) : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < LIST_SPAN / 256; ++k) {
        const uint64_t below = open[k] & ((1ull << lane) - 1ull);
        if ((open[k] >> lane) & 1ull)
            list[at + waves[k * 4 + wave] + __popcll(below)] = base + k * 256 + threadIdx.x;
    }
}

// Largest batch that the match search decodes in one launch.  A first pass
// saves it the short searches, but is a launch of its own, and a wave that takes
// one block beside the others is as quick as one that takes none.  One launch
// against two, us: BCH(127,113) at 5 dB 8192 blocks 17.1 / 20.3, 24576 blocks
// 24.6 / 24.7, 32768 blocks 30.7 / 27.6; n = 256, m = 16 at 24576 blocks 36.9 /
// 45.8; n = 64, m = 12 19.6 / 23.3; n = 32, m = 6 at 8192 blocks 13.9 / 15.8.
#define ORBG_MATCH_DIRECT 24576

hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream)
{
    if (a.nblocks < 1) return hipSuccess;
    int nk = 1, mmax = 0;
    for (int i = 0; i < a.codes.ncodes; ++i) {
        nk = a.codes.c[i].nk > nk ? a.codes.c[i].nk : nk;
        mmax = a.codes.c[i].m > mmax ? a.codes.c[i].m : mmax;
    }
    const bool s32 = mmax <= 32;
    if (a.oneline && (a.mixed || a.order)) return hipErrorInvalidValue;   // one code, plain batch order
    if (a.mixed && nk > 4) return hipErrorInvalidValue;                  // mixed launches take n <= 256
    if (!uses_match(a)) {
        hipError_t e = launch_light(a, nk, s32, stream);
        if (e == hipSuccess && a.list_only) {
            list_open_kernel<<<(unsigned)((a.nblocks + LIST_SPAN - 1) / LIST_SPAN), 256, 0, stream>>>(
                a.abandoned, a.nblocks, a.list, a.ctrs + ORBG_CTR_HEAVY_COUNT);
            e = hipGetLastError();
        }
        return e;
    }
    if (a.order || a.nblocks <= ORBG_MATCH_DIRECT) return launch_match(a, nk, s32, false, stream);
    // else a first pass (screening and the first batch of patterns), then the
    // match search of the blocks it leaves; at most ORBG_PAST bytes of codewords
    // at a time (the first pass addresses them by 32-bit offsets)
    const int64_t most = a.mixed ? 0x40000000ll : 0x40000000ll / a.codes.c[0].n;
    for (int64_t from = 0; from < a.nblocks; from += most) {
        DecodeArgs p = a;
        p.nblocks = a.nblocks - from < most ? a.nblocks - from : most;
        if (a.mixed) {
            p.block_code += from;
            p.row_off += from;
        } else {
            p.llr += from * a.codes.c[0].n;
            p.cw += from * a.codes.c[0].n;
        }
        p.queries += from;
        p.abandoned += from;
        hipError_t e = launch_first(p, nk, s32, stream);
        if (e == hipSuccess) e = launch_match(p, nk, s32, true, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace orbg
