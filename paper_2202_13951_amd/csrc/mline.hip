// Full (m-line) ORBGRAND decode (Sec. III-D; fit of Sec. III-E): the device
// table of subset counts the unranking reads, and the launch, which picks the
// kernel compiled for the request's largest segment count (mline_impl.h).
#include <map>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "orbg_device.h"
#include "orbg_internal.h"
#include "orbg_mline.h"

namespace orbg {

namespace {

constexpr int WL = ORBG_ML_WMAX;          // partial Hamming weights 0..22
constexpr int SL = ORBG_ML_SMAX;          // partial logistic weights 0..4095

// One step of the subset-count recursion: table for `len` from the one for len - 1.
__global__ void __launch_bounds__(256) subset_table_step(uint32_t* t, int len)
{
    const int cells = (WL + 1) * SL;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    uint32_t* cur = t + (size_t)len * cells;
    if (len == 0) {
        cur[c] = c == 0 ? 1u : 0u;
        return;
    }
    const uint32_t* prev = t + (size_t)(len - 1) * cells;
    const int w = c / SL, s = c % SL;
    uint64_t v = prev[c];
    if (w >= 1 && s >= len) v += prev[(w - 1) * SL + (s - len)];
    cur[c] = v > 0xffffffffull ? 0xffffffffu : (uint32_t)v;
}

}  // namespace

hipError_t build_subset_table(uint32_t* t, hipStream_t stream)
{
    const int cells = (WL + 1) * SL;
    for (int len = 0; len <= ORBG_ML_LMAX; ++len) {
        subset_table_step<<<(cells + 255) / 256, 256, 0, stream>>>(t, len);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {

std::mutex sets_mu;
std::map<std::pair<int, int>, MlineSets> sets_of;         // (device, min(n, 254))

// Lists of MlineSets, made on the host once per device and length: one walk per
// size counts the sets by rank sum (a recursion over the ranks), a second one
// places those up to the list's limit.
hipError_t make_sets(int top, MlineSets* out)
{
    const int S = ORBG_MM_SUMS;
    std::vector<uint64_t> cnt((size_t)8 * S, 0ull);
    cnt[0] = 1;
    for (int r = ORBG_LOW_RANKS + 1; r <= top; ++r)
        for (int c = 7; c >= 1; --c)
            for (int s = S - 1; s >= r; --s) cnt[(size_t)c * S + s] += cnt[(size_t)(c - 1) * S + s - r];
    std::vector<uint32_t> end((size_t)8 * S, 0u);
    std::vector<int> limit(8, S);
    std::vector<uint2> sets;
    for (int c = 1; c <= 7; ++c) {
        uint64_t sum = 0;
        for (int s = 0; s < S; ++s) {
            const uint64_t next = sum + cnt[(size_t)c * S + s];
            // (a third of the room for the larger sets: their lists reach further in weight)
            if (next > (c <= 3 ? ORBG_MM_LIST : ORBG_MM_LIST / 3) && limit[c] == S) limit[c] = s - 1;
            if (limit[c] == S) sum = next;
            end[(size_t)c * S + s] = (uint32_t)sum;
        }
        const uint2 mark = make_uint2((uint32_t)((top <= ORBG_MATCH_RANKS ? ORBG_MATCH_RANKS : ORBG_MM_RANKS) + 1) << 24, 0u);
        out->start[c] = (uint32_t)sets.size();
        sets.resize(sets.size() + ((size_t)sum + 63) / 64 * 64 + 128, mark);
        std::vector<uint32_t> at(S, 0u);
        for (int s = 1; s < S; ++s) at[s] = end[(size_t)c * S + s - 1];
        uint2* base = sets.data() + out->start[c];
        const int most = limit[c];
        uint8_t v[7];
        auto walk = [&](auto&& self, int depth, int from, int s) -> void {
            if (depth == c) {
                uint64_t e = 0;
                for (int i = 0; i < 7; ++i) e = (e << 8) | (i < c ? v[i] : 0u);
                e <<= 8;
                base[at[s]++] = make_uint2((uint32_t)(e >> 32), (uint32_t)e);
                return;
            }
            const int left = c - depth;                   // r, r + 1, ... is the least way on
            for (int r = from; r <= top && s + left * r + left * (left - 1) / 2 <= most; ++r) {
                v[depth] = (uint8_t)r;
                self(self, depth + 1, r + 1, s + r);
            }
        };
        walk(walk, 0, ORBG_LOW_RANKS + 1, 0);
    }
    out->start[0] = 0;
    void *d_sets = nullptr, *d_end = nullptr, *d_limit = nullptr;
    hipError_t e = hipMalloc(&d_sets, sets.size() * sizeof(uint2));
    if (e == hipSuccess) e = hipMalloc(&d_end, end.size() * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc(&d_limit, limit.size() * sizeof(int));
    if (e == hipSuccess) e = hipMemcpy(d_sets, sets.data(), sets.size() * sizeof(uint2), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d_end, end.data(), end.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(d_limit, limit.data(), limit.size() * sizeof(int), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(d_sets);
        (void)hipFree(d_end);
        (void)hipFree(d_limit);
        return e;
    }
    out->sets = (const uint2*)d_sets;
    out->end = (const uint32_t*)d_end;
    out->limit = (const int*)d_limit;
    return hipSuccess;
}

// The lists for length n; false where they cannot be made now (no memory, or
// the stream is being captured): mline_kernel then decodes every block.
bool get_sets(int n, hipStream_t stream, MlineSets* out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    // (widths as in mm_ranks)
    const int top = n < ORBG_MM_RANKS ? n : ORBG_MM_RANKS;
    std::lock_guard<std::mutex> lk(sets_mu);
    const auto it = sets_of.find({dev, top});
    if (it != sets_of.end()) { *out = it->second; return true; }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return false;
    MlineSets t = {};
    try {
        if (make_sets(top, &t) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        sets_of[{dev, top}] = t;
    } catch (const std::bad_alloc&) {
        return false;
    }
    *out = t;
    return true;
}

hipError_t launch_walk(const MlineArgs& a, int grid, hipStream_t stream)
{
    switch (a.mseg) {
    case 1: return launch_mline_m<1>(a, grid, stream);
    case 2: return launch_mline_m<2>(a, grid, stream);
    case 3: return launch_mline_m<3>(a, grid, stream);
    default: return launch_mline_m<4>(a, grid, stream);
    }
}

}  // namespace

// Small batches (up to ORBG_ML_SMALL blocks, n <= 256) go through the searches and the
// walk in one launch.  us, one launch / two: n = 127, two lines, 63 blocks 18.8 / 20.9,
// 1000 blocks 58.9 / 58.0; n = 256, three lines, 300 blocks 88.2 / 88.4, 1000 blocks
// 143.6 / 143.6; 1000 blocks of n = 64 at 9 dB 15.8 / 18.6.  But 2000 blocks of n = 64
// 26.0 / 22.4, and 16 blocks of n = 512, two lines, 63.7 / 54.5.
// Else the narrow search decodes nearly every block and mline_kernel those that it
// marks, in spans as short as give no more waves than its registers let the chip hold:
// a wave that only reads its flags costs its launch (8000 blocks of n = 256 at 9 dB,
// us: spans of one flag 29.5, of three 28.4), and one with many of the marked blocks
// keeps the others waiting (64 blocks of n = 512 that no search covers, two lines,
// 20000 queries: one span of 64 496 ms, of one 11.9; 8000 such blocks of n = 256, one
// line, 30000 queries: of three 5.7 ms, of eight 12.7).
#define ORBG_ML_SMALL 1024
hipError_t launch_mline(const MlineArgs& a, int grid, hipStream_t stream)
{
    if (a.nblocks <= 0) return hipSuccess;
    MlineArgs w = a;
    w.span = 0;
    if (!get_sets(a.n, stream, &w.sets)) return launch_walk(w, grid, stream);
    if (a.nblocks <= ORBG_ML_SMALL && a.n <= 4 * ORBG_WAVE) {
        if (a.n <= ORBG_WAVE) return launch_mline_all_nk<1>(w, (int)a.nblocks, stream);
        if (a.n <= 2 * ORBG_WAVE) return launch_mline_all_nk<2>(w, (int)a.nblocks, stream);
        return launch_mline_all_nk<4>(w, (int)a.nblocks, stream);
    }
    const int64_t most = a.n <= 4 * ORBG_WAVE ? 3 * 1024 : 2 * 1024;
    const int64_t span = (a.nblocks + most - 1) / most;
    w.span = span < ORBG_WAVE ? (int)span : ORBG_WAVE;
    const int64_t spans = (a.nblocks + w.span - 1) / w.span;
    hipError_t e;
    if (a.n <= ORBG_WAVE) e = launch_mline_match_nk<1>(w, grid, stream);
    else if (a.n <= 2 * ORBG_WAVE) e = launch_mline_match_nk<2>(w, grid, stream);
    else if (a.n <= 4 * ORBG_WAVE) e = launch_mline_match_nk<4>(w, grid, stream);
    else e = launch_mline_match_nk<8>(w, grid, stream);
    return e != hipSuccess ? e : launch_walk(w, (int)(spans < grid ? spans : grid), stream);
}

}  // namespace orbg
