// Kernel launchers of liborbgrand (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define ORBG_MAX_CODES 8       // codes one launch may mix
#define ORBG_MATCH_M 9         // check bits from which an ordered search rarely ends in its first steps
#define ORBG_MIXED_COLS 2048   // packed columns of all codes of a mixed launch (sum of n)

namespace orbg {

// One code of a launch (device pointers into the library's caches).
struct CodeDesc {
    int n;                     // code length
    int m;                     // n - k
    int nk;                    // keys per lane of the rank sort: power of two >= n / 64
    int rdepth;                // ranks whose columns are staged (<= 255)
    int rdepth0;               // ranks the first batch of 64 entries reaches
    uint32_t slen;             // schedule entries
    uint32_t col_base;         // first column of this code in the launch's LDS column table
    uint32_t row_base;         // first word of this code's rows in the launch's LDS row table
    const uint64_t* cols;      // n packed parity-check columns
    const uint64_t* rows;      // m x nk packed parity-check rows (bit l of word j = H[r][64 j + l])
    const uint2* sched;        // schedule entries for this n (1-line: the schedule of offset -1)
    const uint2* sets;         // match search: sets of ranks above 8, or nullptr (step search only)
    const uint32_t* below;     // match search: count tables (MatchTable)
    const uint32_t* above;
    int wprefix;               // match search: logistic weight of query 4096
    int wlim;                  // match search: logistic weight of the last query within the budget
    int j0max;                 // 1-line: largest offset with a schedule of its own
    uint32_t sstride;          // 1-line: entries between the schedules of consecutive offsets
};

struct CodeTable {
    int ncodes;
    int rwords;                // row words of all codes (LDS row table size)
    CodeDesc c[ORBG_MAX_CODES];
};

// Launch shape (the autotuner's knobs) of the search by steps.
struct LaunchParams {
    int wg_per_cu;             // light pass: one-wave workgroups per compute unit
    int chunk;                 // blocks per work-counter increment (0 = about 16 per wave)
    int split_steps;           // light pass stops a block after this many 64-query steps (0 = never)
    int heavy_waves;           // waves that share one heavy block (4, 8 or 16)
    int heavy_wg_per_cu;       // heavy pass: workgroups per compute unit
    int naive;                 // 1: one one-wave workgroup per block, no work counter, no heavy pass
};

struct DecodeArgs {
    CodeTable codes;
    bool mixed;                // per-block code index and row offsets given
    const uint8_t* block_code; // device, nblocks (mixed)
    const int64_t* row_off;    // device, nblocks: element offset of the row in llr and codeword (mixed)
    int64_t row_limit;         // mixed: rows must end within this many elements of llr and codeword
    const float* llr;
    int64_t nblocks;
    uint32_t budget;
    const uint8_t* order;      // device, nblocks x 64, or nullptr for plain order
    bool oneline;              // 1-line ORBGRAND order (one code, plain batch order)
    int32_t* j0;               // device, nblocks 1-line offsets, or nullptr
    uint8_t* cw;
    uint64_t* queries;
    uint8_t* abandoned;
    unsigned long long* ctrs;  // device work counters (8 slices, heavy count, heavy next)
    int64_t* heavy;            // device heavy-block list, capacity >= nblocks when splitting
    bool list_only;            // blocks left after split_steps are only listed (no heavy pass):
    int64_t* list;             // in list (room for nblocks), their number in the heavy-block counter
    const int64_t* ids;        // device, nblocks: caller's block index of each position, or nullptr
                               // (one code, no heavy pass; the batch order stays per position)
    bool skip0;                // ordered decode of blocks known to hold no member in batch 0:
                               // the search starts at step 1
    int cus;                   // compute units of the device
    LaunchParams p;
};

// Work slices of the light pass (8 per XCD), their stripe length in chunks, and
// the counter slots (u64 index, each on its own 128-byte line).
#define ORBG_SLICES 64
#define ORBG_STRIPE 64
#define ORBG_CTR_SLICE(x) ((x) * 16)
#define ORBG_CTR_HEAVY_COUNT (ORBG_SLICES * 16)
#define ORBG_CTR_HEAVY_NEXT ((ORBG_SLICES + 1) * 16)
#define ORBG_CTR_WORDS ((ORBG_SLICES + 2) * 16)

hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream);

// A block left by a pass for the next one has this abandon flag in between.
#define ORBG_OPEN 2

// The match search decodes every code that has its tables, but not the 1-line
// order, nor where the first batch alone or the naive launch is asked for; with
// a batch order it takes codes of ORBG_MATCH_M check bits or more (with fewer,
// 4096 patterns hold many members, and the first steps of the order find one:
// 30000 blocks of n = 64 at 4 dB, us with the match search / by steps: m = 8
// 131 / 100, m = 9 82 / 104, m = 10 60 / 109, m = 12 40 / 121).
inline bool many_checks(const DecodeArgs& a)
{
    for (int i = 0; i < a.codes.ncodes; ++i)
        if (a.codes.c[i].m < ORBG_MATCH_M) return false;
    return true;
}
inline bool uses_match(const DecodeArgs& a)
{
    if (a.oneline || a.list_only || a.p.naive) return false;
    for (int i = 0; i < a.codes.ncodes; ++i)
        if (a.codes.c[i].sets == nullptr) return false;
    return a.order == nullptr || many_checks(a);
}

}  // namespace orbg
