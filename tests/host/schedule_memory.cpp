// Host driver of orbg_build_schedule without a device (test infrastructure): the
// HIP calls it makes are defined here, device memory is host memory, kernels do
// nothing, and one allocation of the driver's choice fails.  Where the schedule
// itself cannot be placed the call fails; where only the match-search tables
// cannot, it succeeds without them (decodes then go by steps of the order).
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <set>

#include "orbg_internal.h"

static int n_alloc, fail_at, last_error;
static std::set<void*> live;

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes)
{
    if (++n_alloc == fail_at) {
        *p = nullptr;
        return (hipError_t)(last_error = hipErrorOutOfMemory);
    }
    live.insert(*p = std::calloc(1, bytes));
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (p != nullptr && live.erase(p) == 0) std::abort();
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t bytes, hipMemcpyKind)
{
    std::memcpy(d, s, bytes);
    return hipSuccess;
}
// the two small read-backs: classes and weight of the last entry, ranks reached
hipError_t hipMemcpyAsync(void* d, const void*, size_t, hipMemcpyKind, hipStream_t)
{
    static_cast<int*>(d)[0] = 50;
    static_cast<int*>(d)[1] = 30;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return (hipError_t)e;
}
}

int main()
{
    for (fail_at = 0; fail_at <= 6; ++fail_at) {
        n_alloc = 0;
        orbg::Schedule s = {};
        char err[256] = {0};
        const int rc = orbg::orbg_build_schedule(64, 4096, nullptr, &s, err, sizeof(err));
        const int left = last_error;
        const bool whole = fail_at == 0, tables = fail_at >= 4;
        const size_t want_live = whole ? 4 : tables ? 1 : 0;    // entries, and the three tables
        const bool ok = rc == (whole || tables ? 0 : -2) && (s.match.sets != nullptr) == whole &&
                        (s.match.below != nullptr) == whole && (s.match.above != nullptr) == whole &&
                        live.size() == want_live && (!tables || left == 0);
        if (!ok) {
            std::fprintf(stderr, "allocation %d fails: rc %d, tables %d, %zu live, error left %d\n", fail_at, rc,
                         s.match.sets != nullptr, live.size(), left);
            return 1;
        }
        while (!live.empty()) (void)hipFree(*live.begin());
        last_error = 0;
    }
    std::printf("all checks passed\n");
    return 0;
}
