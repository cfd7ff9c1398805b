// How the workgroups of one launch that share a sum hand it over: the last to arrive adds up what the others left in memory.
// Device code; include from a .hip file only.
#pragma once
#include <hip/hip_runtime.h>

namespace lamps {
namespace {

// The hand-over between the runs of a tile goes through memory that every XCD sees alike:
// agent-scope accesses, relaxed; the writer waits for its stores before it reports.  (A release or
// acquire fence would write back or invalidate a whole L2.)
__device__ __forceinline__ void put_shared(float *p, float x, float y)
{
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, make_float2(x, y)), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 get_shared(const float *p)
{
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}
// Reports one run of a tile of `total` runs, whose words are `stride` apart from `first` on; true for the last.  By a whole wave.
// The words count only with the launch's own tag, so whatever the memory held before is nothing, and are taken away by the
// last run, for the launch may be replayed with the same tag.
//
// MANY: for tiles of 64 columns (contexts under wider ones are cut into few runs).  Up to four runs are counted in the first
// word, (tag, reports so far), by compare-and-swap: each failure is another run's report.  More of them, that end together,
// would take a round trip each (2 new tokens on 8 000 cached, 32 / 8 heads: 33.4 us, 24.4 with flags; 16 on 3 000 25.5 and 24.1; with
// flags for all, a dozen responses 30.3, 29.6 so): there each run sets its own word, waits until that has arrived, and looks at
// the others.  The last to arrive finds them all; of those that do at the same time the one that takes the first word away
// is the one.
template <bool MANY>
__device__ __forceinline__ bool report_run(uint64_t *first, int stride, int mine, int total, uint64_t tag)
{
    const int lane = threadIdx.x & 63;
    int last = 0;
    if (!MANY || total <= 4) {
        if (lane == 0) {
            uint64_t old = 0;                         // (a guess, most often right for the first)
            for (;;) {
                const int n = (old >> 16) == tag ? (int)(old & 0xFFFF) + 1 : 1;
                const uint64_t want = n == total ? 0 : (tag << 16) + (uint64_t)n;
                if (__hip_atomic_compare_exchange_strong(first, &old, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    last = n == total;
                    break;
                }
            }
        }
    } else {
        if (lane == 0) {                              // (an exchange: what it returns has been where all XCDs look)
            const uint64_t was = __hip_atomic_exchange(first + (size_t)mine * stride, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::"v"((uint32_t)was) : "memory");
        }
        bool all = true;
        for (int k = lane; k < total; k += 64)
            all = all && __hip_atomic_load(first + (size_t)k * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
        if (__all(all)) {
            if (lane == 0) last = __hip_atomic_exchange(first, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
            for (int k = lane; k < total; k += 64)
                if (k > 0) __hip_atomic_store(first + (size_t)k * stride, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    return __builtin_amdgcn_readfirstlane(last) != 0;
}

}  // namespace
}  // namespace lamps
