// Finding the request a workgroup works for.  Device code; include from a .hip file only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lamps {
namespace {

// The last request r < batch with key(q_start[r], r) <= x; key grows with r.  By every wave, 64
// requests per round trip to memory (one by one halving, each round waits for the one before: 4 to 6
// of them were half the time of a call with few tokens).
template <typename Key>
__device__ __forceinline__ int last_request(const int32_t *q_start, int batch, int x, Key key)
{
    const int lane = threadIdx.x & 63;
    int lo = 0, n = batch;                            // it is one of lo .. lo + n - 1 (or lo, if none is)
    while (n > 1) {
        const int step = (n + 63) >> 6, r = lo + lane * step;
        const unsigned long long le = __ballot(lane * step < n && key(q_start[min(r, batch - 1)], r) <= x);
        const int at = max(0, 63 - __clzll((long long)le)) * step;     // (none: clz 64)
        lo += at;
        n = min(step, n - at);
    }
    return lo;
}

// The same one by one, by scalar loads, which come sooner: for a few requests.
constexpr int kFew = 16;
template <typename Key>
__device__ __forceinline__ int last_of_few(const int32_t *q_start, int batch, int x, Key key)
{
    int lo = 0, hi = batch;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (key(q_start[mid], mid) <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Where a token form's workgroup works: a request, the row of its first new token, how many of them it has, its context's length.
struct NewTokens {
    int r, first, count, ctx;
};
// That of the last request with key(q_start[r], r) <= x, by every wave.  Up to 64 requests in one round trip: each lane asks for all of one request, and
// the wave takes its request's out of the registers.
template <typename Key>
__device__ __forceinline__ NewTokens new_tokens_at(const int32_t *q_start, const int32_t *ctx_lens, int batch, int x, Key key)
{
    if (batch > 64) {
        const int r = last_request(q_start, batch, x, key), first = q_start[r];
        return {r, first, q_start[r + 1] - first, ctx_lens[r]};
    }
    const int lane = threadIdx.x & 63, i = min(lane, batch - 1);
    const int first = q_start[i], next = q_start[i + 1], ctx = ctx_lens[i];
    const unsigned long long le = __ballot(lane < batch && key(first, lane) <= x);
    const int r = max(0, 63 - __clzll((long long)le));     // (none: clz 64)
    const int from = __builtin_amdgcn_readlane(first, r);
    return {r, from, __builtin_amdgcn_readlane(next, r) - from, __builtin_amdgcn_readlane(ctx, r)};
}

}  // namespace
}  // namespace lamps
