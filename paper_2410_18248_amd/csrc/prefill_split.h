// How a prefill launch that splits the contexts divides its work: the arithmetic alone, the same on the
// host (where a test walks through it) and in the kernel, where a wave holds one request per lane.
//
// The stages (32 cached positions) of every tile are cut into runs of `per` stages, each a workgroup
// of its own, an item.  `per` is the smallest that gives no more items than workgroups (slots), and at
// least kMinRun.
#pragma once
#include <stdint.h>

#ifndef __HIP__
#define __host__
#define __device__
#endif

namespace lamps {
namespace split {

constexpr int kMinRun = 12;              // stages: 384 positions (8 and 16 measured 0-4 % and 0-10 % slower)
struct Sums {
    int stages, tiles;                   // of all requests: stages x tiles, tiles
};
struct Piece {
    int head, run, tile;
};

__host__ __device__ inline float reciprocal(float x)
{
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.0f / x;
#endif
}

// a / b for 0 <= a < 2^19, 0 < b < 2^19: (a + 1/2) / b is at least 1 / 2 b away from a whole number, and
// two roundings and a reciprocal one unit off move it by less.  (A general division is 30 instructions
// in front of the first byte of every workgroup.)
__host__ __device__ inline int small_div(int a, int b) { return (int)(((float)a + 0.5f) * reciprocal((float)b)); }

// Tiles of wt new tokens a request of n_new has, at most `tiles` (tiles * wt below 2^18).
__host__ __device__ inline int tiles_of(int n_new, int wt, int tiles)
{
    return small_div((n_new < tiles * wt ? n_new : tiles * wt) + wt - 1, wt);
}

// Stages of a run.  head_slots: slots per kv head.
__host__ __device__ inline int run_length(const Sums &s, int head_slots)
{
    // a tile's last run may be short: the sum over tiles of ceil(stages / per) stays within the slots
    const int spare = head_slots - s.tiles > 1 ? head_slots - s.tiles : 1;
    if (s.stages <= (long long)kMinRun * spare) return kMinRun;
    return (int)(((unsigned)s.stages + (unsigned)spare - 1) / (unsigned)spare);
}

// Runs of a request whose last tile has so many stages (earlier ones have as many or fewer).
__host__ __device__ inline int runs_of(int stages, int per, int slots)
{
    const int n = (int)(((unsigned)stages + (unsigned)per - 1) / (unsigned)per);
    return n < slots ? n : slots;
}

// The item of workgroup `block` of `slots`, or -1.  Each XCD takes an eighth of the items there are, in
// order (workgroups are dealt to the XCDs in turn): neighbours share blocks, and every XCD has work
// however few items there are.  (With an eighth of the slots each, 64 items were all on one XCD: one
// request of 500 new on 32 / 8 heads of 128 took 32 us, 23 on all of them.)
__host__ __device__ inline int item_of(int block, int items, int slots)
{
    const int eighth = (items + 7) >> 3, each = eighth < slots >> 3 ? eighth : slots >> 3;
    return (block >> 3) < each ? (block & 7) * each + (block >> 3) : -1;
}

// Item x of a request's, ordered (kv head, run, tile).  The runs that earlier tiles do not have are
// spread over all heads, and with them over the XCDs.
__host__ __device__ inline Piece piece_of(int x, int tiles, int runs)
{
    Piece p;
    const int strip = small_div(x, tiles);
    p.head = small_div(strip, runs);
    p.run = strip - p.head * runs;
    p.tile = x - strip * tiles;
    return p;
}

}  // namespace split
}  // namespace lamps
