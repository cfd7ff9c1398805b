// How a prefill launch that splits the contexts divides its work: the arithmetic alone, the same on the
// host (where a test walks through it) and in the kernel, where a wave holds one request per lane.
//
// The stages (32 cached positions) of every tile are cut into runs of `per` stages, each a workgroup
// of its own, an item.  `per` is the smallest that gives no more items than workgroups (slots); but a
// run is at least kMinRun stages, and a request is cut only where that pays for the hand-over.
#pragma once
#include <stdint.h>

#ifndef __HIP__
#define __host__
#define __device__
#endif

namespace lamps {
namespace split {

constexpr int kMinRun = 12;              // stages: 384 positions (8 and 16 measured 0-4 % and 0-10 % slower)
// A request is cut where its tiles are longer than a run by more than this: what the hand-over costs.
// (One request of 100 new on 700 cached, 24 stages, 32 / 8 heads of 128: 16.3 us cut, 19.0 not; with 12
// in place of 6, twelve requests of 4 to 64 new on 300 to 2 500: 35.4 us, 32.7 with 6.)
constexpr int kMargin = 6;

struct Sums {
    int stages, tiles, most;             // of all requests: stages x tiles, tiles; the most stages of one
};
struct Cut {
    int per, worth;                      // stages of a run; requests with more stages than `worth` are cut
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

constexpr int kMostDividend = 1 << 19;
// a / b for 0 <= a < 2^19, 0 < b < 2^19: (a + 1/2) / b is at least 1 / 2 b away from a whole number, and
// two roundings and a reciprocal one unit off move it by less.  (A general division is 30 instructions
// in front of the first byte of every workgroup.)
__host__ __device__ inline int small_div(int a, int b) { return (int)(((float)a + 0.5f) * reciprocal((float)b)); }

// Tiles of wt new tokens a request of n_new has, at most `tiles` (tiles * wt below 2^18).
__host__ __device__ inline int tiles_of(int n_new, int wt, int tiles)
{
    return small_div((n_new < tiles * wt ? n_new : tiles * wt) + wt - 1, wt);
}

// head_slots: slots per kv head.  group: stages a workgroup loads at a time.  wide: tiles of 128 columns
// or of head size 256, whose items are 64 KiB and more and of which two hinder each other on a CU.
__host__ __device__ inline Cut cut_of(const Sums &s, int head_slots, int heads, int group, int head_dim, bool wide)
{
    // a tile's last run may be short: the sum over tiles of ceil(stages / per) stays within the slots
    const int spare = head_slots - s.tiles > 1 ? head_slots - s.tiles : 1;
    Cut c;
    c.per = kMinRun;
    if (s.stages > (long long)kMinRun * spare) c.per = (int)(((unsigned)s.stages + (unsigned)spare - 1) / (unsigned)spare);
    c.per = (c.per + group - 1) / group * group;      // whole groups
    c.worth = c.per + kMargin;
    if (wide) {
        // Cut, the launch takes as long as a run or as all the work on 256 CUs, and the hand-over: 6 stages,
        // and one more for every 24 items that go through memory (48 of head size 256, whose stages take
        // longer).  If its longest request takes no longer as it is, nothing is cut.  (One request, new on
        // cached, us as it is / cut: 400 on 600, 32 / 8 heads of 128: 29.6 / 29.5; 260 on 600: 26.9 / 22.5;
        // 900 on none, 16 / 1 heads: 26.8 / 32.7; 16 heads of 256, 500 on none: 19.5 / 20.7; 400 on 700:
        // 34.0 / 32.7; 900 on 700: 48.7 / 62.2; 700 on 3 000: 97 / 84.)
        const float work = 2.0f * (float)s.stages * reciprocal((float)head_slots);
        const float items = ((float)s.stages * reciprocal((float)c.per) + 0.5f * (float)s.tiles) * (float)heads;
        float least = (work > (float)c.per ? work : (float)c.per) + 6.0f + items * (head_dim >= 256 ? 1.0f / 48 : 1.0f / 24);
        if (least < 20.0f) least = 20.0f;
        if ((float)s.most <= least) c.worth = s.most;
    }
    return c;
}

// Runs of a request whose last tile has so many stages (earlier ones have as many or fewer).
__host__ __device__ inline int runs_of(int stages, const Cut &c, int slots)
{
    if (stages <= c.worth) return 1;
    const int n = (int)(((unsigned)stages + (unsigned)c.per - 1) / (unsigned)c.per);
    return n < slots ? n : slots;
}

// The item of workgroup `block` of `slots`, or -1.  Each XCD takes an eighth of the items there are, in
// order (workgroups are dealt to the XCDs in turn): neighbours share blocks, and every XCD has work
// however few items there are.  (With an eighth of the slots each, 64 items were all on one XCD: one
// request of 500 new on 32 / 8 heads of 128 took 32 us, 22 on all of them, cut alike.)
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
