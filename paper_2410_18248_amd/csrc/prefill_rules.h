// In which order the tiles of a prefill launch that splits no context start: the arithmetic alone, the same on the host
// (where a test walks through it) and in the kernel.
#pragma once
#include "prefill_split.h"

namespace lamps {
namespace rules {

struct Turn {
    int pair, t;                         // of the pairs of an XCD; tiles behind the longest
};
// The place of an XCD's slot-th workgroup, of `pairs` x `tiles`, where `abreast` pairs go together: the longest tiles of all
// of them, the next ones, and so on.  The pairs of a level begin with another one every other level: an XCD's
// workgroups go to its four shader engines in turn, and where a level has as many pairs as that, or a multiple, each engine
// would get the tiles of the same requests all along and the launch end with the engine that has the longest (us, without /
// with: 4 prompts of 1 500 to 2 000, 32 / 8 heads of 128, one pair of each on an XCD, 142 / 115, of 3 000 to 4 000 468 / 400; 8 of
// 1 500 to 2 000 on 32 / 4 heads 256 / 223; 16 of 154 to 272 there 31.3 / 27.0; equal lengths level).  Divisions by reciprocal, for there are at
// most kMostDividend slots: two general ones are in front of the first byte of launches that take 6 us (30 fp32 prompts of 52 to 62
// tokens on 8 / 2 heads of 32: 6.17 us one by one, 6.60 with those, 6.28).
__host__ __device__ inline Turn abreast_at(int slot, int tiles, int pairs, int abreast)
{
    const int first = split::small_div(slot, abreast * tiles) * abreast, n = abreast < pairs - first ? abreast : pairs - first;
    const int t = split::small_div(slot - first * tiles, n);
    const int shift = n & 1 ? 0 : n & 2 ? t >> 1 & 1 : t & 3;
    const int k = slot - first * tiles - t * n + shift;
    return {first + (k < n ? k : k - n), t};
}

}  // namespace rules
}  // namespace lamps
