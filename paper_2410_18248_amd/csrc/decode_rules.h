// Which form a decode launch takes, by what the host knows of it: the ranges, (request, kv head / pass), there can be, and the longest a context
// can be, a table row, in rounds: the chunks that one of four waves walks through.  Lengths and masks are on the device; the forms of longer walks
// look at them there, by the arithmetic at the end, which is the same on the host (where a test walks through it) and in the kernels.
#pragma once
#include <stddef.h>

#include "prefill_split.h"

namespace lamps {
namespace rules {

struct DecodeLaunch {
    long long ranges;
    int batch, head_dim;
    long long row;                       // positions of a table row
    int round;                           // positions of a round: four chunks
    bool matrix;                         // MfmaReducer (else ValuReducer)
    bool bounded;                        // a row has no more blocks than the pool
    size_t state;                        // bytes of a range's (outputs, maximum, sum)
    size_t capacity;                     // bytes of partial states a launch may leave behind
};
enum DecodeForm { kPlan, kWholeTwo, kWholeFour, kWholeEight, kCut, kParts };

constexpr int kMostCuts = 64;            // parts of a range in a kParts launch
constexpr int kPartBatch = 64;           // requests of one, a lane's each
constexpr int kCutBatch = 256;           // requests that a wave of a kCut launch can hold
constexpr long long kMostItems = 1 << 19;   // workgroups of one (its divisions, and 64 rounds of chunks for each, 256 for few, in 32 bits)

// Workgroups of a kCut launch beyond one for each range: about what the chip holds at once, so that a launch in which much is cut is cut
// evenly (512 / 1 024, time over the plan's, vector path: 512 to 1 024 ranges, 8 to 32 rounds 0.95 / 0.92, the slowest 1.22 / 1.08; 2 048 and more
// 0.93 / 0.93, 1.32 / 1.10; matrix path, 256 to 512 ranges, 8 to 64 rounds 0.71 / 0.80, 1.06 / 1.05).
constexpr int cut_spare(bool matrix) { return matrix ? 512 : 1024; }

// All lines below are drawn through launches of which two thirds are skewed: one long context among short ones, a few, 2 to 60 % of the
// requests running, or rows of 4 and 16 times the longest; 12 000 launches of 1 to 700 requests with rows of 17 to 65 536 positions, as many again with
// each form in turn.  Figures are time over the plan's (decode_balanced and its second launch), geometric mean and slowest.

// Parts of a range if all are alike, each a workgroup's (decode_parts); 0: not this way.  For few ranges of longer rows, where the plan and the
// records of decode_balanced are a third of the time:
//   vector path, fewer than 16 ranges, 4 to 400 rounds 0.85, 0.99 (to 1 024 0.95, 1.28; fewer than 4 1.06, 1.36);  16 to 32, 4 to 64 0.83, 0.94;  32 to 64, 4 to 32
//      0.84, 0.97;  64 to 128, 4 to 16 0.87, 0.99;  16 to 128 on longer rows, to 400 0.90, 1.13, to 1 024 0.94, 1.24 (all contexts long 0.99, 1.11)
//   matrix path, fewer than 16 ranges, 8 to 400 rounds 0.77, 0.94;  16 to 32, 8 to 128 0.79, 0.96, to 400 0.82, 0.97;  32 to 64, 8 to 32 0.80, 0.92;  all of them 401 to
//      1 024 0.88, 1.17 (all contexts long 0.89, 1.00; more rounds 0.93, 1.43 and 0.96);  64 to 96, 16 to 32 0.85, 1.02 (to 128 0.93, 1.26; 96 to 128 0.96, 1.07)
// (With the same number of parts for every range there can be: a context among 11 of 32 ranges, or 2 of 29 requests running, took up to 1.6 times the
// plan's time.  Rows longer than the contexts, a server's, are those of the contexts: one request of 1 999 tokens, 32 / 8 heads, 7.0 to 7.5 us with any row to 32 768, the plan 9.1.)
// Workgroups in all 256, or 512 where rows are long for them (256 / 512 / 1 024, even batches: vector path, fewer than 16 ranges, 4 to 64 rounds 0.86 / 0.89 /
// 0.89, more 0.93 / 0.87 / 0.87; 16 to 32 ranges to 16 rounds 0.85 / 0.86 / 0.90; 32 to 64 0.92 / 0.87 / 0.90; 16 to 64, 65 to 1 024 rounds 0.97 / 0.91; matrix path, fewer than 32, 8 to 128
// rounds 0.79 / 0.84 / 0.86; 32 to 64 0.89 / 0.89 / 0.96; fewer than 64 with more rounds 0.86 / 0.89; 64 to 128, 16 to 32 rounds, 0.91 / 0.87 / 0.91).
inline int decode_most_cuts(const DecodeLaunch &l)   // of one range, where others are shorter
{
    const long long room = (long long)(l.capacity / l.state) / l.ranges;
    return room < kMostCuts ? (int)room : kMostCuts;
}
inline int decode_cuts(const DecodeLaunch &l)
{
    if (!l.bounded || l.ranges >= 128 || l.batch > kPartBatch) return 0;
    if ((l.row / l.round + 1) * 8 * l.batch + (1 << 12) >= split::kMostDividend) return 0;   // (half-chunks of all requests, and what is added to round up)
    const auto rounds_to = [&l](int n) { return l.row <= (long long)n * l.round; };
    const int most = l.matrix ? (l.ranges < 64 ? 1024 : l.ranges < 96 ? 32 : 0) : l.ranges < 4 ? 400 : 1024;
    const int least = l.matrix ? (l.ranges >= 64 ? 16 : l.head_dim < 128 ? 12 : l.head_dim < 256 ? 8 : 5) : 4;
    if (rounds_to(least) || !rounds_to(most)) return 0;
    const bool few = l.matrix ? l.ranges < 64 : l.ranges < (rounds_to(16) ? 32 : rounds_to(64) ? 16 : 0);
    const int share = (few ? 256 : 512) / (int)l.ranges, cuts = share < kMostCuts ? share : kMostCuts;
    return cuts <= decode_most_cuts(l) ? cuts : 0;
}

inline DecodeForm decode_form(const DecodeLaunch &l)
{
    const long long n = l.ranges;
    // (a row of more blocks than the pool has is sized for requests that are not there: left to the plan, which goes by the lengths alone)
    if (!l.bounded || n > 0x7fffffff / 256) return kPlan;
    const auto rounds_to = [&l](int k) { return l.row <= (long long)k * l.round; };
    const bool sorts = l.batch <= kCutBatch && n + cut_spare(l.matrix) < kMostItems && (size_t)(n + cut_spare(l.matrix)) * (l.state + 8) <= l.capacity;
    const bool eight = 8 * l.state <= (80u << 10);    // of the LDS: two workgroups to a CU
    if (decode_cuts(l) > 0) return kParts;
    // Ranges that are short: by two waves where there are thousands of a round (1 024 and more, two / four: vector path 0.62, 0.86 / 0.65, 0.97;
    // 4 096 and more 0.79, 1.10 / 0.95, 1.32; matrix path 0.57 / 0.65), or of a few.  A waiting request's workgroups leave at once, but there are tens of
    // thousands of them: 565 requests of 161 positions at most, 40 heads, 18 of them running, 18.4 us by the plan and 20.7.
    if (rounds_to(1)) return n >= 1024 ? kWholeTwo : kWholeFour;
    if (l.matrix) {
        if (n >= (rounds_to(3) ? 1024 : 4096) && rounds_to(12)) return kWholeTwo;   // 4 096 and more, 4 to 12 rounds, two / four 0.69, 1.22 / 0.73, 1.32
        // Heads of 256: a walk is as much longer as a chunk has products.  By four waves / eight / in parts of 256 workgroups: fewer than 64 ranges, to 4
        // rounds 0.67, 0.97 / 0.69, 0.93 / 0.92, 1.14; 5 0.75, 1.15 / 0.76, 1.11 / 0.92, 1.01; 6 to 12 0.94, 1.90 / 0.91, 1.76 / 0.89, 1.08.  64 to 128, 5 to
        // 9 rounds 0.82, 1.43 / 0.82, 1.31, to 12 0.97, 1.91 / 0.95, 1.73: the plan.  128 to 256, to 10 rounds 0.56, 1.45 / 0.57, 1.30; 11 to 16 0.69, 1.99 /
        // 0.68, 1.81, cut by the lengths 0.66, 1.30; 256 to 1 024, 11 and 12, 0.77, 1.61 / cut 0.76, 1.39
        const bool wide = l.head_dim >= 256;
        if (wide && n < 128 && !rounds_to(9)) return kPlan;
        if (wide && n < 1024 && !rounds_to(10) && rounds_to(16) && sorts) return kCut;
        // to 12 rounds, any number of requests, 0.38 to 0.80, 1.11; fewer than 256 from 8 on by eight waves (0.80, by four 0.85), 64 and more to 16
        // (0.83; with one long context among a dozen of 20 to 100 positions up to 1.25, 10.6 us against 8.5)
        if (rounds_to(12)) return n < 256 && eight && !rounds_to(wide ? 4 : 8) ? kWholeEight : kWholeFour;
        if (n < 256) return n >= 64 && eight && rounds_to(16) ? kWholeEight : kPlan;
        // 256 to 512 ranges, to 32 rounds 0.67, 1.38 (to 128 0.84, but all contexts alike up to 1.17: 258 ranges of 8 500 tokens 91 us, and 106 by twice as many halves on 512
        // places); 512 to 4 096, 13 to 64 0.75, 1.39, to 256 0.85, 1.36 (all contexts long 0.92, 1.15; more 0.97, 2.36 and 1.07).  The slowest have 2 to 15 % of their requests
        // running.  Whole by eight waves or longest first, without a look at the work: to 64 rounds 0.87, 1.21 and 0.94, 1.65
        return rounds_to(n < 512 ? 32 : n < 4096 ? 256 : 64) && sorts ? kCut : kPlan;
    }
    // 2 and 3 rounds, up to 4 096 ranges, by four waves / two 0.67, 1.18 / 0.69, 1.10; more 0.74, 1.73 / 0.72, 1.49 (the slowest have contexts of 2 to 10 % of the
    // row; without one range's waves taking the other's place, 0.75, 1.84: few of thousands of requests running)
    if (rounds_to(3)) return n < 4096 ? kWholeFour : kWholeTwo;
    if (l.batch > kCutBatch) return !rounds_to(6) ? kPlan : n < 8192 ? kWholeFour : kWholeTwo;   // 0.60, 1.13; two / four 0.70, 1.36 / 0.73, 1.37 (more than 6 rounds 0.89 to 1.09, 2.66)
    // to 4 by eight waves 0.78, 0.91 (by four 0.91, 1.14); more by either 0.91 to 0.97, 1.07 to 1.41
    if (n < 256) return rounds_to(4) ? kWholeEight : kPlan;
    // 256 to 512 ranges, to 16 rounds 0.84, 1.13, to 32 0.92, 1.23 (all contexts long 0.97; more 0.95, 1.22 and 1.03); 512 to 4 096, to 32 0.84, 1.23, to 128 0.92, 1.32
    // (1.00; more 0.99, 1.37 and 1.05; of 2 048 and more with contexts of a few tokens, which the plan puts several of into a share, 1.42); more ranges, to 8 rounds 0.97,
    // 1.30.  A row that is sized for a server's longest possible request is most often much longer than the contexts, whose lengths are all that the launch goes by:
    // 4 layers of append + decode of 16 requests of 60 to 1 500 tokens, 40 heads, take 91 us with any row to here, 103 by the plan.  The slowest have 2 to 15 % of
    // their requests running and take 8 to 16 us.  Whole by eight waves or longest first, without a look at the work: 0.97 to 1.03, 1.5 to 2.2
    return n < 4096 && rounds_to(n < 512 || n >= 2048 ? 32 : 128) && sorts ? kCut : kPlan;
}

// A kCut launch: chunks of a part, and those of a range that is not worth cutting.  An even share of all chunks there are over the spare workgroups, so
// that these are enough for all parts beyond the first of their ranges; two rounds at least.  What is up to half as long again is not worth the
// hand-over (up to two rounds longer: 16 requests of 60 to 1 500 tokens, 40 heads, 23.7 us and 24.8).  round: chunks of four waves.
struct CutSize {
    int size, worth;
};
__host__ __device__ inline CutSize cut_size(unsigned all, int spare, int round)
{
    const int even = (int)(all / (unsigned)spare) + 1, least = even > 2 * round ? even : 2 * round;
    const int size = (least + round - 1) / round * round;
    return CutSize{size, size + size / 2};
}
__host__ __device__ inline int cut_parts(int n, CutSize c) { return n > c.worth ? split::small_div(n + c.size - 1, c.size) : 0; }
// Chunks of each part of a range that is cut into so many: whole chunks of a wave.
__host__ __device__ inline int cut_each(int n, int parts, int chunk) { return (split::small_div(n + parts - 1, parts) + chunk - 1) / chunk * chunk; }

// A kParts launch: chunks of a part, the fewest (a chunk per wave at least) that give no more parts than `even` for each request there can be and one
// for each that runs, and no range more than `most`.  chunk: of a wave, one or two.  From there the waves go up by a chunk while there are more parts
// than `even` for each request, so many times at most: a part of a chunk or two beyond what the chip holds at once waits for the first to end (25
// requests of 5 298 tokens and up to 60 fewer, 32 / 2 heads of 128, 34.8 us, 26.7 so; 36 of 1 697 19.8 and 17.0).
constexpr int kPartTries = 8;
__host__ __device__ inline int part_size(int sum, int longest, int batch, int even, int most, int waves, int chunk)
{
    const int all = even * batch, share = split::small_div(sum + all - 1, all), room = split::small_div(longest + most - 1, most);
    int size = waves * chunk > share ? waves * chunk : share;
    size = size > room ? size : room;
    return (size + chunk - 1) & -chunk;
}

}  // namespace rules
}  // namespace lamps
