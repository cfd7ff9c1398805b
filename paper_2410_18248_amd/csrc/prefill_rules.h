// How wide the tiles of a prefill launch that splits no context are, and in which order they start: the arithmetic alone, the
// same on the host (where a test walks through it) and in the kernel.
#pragma once
#include "prefill_split.h"

namespace lamps {
namespace rules {

struct Launch {
    int heads, group, head_dim, batch, total, most;   // heads: kv heads, of fp32 tiles passes over them; total, most: new tokens
    long long row;                       // positions
};

struct Turn {
    int pair, t, slot;                   // t: tiles behind the longest
};
// The place of an XCD's slot-th workgroup, of `pairs` x `tiles`, where `abreast` pairs go together: the longest tiles of all
// of them, the next ones, and so on.  Which pair a level begins with changes from level to level: an XCD's workgroups go to
// its four shader engines in turn, and where a level has four pairs or a multiple (an even number: every other level), each
// engine would get the tiles of the same requests all along, and the launch end with the one that has the longest (us, without /
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
    return {first + (k < n ? k : k - n), t, slot};
}
// A workgroup's pair and tile in a grid of `pairs` x `tiles`: groups of 8 pairs, one on each XCD, whose place among those is `slot`; the
// pairs left over, -1, are dealt round-robin over the XCDs -- in front of pairs that go abreast, which end with their short
// tiles (behind them, us attention alone, one by one / abreast / in front: 9 prompts of 599 to 665 on 32 / 4 heads of 128 62.3 / 65.6 / 54.5; 9 of
// 1 714 to 1 769 on 8 / 2 heads of 64 58.6 / 60.7 / 43.8; 7 of 1 000 on 20 heads of 128 83.5 / 81.2 / 63.3).
__host__ __device__ inline Turn deal(int block, int pairs, int groups, int tiles, int abreast)
{
    const int xcd = block & 7, rest = pairs - 8 * groups, ahead = abreast > 1 ? (rest * tiles + 7) >> 3 : 0;
    const int slot = (block >> 3) - ahead;
    if (slot >= 0 && slot < groups * tiles) {
        if (abreast <= 1) return {xcd + 8 * (slot / tiles), slot % tiles, slot};
        const Turn turn = abreast_at(slot, tiles, groups, abreast);
        return {xcd + 8 * turn.pair, turn.t, slot};
    }
    const int i = (abreast > 1 ? block >> 3 : slot - groups * tiles) * 8 + xcd;   // (rest is 1..7: the grid has no such slots otherwise)
    return {8 * groups + i % rest, i / rest, -1};
}

// Pairs of an XCD (of the `groups` it has) whose tiles are dealt together, the longest of all of them first.  One pair after
// the other, a launch ends with the long tiles of its last pairs while most of the chip has nothing left; all together,
// their K / V streams no longer share an L2.  So they go together in even parts of up to 20 MB (head size 256, whose tiles of 64
// columns read each byte twice as often: 10), for the longest context; not where the chip holds the launch at once, nor where many
// workgroups have no tile (6 fp32 prompts of 20 to 428 tokens: 14.5 us, 15.4: those that have one land on half of the CUs).
// us, append included, one by one / in parts of 4 / 8 or 10 / all: 4 prompts of 1 000, 32 heads of 128 (16 pairs an XCD, 8 MB) 100.9 /
// 84.6 / 80.7 / 79.0; 4 of 2 048, 40 heads (20 MB) 302 / 271 / 276 / 264; 4 of 4 096 (40 MB) 884 / 830 / 840 / 914; one (5 pairs)
// 255 / 271 (the last one alone) / - / 214; 8 of 500 on 4 000 cached, 32 heads (72 MB) 343 / 340 / 344 / 396; 8 of 1 900, 8 heads of
// 64, 76.0 / 71.3 / 60.9; 4 of 4 000, 16 heads of 256 (32 MB), 715 / 729 (in parts of 2: 714) / 758; 4 of 2 000 238 / 222 / 226.
// Nor over cached positions of more than twice what is new, of as much where a pair's neighbours are another request's:
// there a tile's place says less of its length, and the last tiles of the longest contexts end the launch (attention alone, one
// by one / abreast: 16 requests of 500 on 675 to 2 250, 8 fp32 heads of 64, 251 / 322; 10 of 200 on 270 to 900, 32 heads of 128, 47.4 / 52.1; 16 of
// 500 on 450 to 1 500, 32 / 8 heads, 188 / 213; 10 of 500 on 225 to 750 there 87 / 82, 32 / 4 heads 81 / 88) -- but if a request has only
// a few tiles and many have fewer: the workgroups without one would be all through the launch (10 of 100 to 250 on 340 to 1 125,
// 32 heads of 128, 58.3 / 47.3; 16 there, heads of 64, 46.1 / 34.0).
// Nor up to three tiles of requests that have about as many each: there is next to no tail to fill, and one by one a pair's tiles read
// its K / V at the same time (27 prompts of 300 to 362, 32 heads of 128, 80.7 / 93.3; 16 of 200 there, row of 300, 34.7 / 36.2; but 4 tiles, 16 of
// 500, 115 / 103).
// The host knows the longest context by its bound, the length of a table row.  Where that rules nothing out it decides; where it does, a
// server's rows may be as long as its longest possible request, and the workgroups look at the contexts themselves (a load per lane, so up
// to 64 requests; 0.2 to 0.5 us in front of everything, so from 128 new tokens on).  Row of 4 096, by the row / by the contexts: 4 prompts of 1 000 on 32
// heads 99.4 / 79.0; row of 32 768: 4 of 2 048 on 40 heads 302 / 269, one of 4 096 256 / 216, 8 of 1 900 on 8 heads of 64 80.6 / 64.6; contexts that rule it
// out level.
struct Together {
    int longest;                         // pairs go abreast over contexts up to this long, in positions; 0: not at all
    int part;                            // in parts of this many positions of all of an XCD's pairs
};
// grid: pairs x tiles; there_are: tiles the requests can have, at most; chip: workgroups that it holds at once.  bytes: of a cached element, keys and values.
inline Together together(const Launch &l, int bytes, long long tiles, long long grid, long long there_are, int groups, int chip)
{
    if (grid <= chip || grid >= 8LL * split::kMostDividend || groups < 2 || grid > there_are + there_are / 4) return {0, 1};
    const bool ragged = tiles <= 4 && 20LL * l.most * l.batch >= 27LL * l.total;
    if (!ragged && tiles <= 3) return {0, 1};
    const long long longest = (ragged ? 6LL : l.heads % 8 == 0 ? 3LL : 2LL) * l.most, top = 1 << 30;
    const long long part = ((l.head_dim >= 256 ? 10LL : 20LL) << 20) / ((long long)l.head_dim * bytes * groups);
    return {(int)(longest < top ? longest : top), part < 1 ? 1 : (int)part};
}
// The pairs that go abreast, of `groups`, over contexts up to `longest`.
__host__ __device__ inline int pairs_abreast(const Together &w, int longest, int groups)
{
    if (longest > w.longest) return 1;
    if (longest <= w.part) return groups;
    const unsigned parts = ((unsigned)longest + w.part - 1) / w.part;
    return parts < (unsigned)groups ? (groups + parts - 1) / parts : 1;
}

// Tiles of 64 columns (16 per wave, a stage at a time) instead of 128: three (head size 128, grouped heads) or four workgroups and more
// to a CU, finer grain, half the columns that a short prompt leaves unused -- but each K / V byte read from LDS for half as
// many products.  They are the better ones while a launch is bound by the way to each tile's first bytes, not by the matrix
// cores, that is up to so many tiles of 128 (`wide`, at most), the more the shorter the prompts.  The lines are drawn through 1 050 random
// launches timed both ways (1 to 250 requests, groups of 1 to 16, 1 to 5 600 new tokens, up to 6 000 cached), where the mean over
// a range of `wide` comes near level; time of narrow tiles over wide ones, attention alone, below a line / above it:
//   prompts of 130 on average   plain heads of 128 0.57 (5 800), of 64 0.81 (4 100) / 1.17; grouped, of 128 0.89 (5 800), of 64 0.94 (4 100)
//      of 220                   plain 128 0.93 (2 000), 64 0.85 (2 000) / 1.17; grouped 128 0.95 (2 900) / 1.0, 64 0.94 (1 450) / 1.0 to 1.06
//      of 700                   plain 128 0.90 (1 450) / 1.08 (12 of 512), 64 0.91 (2 000) / 1.13; grouped 128 0.93 (1 250) / 1.04, 64 0.9 (900) / 1.0 to 1.1
//      longer                   plain 128 0.94 (1 000) / 1.03 to 1.10, 64 0.97 (1 400) / 1.0; grouped 128 0.89 (500) / 1.03, 64 0.86 (500) / 1.0 to 1.08
//   up to 8 new on cached       plain 128 1.02 to 1.06 (800 to 1 000)
//   new on up to 1 500 cached   heads of 128 0.95 (900) / 0.99, of 64 0.93 (1 100) / 0.97
//   on more, an average request's up to half a wide tile   128 0.95 (700) / 0.99, 64 0.94 (800); up to a tile 0.96 (500) / 1.02, 0.94 (800)
//      up to five               128 0.94 (720) / 1.0, 64 0.93 (720) / 0.96 to 1.04
//      more                     128 0.95 (360) / 1.02 and up to 1.3, 64 0.93 (500) / 1.02
// Single launches scatter by 0.1 about the mean (how the tiles fill the last round): over cached positions, below the lines, one in fourteen is
// 5 % and more slower with narrow tiles, up to 24 % (15 of 64 to 128 on 1 000 to 2 000, 32 / 4 heads), above them up to 40 % (21 of 12 to 128 on 1 500 to
// 2 500, 32 heads of 64), so the lines over long contexts stay at 800 or 900 also where the mean is still 0.95; nothing the host knows tells them.
// A wave of 16 columns should hold half the tokens that one of 32 does; with groups of 6 it holds two fifths, of 9 and 10 a third, and
// fewer launches are better off (6: prompts of up to 400 0.94 (1 800), longer 0.92 (400) / 1.17, cached 0.94 (400) / 1.10; 9 and 10: 0.89 (300) /
// 0.9 to 1.1, longer 1.2 to 1.5; cached 0.79 (200) / 0.9 to 1.3).
//
// The length of the contexts is known to the host as that of a row of the block table, their bound: rows longer than twice
// the most new tokens count as mostly cached.  A caller whose rows are as long as its longest possible request gets the lines for those.
inline bool narrow_tiles(const Launch &l, bool tiled)
{
    if (l.group > 16) return false;
    const int wt = 4 * (32 / l.group);   // new tokens of a wide tile
    const long long wide = (long long)l.heads * (l.total / wt + l.batch);
    const bool prompts = l.row <= 2LL * l.most, d64 = l.head_dim == 64;
    auto average_to = [&l](long long n) { return l.total <= n * l.batch; };
    if (2 * (16 / l.group) < 32 / l.group) {
        if (l.group == 6) return wide <= (l.most > 400 ? (prompts ? 500 : 250) : prompts ? 1800 : 500);
        return wide <= (prompts ? 400 : 250) && (prompts || l.most < 384);
    }
    if (!prompts && !tiled && !d64 && average_to(8)) return wide <= 400;
    if (!prompts && l.row <= 1500) return wide <= (d64 ? 1100 : 900);
    if (!prompts && average_to(5 * wt)) return wide <= (d64 || tiled ? 800 : 900) && (wide <= 600 || d64 || average_to(wt / 2) || !average_to(wt));
    if (!prompts) return wide <= (d64 ? 600 : 400);
    if (average_to(130)) return wide <= (d64 && !tiled ? 4500 : 6000);
    if (average_to(220)) return wide <= (tiled ? (d64 ? 1800 : 3200) : d64 ? 2400 : 2800);
    if (average_to(700)) return wide <= (tiled ? (d64 ? 1000 : 1300) : d64 ? 2100 : 1800);
    return wide <= (tiled ? 600 : d64 ? 1400 : 1100);
}

// prefill_teams: tiles of 256 columns (of 128 at head size 256), one to a CU.  They are the better ones where a CU gets one and a half and more
// and the requests fill theirs: a tile's start and end (5 us of the 60 of an average one) are behind nothing.  The lines are drawn through 660
// random launches timed both ways (1 to 48 requests, groups of 1 to 8, 24 to 6 000 new tokens, up to 6 000 cached), where the mean
// over a range of tiles (`all`, at most) comes near level; time over that of the other kernels, attention alone, above a line / below it:
//   prompts of four tiles and more on average   heads of 128 0.94 (400 and more) / 1.01 to 1.13, plain 0.95 / 1.09; plain heads of 256 0.92 (250) / 1.05
//      of two to four       heads of 128 0.94 (1 500) / 1.02 to 1.18, plain 0.99 to 1.07 / 1.08; plain heads of 256 0.88 (1 500) / 1.0
//   on cached positions, four and more          heads of 128 0.90 (250) / 1.14, plain 0.93 / 1.3; plain heads of 256 0.87 / 0.9 to 1.05
//      two to four          heads of 128 0.92 (250) / 1.06, plain 0.99 (700) / 1.1; plain heads of 256 0.92 / 1.06
//      four fifths to two   plain heads of 128 0.93 (700) / 1.05; of 256 0.77 (250) / 1.2
// Not for short walks: grouped heads of 128, prompts of 150 to 200 on average 1.05 to 1.2, of 300 to 430 1.03 to 1.07; 20 of 72 to 103 on 97 to 486 1.24.
// Grouped heads of 256, whose other kernel holds one workgroup of four waves to a CU: 0.91 throughout (47 launches).
inline bool teams(const Launch &l)
{
    const int columns = l.head_dim >= 256 ? 16 : 32;
    if (l.group > columns) return false;
    if (l.head_dim >= 256 && l.group > 1) return true;
    const long long wt = 8 * (columns / l.group), all = l.heads * (l.total / wt + l.batch);
    const bool prompts = l.row <= 2LL * l.most, plain = l.group == 1;
    auto tiles = [&l, wt](int n) { return l.total >= n * wt * l.batch; };   // on average
    if (prompts ? l.total < 450LL * l.batch : l.row < 600) return false;
    // few tiles: the average request's leave little of them empty (25 of 235 to 336 on 134 to 672, 16 plain heads of 128, 1.27; 10 of 324 to 464 on 40 1.11)
    const long long average = l.total / l.batch, filled = (average + wt - 1) / wt * wt;
    if (!tiles(4) && 5 * average < 4 * filled) return false;
    if (prompts) return all >= (tiles(4) ? (l.head_dim >= 256 ? 256 : 400) : tiles(2) && (!plain || l.head_dim >= 256) ? 1500 : 1LL << 40);
    if (tiles(4)) return all >= 256;
    if (tiles(2)) return all >= (plain && l.head_dim < 256 ? 700 : 256);
    // nor where some request has a tile more than the average one's, which then is nearly empty (42 launches 0.87 without such a request, 0.85 to 0.99,
    // and 0.98 with one, 0.84 to 1.32: 13 of 116 to 321 on 878 to 2 322, 32 plain heads of 128)
    return plain && l.most <= filled && all >= (l.head_dim < 256 ? 700 : 256);
}

}  // namespace rules
}  // namespace lamps
