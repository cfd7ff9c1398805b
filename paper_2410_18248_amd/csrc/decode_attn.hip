// Paged single-query decode attention for gfx950 (MI355X).
//
// Computes, for every running request r and query head h, the Section 2.2
// equation of arXiv 2410.18248,  out = softmax(q K^T * scale) V,  over the
// first ctx_lens[r] cached positions of r, with K and V reached through the
// block table (paged attention, Section 7).
//
// Work decomposition.  The unit of work is a chunk of CT tokens of one range: a (request, kv head, pass over GH query heads of
// the group); in small launches cut in GT tokens.  All forms share the inner loops; decode_rules.h chooses among them by the ranges there can be and
// the table row:
//   whole (decode_whole): a workgroup takes a range, two, four or eight waves a stretch each, added up in LDS.  For rows of
//     a few rounds of chunks: no plan, no pieces, no second launch.
//   cut (decode_cut): the same for hundreds of ranges on longer rows, by the lengths: the longest first, those beyond an even share in parts,
//     which the last of a range's workgroups to arrive adds up.
//   parts (decode_parts, decode_merge_parts): few ranges, cut into parts of one size that both launches work out from the lengths.
//   shares (decode_balanced, decode_merge_balanced): everything else.  All chunks of all running requests form one flat
//     sequence (head outermost, then request, then position), cut into shares.
//     With many ranges for the chip: as many wavefronts as it
//     holds at once each take an equal contiguous share, so every wavefront ends within
//     a chunk of the others however skewed the context lengths are.  With eight resident
//     waves and more to a range: a share belongs to a workgroup, whose four waves
//     take a quarter of each of its ranges.  With few chunks to a
//     share: the shares are pieces of one range each, if there are enough.  A share is at most: the
//     tail of one range, some whole ones, and the head of another;
//     whole ones are written out directly, the two partial ends go to
//     per-share slots that the second kernel merges.
//   fixed partitions (part_tokens > 0): the context is cut every part_tokens
//     tokens, one wavefront per (partition, request, kv head) in a dense grid.
// The inner loops of a wavefront use no LDS and no barrier; where waves cooperate, they meet once per range, part or piece.
// Pieces of shares, parts of few ranges and partitions are merged by a separate launch: a kernel boundary
// makes them visible across the eight XCDs' L2s once, whereas a
// device-scope fence per workgroup writes back and invalidates an L2 each time, and where all of them end at the same time a hand-over by
// agent-scope stores is on the way of each.  Only decode_cut, where what is cut is the exception, hands over inside the launch.
//
// Inner loops.  The path is a stream over K and V: every byte is used once, by
// the G query heads of its group.
//   G == 1 (and all fp32): ~1 flop per byte, a matrix-vector product.  Vector
//     ALUs, no MFMA: a tile is block_size*head_dim contiguous elements read
//     with coalesced non-temporal 16-byte-per-lane loads, LPT = head_dim*size/16
//     lanes per token; q slices stay in registers; the dot product ends with
//     DPP adds inside the LPT lanes; each group of LPT lanes ("row") carries
//     its own running max / sum / accumulator, rows are merged by shuffles.
//   bf16 with G >= 2: the group's heads make q a G x d_h matrix and both
//     products real (skinny) contractions, and on the vector ALUs their cost
//     grows with G until it co-limits with HBM.  They go to MFMA instead
//     (16x16x32 for K q^T, 16x16x16 for V^T p^T, up to 16 heads per pass), and
//     the pools use the tiled layout of lamps.h so that a coalesced 16-byte
//     load IS an MFMA operand: no LDS staging, no shuffles.  The weights p are
//     fed as a bf16 pair (high part + remainder), which keeps fp32-grade
//     weights at the price of a second, nearly free, MFMA.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "attn_reducers.h"
#include "decode_rules.h"
#include "handover.h"
#include "internal.h"
#include "lamps.h"
#include "prefill_split.h"

namespace lamps {
namespace {

// ---------------------------------------------------------------- fixed partitions

// One wavefront: one (partition, request, kv head / pass), decoded from a 1-D
// index.  The heads of one pass share the K/V stream.
template <typename R>
__global__ __launch_bounds__(kThreads) void decode_partial(const DecodeArgs a)
{
    constexpr int D = R::D;
    // Workgroups are handed to the eight XCDs round-robin in launch order, so the
    // index that varies fastest must be one along which the work is even: the
    // kv head (and pass), then the request, then the partition.  (With the
    // partition fastest and eight partitions, all first partitions -- most of
    // the work -- would land on one XCD.)
    const int G = a.num_q_heads / a.num_kv_heads;
    const int GH = a.heads_per_pass;
    const int passes = G / GH;
    const int hc_count = a.num_kv_heads * passes;
    const long long item = (long long)blockIdx.x * kWaves +
                           __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= (long long)a.max_parts * hc_count * a.batch) return;
    const int hc = (int)(item % hc_count);
    const int r = (int)((item / hc_count) % a.batch);
    const int part = (int)(item / ((long long)hc_count * a.batch));
    const int running = a.running[r];          // both loads are in flight together
    const int C = ctx_len(a, r);
    if (!running) return;                      // Preserve / Swap / Discard: not in the batch
    const int t_begin = part * a.part_tokens;
    if (t_begin >= C && part != 0) return;     // partition 0 of an empty context writes zeros
    const int t_end = min(C, t_begin + a.part_tokens);
    const int n_parts = max(1, (C + a.part_tokens - 1) / a.part_tokens);
    const int g = hc / passes;
    const int h0 = g * G + (hc % passes) * GH;
    const size_t rh0 = (size_t)r * a.num_q_heads + h0;

    const bool wide = ((uintptr_t)a.out & 15) == 0;
    R::run(a, r, (size_t)r, g, h0, GH, t_begin, t_end, [&](int h, int d, float M, float L, const auto &A) {
        if (n_parts == 1)
            store_out<R::kBF16>(a.out, (rh0 + h) * D + d, wide, L, A);
        else
            store_partial(a.partials + ((rh0 + h) * a.max_parts + part) * (D + 2), D, d, M, L, A);
    });
}

// Merge of the partitions of one (request, query head), always in partition
// order; block = head_dim threads.
template <bool BF16>
__global__ void decode_merge(const DecodeArgs a)
{
    const int r = blockIdx.y, h = blockIdx.x, d = threadIdx.x;
    if (!a.running[r]) return;
    const int C = ctx_len(a, r);
    const int n_parts = (C + a.part_tokens - 1) / a.part_tokens;
    if (n_parts <= 1) return;                  // written by the partial kernel already
    const int D = a.head_dim;
    const size_t rh = (size_t)r * a.num_q_heads + h;
    const float *pp = a.partials + rh * a.max_parts * (D + 2);
    float M = kLowest, L = 0.0f, A = 0.0f;
    for (int p0 = 0; p0 < n_parts; p0 += 8) {         // eight partitions' loads in flight together
        float mo[8], lo[8], ao[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool ok = p0 + k < n_parts;
            const float *x = pp + (size_t)(ok ? p0 + k : 0) * (D + 2);
            mo[k] = ok ? x[D] : kLowest;
            lo[k] = ok ? x[D + 1] : 0.0f;
            ao[k] = ok ? x[d] : 0.0f;
        }
        float Mn = M;
#pragma unroll
        for (int k = 0; k < 8; ++k) Mn = fmaxf(Mn, mo[k]);
        const float f0 = fast_exp2(M - Mn);
        L *= f0;
        A *= f0;
        M = Mn;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float f = fast_exp2(mo[k] - M);
            L += lo[k] * f;
            A += ao[k] * f;
        }
    }
    store_out<BF16>(a.out, rh * D + d, L > 0.0f ? A / L : 0.0f);
}

// ---------------------------------------------------------------- balanced shares

// Share w of P has the positions [floor(w * total / P), floor((w + 1) * total / P)) of the flat chunk
// sequence.  The sequence practically always has less than 2^31 positions, and then a few 32-bit
// divisions do: the general 64-bit ones were 1 us in the prologue of every wave, of 3 to 4.
__device__ __forceinline__ bool fits32(long long total) { return total <= 0x7fffffff; }
__device__ __forceinline__ long long share_begin(int w, long long total, int P)
{
    if (!fits32(total)) return (long long)w * total / P;
    const unsigned q = (unsigned)total / (unsigned)P, rem = (unsigned)total - q * (unsigned)P;
    return w * q + (unsigned)w * rem / (unsigned)P;   // w * rem < kMaxShares^2
}
// The share that position x belongs to.
__device__ __forceinline__ int share_of(long long x, long long total, int P)
{
    if (!fits32(total)) return (int)(((x + 1) * P - 1) / total);
    // exact: the quotient is a multiple of 1 / total and below kMaxShares, and rounding to 53 bits
    // cannot carry one that is no whole number up to the next
    return (int)((double)((x + 1) * P - 1) / (double)total);
}

constexpr int kLaneBatch = 64;           // requests of a batch that a wave holds one per lane
constexpr int kPieceMost = 64;           // chunks of a piece

// Chunks a running request contributes per (kv head, pass): an empty context
// still gets one (empty) chunk so that its zero row is written.
__device__ __forceinline__ int chunks_of(int running, int C, int GT) { return running ? max(1, (C + GT - 1) >> __builtin_ctz(GT)) : 0; }
// Masks and lengths of K requests from r on, asked for together and not one behind the other: no load is conditional, and
// nothing is looked at before the last of them has been asked for.  Those past the batch do not run.  (Four round trips, one for
// each request of a lane, and one: 256 requests of 16 to 80 tokens, 8 heads of 64, 13.9 and 13.3 us; 180 on 40 heads of 128 36.5 and 35.7.)
template <int K>
__device__ __forceinline__ void requests_of(const DecodeArgs &a, int r, int2 (&q)[K])
{
    int running[K], C[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = min(r + k, a.batch - 1);
        running[k] = a.running[i];
        C[k] = a.ctx_lens[i];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(running[k]), "+v"(C[k]));
#pragma unroll
    for (int k = 0; k < K; ++k) q[k] = make_int2(r + k < a.batch ? running[k] : 0, min(C[k], a.max_blocks * a.block_size));
}
__device__ __forceinline__ int2 request_of(const DecodeArgs &a, int r)
{
    int2 q[1];
    requests_of(a, r, q);
    return q[0];
}

// The flat chunk sequence of a launch in LDS: the chunks before each request, per head / pass, and its length.  Batches of up
// to 256: pairs of the two, and the chunks of all behind them, written by every wave (each the same, so no wave waits for
// another).  Not kept in registers, one request per lane, for batches of up to 64: two registers through the loop took a
// workgroup off a CU with fp32 heads of 32 (250 requests of 100 to 1 500 tokens on 8 / 2 of them, by workgroups: 26.5 us with four,
// 21.7 with five).  Larger batches: the prefix alone, by all waves of a workgroup.
struct Request {
    int before, count, ctx;
};
struct Sequence {
    const int *prefix;                                // LDS
    const DecodeArgs *a;
    int upto;                                         // chunks up to and of the lane's requests
    __device__ __forceinline__ Request operator[](int r) const
    {
        if (a->batch <= 4 * kLaneBatch) {
            const int2 x = reinterpret_cast<const int2 *>(prefix)[r];
            const int before = __builtin_amdgcn_readfirstlane(x.x);
            return Request{before, __builtin_amdgcn_readfirstlane(prefix[2 * r + 2]) - before, __builtin_amdgcn_readfirstlane(x.y)};
        }
        const int before = __builtin_amdgcn_readfirstlane(prefix[r]);
        return Request{before, __builtin_amdgcn_readfirstlane(prefix[r + 1]) - before, ctx_len(*a, r)};
    }
};
// Ints of it in a launch's dynamic LDS.
__host__ __device__ __forceinline__ int balanced_ints(int batch)
{
    return batch <= 4 * kLaneBatch ? (batch <= kLaneBatch ? 2 : 8) * kLaneBatch + 4 : (batch + 1 + 3) & ~3;
}

// gridDim.x * 4 wavefronts, each an equal contiguous share of the flat chunk
// sequence ordered (kv head / pass, request, chunk).  Every wave (of batches above 256: every workgroup, through the
// prefix in dynamic LDS) works the sequence out for itself from ctx_lens / running (loads that hit
// in L2), which costs less than a dependent launch.
//
// Which share a wavefront takes: with the heads outermost, the shares that read
// the same blocks for different heads lie shares / heads apart.  Workgroups go to
// the eight XCDs in turn, each XCD translates addresses for itself, and a block's
// heads share its pages; so the shares are handed out in the order of their
// position inside a head's stretch, XCD 0 first: the waves that walk the same
// blocks at the same time then sit on one XCD, next to each other.  With pools of
// 100 GB and more this is worth several per cent; with small pools it is neutral.
//
// Small launches are bound by the way to the first K / V byte: mask and lengths are asked for
// together, scans are DPP adds, nothing waits at a barrier, divisions are by reciprocal or 32 bits wide (beyond 2^31 chunks 64), lengths
// come out of LDS, and the cut is by half-chunks, so that no wave has twice another's work.  One
// request of 1 999 tokens, both launches: 13.2 -> 10.3 us with half of that, 9.85 -> 9.05 with the rest.
//
// TOGETHER: a share belongs to a workgroup, whose four waves take a quarter of each of its ranges
// and add the quarters up in LDS.  For launches with few ranges for the waves (a few requests, or
// long ones): a quarter of the pieces to write, and to read and add up in the second kernel.  Both
// launches, a share per wave -> per workgroup: 24 fp32 requests of 17 to 2 500 tokens, 32 / 8 heads of
// 128, 40.8 -> 33.0 us; 19 of 32 requests of 4 096 to 32 768 tokens, 32 / 8 heads, 209.7 -> 205.3; one
// request of 1 999 tokens 14.5 -> 13.2.
template <typename R, bool TOGETHER>
__global__ __launch_bounds__(kThreads, R::kLeastPerCu) void decode_balanced(const DecodeArgs a)
{
    constexpr int D = R::D;
    extern __shared__ __align__(16) int prefix[];     // balanced_ints; then, TOGETHER, [wave][head][D + 2] floats
    __shared__ int wave_total[2][kWaves], wave_longest[kWaves];

    const int B = a.batch;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr bool kCut = R::CT != R::GT;            // (else chunk and cut are one)
    const int GH = a.heads_per_pass;
    const int passes = a.passes;
    const int HC = a.num_kv_heads * passes;
    constexpr int kOwnShares = TOGETHER ? 1 : kWaves;  // of a workgroup
    const int sub = TOGETHER ? 0 : wv;
    int P = gridDim.x * kOwnShares;
    int share = blockIdx.x * kOwnShares + sub;
    // Below, a chunk is GT tokens, and a wave loads one of them, or two, at a time.  Cutting by the smaller ones evens
    // launches out whose shares are a chunk or less; it costs a half-empty load where a range is cut, which is
    // all that is left where shares are longer.  By halves / whole: 40 fp32 requests of 60 to 200 tokens, 32 / 16 heads
    // of 128 (1.3 chunks a share, 2 layers) 51 / 54 us; 100 of 60 to 90, 16 heads of 256 (1.8, 3 layers) 100 / 96;
    // 34 of 202 to 532 (2.9) 136 / 129; 110 of 28 to 161 on 40 heads of 128 (3.2) 118 / 116.
    const auto by_whole = [&](int wholes) { return kCut && 2LL * wholes * HC >= 3LL * P; };
    // A launch with little work and a long range in it: equal shares over all wavefronts would
    // cut that range into hundreds of pieces of a chunk each, and the merge of one range is a
    // chain of dependent loads (a 40 000-token request among 70 short ones, 2 heads: 10 us of
    // attention, 200 us of merge).  Then only as many shares are used as gives each 2, 4 or
    // 8 chunks -- for a longest range of 256, 512, 1024 chunks and more -- and the rest stay
    // empty.  TOGETHER: a chunk per wave at least (half of that: 10.6 -> 11.6 us on 3 000 tokens of 8 kv heads, twice: 9.6 ->
    // 11.7 on 8 plain ones), and the rest as for a range a quarter as long (one range of 20 000 tokens 13.3 us, 16.2
    // with a chunk per wave; 40 000: 16.0 and 21.2; twice the length costs 19.4 there).
    const auto least_share = [&](int span) {          // log2, in whole chunks
        return TOGETHER ? (span >= 4096 ? 5 : span >= 2048 ? 4 : span >= 1024 ? 3 : 2)
                        : span >= 1024 ? 3 : span >= 512 ? 2 : span >= 256 ? 1 : 0;
    };
    // A piece may have so many chunks more than an even cut, less than what a share that straddles two ranges loses: a chunk
    // of a wave, but none where that is 32 tokens (32 requests of 100 to 900 tokens, 32 plain heads of 128: 37.0 us
    // without, 39.6 with one more; 60 of 20 to 9 000, 8 / 2 heads of 64: 18.8 us without, 14.5; 250 of 20 to 500, by workgroups,
    // 17.0 with a quarter of a chunk, 12.3).
    const auto piece_slack = [](bool whole_chunks) { return TOGETHER ? (whole_chunks ? 1 : kWaves) : (whole_chunks ? 0 : 1); };
    // Chunks of a piece at most: where shares are longer, they straddle ranges.  By waves and 32 tokens at a time the chip is
    // bound by memory before that, and a piece longer than an even cut is what the launch ends with (straddling / pieces, us: 167 fp32
    // requests of 596 to 775, 8 heads of 32, 4.1 chunks a share, pieces of 5, 45.3 / 46.9; 108 of 691 to 899 on 8 of 64, 5.3 and 6,
    // 61.6 / 62.9; 18 of 1 010 to 1 313 on 32 of 128, 5.3 and 6, 62.7 / 62.3; 61 of 96 to 387 on 16 of 256, 3.5 and 4, 46.8 / 46.2).
    const auto piece_most = [](bool whole_chunks) { return !TOGETHER && whole_chunks ? 4 : kPieceMost; };
    const auto empty_share = [&](int which) {
        if (lane == 0) a.share_info[which] = make_int4(0, 0, 0, kShareEmpty);
    };
    Sequence seq{prefix, &a, 0};
    int GT, T, log2_least;                            // tokens of a chunk; chunks per head / pass; least chunks of a share
    // A share that straddles two ranges is two chains of dependent loads (2.3 to 3.5 us each) behind each other, and
    // the launch ends with the last of them.  Where shares are a few chunks, they are pieces of one range each, if
    // there are enough shares for the pieces of about the size of an even cut.  Both launches, straddling -> pieces (as for
    // the last three, they were before only where a share had less than a chunk): 4 layers of 8 requests of 20 to 159 tokens,
    // 16 heads of 256, append included, 72 -> 57 us; 24 fp32 requests of 17 to 2 500, 32 / 8 heads, 32.9 -> 30.2;
    // 4 layers of 16 of 70 to 914, 40 heads, with the append 112.9 -> 106; 64 of 50 to 300, 32 / 8 heads, 19.7 -> 15.3.
    int r = 0, hc = 0, last_share = -1;               // the first range's request, head / pass; its last share, if known
    long long x = -1, x_end = 0;                      // this share's part of the sequence
    // Batches of up to 64 * K requests, K consecutive ones per lane; every wave by itself, no barrier in front of the
    // first byte.  False: the share is empty, and marked so.  All the waves of a SIMD issue it, four to six of them, so its
    // length is time: where it ends in straddling shares all the same, it must not take longer than the barriers and the
    // one request per thread of larger batches.  (So it did, with a 64-bit division, a scan for every size that might
    // fit, entries of 16 bytes and a binary search through them.  By barriers / so / as it is, us: 250 requests of 100 to 1 500
    // tokens on 8 heads of 64 52.9 / 54.4 / 52.4; 150 of 16 to 80 on 32 heads of 128 27.3 / 27.9 / 26.7; 100 of 50 to 400 on 16 of 256
    // 59.1 / 59.4 / 58.4; 250 fp32 ones of 100 to 1 500 on 8 heads of 32 51.0 / 51.9 / 51.1.)
    const auto plan = [&](auto per_lane) {
        constexpr int K = per_lane;
        int n[K], parts = 0, wholes = 0, longest = 0;
        int2 q[K];
        requests_of(a, K * lane, q);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            n[k] = chunks_of(q[k].x, q[k].y, R::GT);
            parts += n[k];
            wholes += (n[k] + 1) >> 1;
            longest = max(longest, n[k]);
        }
        int upto = wave_scan(parts);
        const int upto_whole = kCut ? wave_scan(wholes) : 0;
        longest = __builtin_amdgcn_readlane(wave_max_to(longest), 63);
        const bool whole_chunks = kCut && by_whole(__builtin_amdgcn_readlane(upto_whole, 63));
        const int log2_whole = kCut && !whole_chunks ? 1 : 0;
        GT = whole_chunks ? R::CT : R::GT;
        if (whole_chunks) {
#pragma unroll
            for (int k = 0; k < K; ++k) n[k] = (n[k] + 1) >> 1;
            parts = wholes;
            upto = upto_whole;
            longest = (longest + 1) >> 1;
        }
        T = __builtin_amdgcn_readlane(upto, 63);
        seq.upto = upto;
        int before = upto - parts;
        if constexpr (K == 1) {
            reinterpret_cast<int2 *>(prefix)[lane] = make_int2(before, q[0].y);
        } else {
#pragma unroll
            for (int k = 0; k < K; k += 2) {
                reinterpret_cast<int4 *>(prefix)[(K * lane + k) / 2] = make_int4(before, q[k].y, before + n[k], q[k + 1].y);
                before += n[k] + n[k + 1];
            }
        }
        if (lane == 63) prefix[2 * K * kLaneBatch] = T;
        log2_least = least_share(longest >> log2_whole) + log2_whole;
        const long long chunks = (long long)T * HC;
        if (chunks > (long long)piece_most(whole_chunks) * P || longest >= split::kMostDividend / 2) return true;
        // The smallest size that gives no more pieces than shares, if it is about that of an even cut.  The lane's pieces of the
        // first size, and from bit 16 on those of the last (together at most T / even + 256 of each): where not even those
        // fit, the launch has lost one scan and no more.
        const auto pieces = [&](int k, int size) { return split::small_div(n[k] + size - 1, size); };
        int size = max(1 << log2_least, (int)((unsigned)(chunks + P - 1) / (unsigned)P));
        const int most = size + piece_slack(whole_chunks);
        int on = longest > most;
#pragma unroll
        for (int k = 0; k < K; ++k) on += __popcll(__ballot(n[k] > 0));
        if (on * HC > P) return true;                 // a piece per request that runs, and one more, do not fit
        int both = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) both += pieces(k, most) << 16;
        if (most > size) {
#pragma unroll
            for (int k = 0; k < K; ++k) both += pieces(k, size);
        } else {
            both |= (unsigned)both >> 16;
        }
        const int both_to = wave_scan(both), both_all = __builtin_amdgcn_readlane(both_to, 63);
        if ((both_all >> 16) * HC > P) return true;
        int own = both & 0xFFFF, upto_own = both_to & 0xFFFF, all = both_all & 0xFFFF;
        while (all * HC > P) {                        // (`most` is the last)
            ++size;
            own = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) own += pieces(k, size);
            upto_own = wave_scan(own);
            all = __builtin_amdgcn_readlane(upto_own, 63);
        }
        int np[K];
#pragma unroll
        for (int k = 0; k < K; ++k) np[k] = pieces(k, size);
        const int N = all * HC;
        // Pieces by position, a position's heads next to each other, an eighth of them to each XCD (workgroups
        // are dealt to those in turn); share numbers go by head, for the second kernel.
        int rank = share, idle = share;
        if (a.share_gcd > 0) {
            const int xcd = blockIdx.x & 7, local = (blockIdx.x >> 3) * kOwnShares + sub, eighth = (N + 7) >> 3;
            const int mine = min(max(N - xcd * eighth, 0), eighth);
            rank = local < mine ? xcd * eighth + local : N;
            idle = N + xcd * (P >> 3) - min(N, xcd * eighth) + local - mine;
        }
        if (rank >= N) {
            empty_share(idle);
            return false;
        }
        int at = split::small_div(rank, HC);
        hc = rank - at * HC;
        share = hc * all + at;
        // the request: the first whose pieces end behind `at`
        const int l = __popcll(__ballot(upto_own <= at));
        at -= __builtin_amdgcn_readlane(upto_own - own, l);
        int of = __builtin_amdgcn_readlane(np[0], l), k = 0, base = __builtin_amdgcn_readlane(upto - parts, l);
        int nr = __builtin_amdgcn_readlane(n[0], l);
#pragma unroll
        for (int j = 1; j < K; ++j)
            if (k == j - 1 && at >= of) {
                at -= of;
                base += nr;
                k = j;
                of = __builtin_amdgcn_readlane(np[j], l);
                nr = __builtin_amdgcn_readlane(n[j], l);
            }
        r = K * l + k;
        const int each = split::small_div(nr + of - 1, of);
        x = (long long)hc * T + base + at * each;
        x_end = (long long)hc * T + base + min((at + 1) * each, nr);
        last_share = share - at + of - 1;
        return true;
    };
    if (B <= kLaneBatch) {
        if (!plan(std::integral_constant<int, 1>{})) return;
    } else if (B <= 4 * kLaneBatch) {
        if (!plan(std::integral_constant<int, 4>{})) return;
    } else {
        const int per = (B + kThreads - 1) / kThreads;   // consecutive requests per thread
        int parts = 0, wholes = 0, longest = 0;          // of this thread's requests, in GT and in CT tokens
        for (int i = 0; i < per; ++i)
            if (tid * per + i < B) {
                const int2 q = request_of(a, tid * per + i);
                const int n = chunks_of(q.x, q.y, R::GT);
                parts += n;
                if (kCut) wholes += (n + 1) >> 1;
                longest = max(longest, n);
            }
        longest = wave_max_to(longest);
        const int parts_to = wave_scan(parts), wholes_to = kCut ? wave_scan(wholes) : 0;   // inclusive, inside the wave
        if (lane == 63) {
            wave_total[0][wv] = parts_to;
            wave_total[1][wv] = wholes_to;
            wave_longest[wv] = longest;
        }
        __syncthreads();
        int T_whole = 0;
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
            longest = max(longest, wave_longest[ww]);
            T_whole += wave_total[1][ww];
        }
        const bool whole_chunks = by_whole(T_whole);
        const int log2_whole = kCut && !whole_chunks ? 1 : 0;
        GT = whole_chunks ? R::CT : R::GT;
        if (whole_chunks) longest = (longest + 1) >> 1;
        int run = (whole_chunks ? wholes_to - wholes : parts_to - parts);
#pragma unroll
        for (int ww = 0; ww < kWaves - 1; ++ww) run += ww < wv ? wave_total[whole_chunks][ww] : 0;
        if (tid == 0) prefix[0] = 0;
        for (int i = 0; i < per; ++i) {
            const int q = tid * per + i;
            if (q < B) {
                const int2 x = request_of(a, q);
                run += chunks_of(x.x, x.y, GT);
                prefix[q + 1] = run;
            }
        }
        __syncthreads();
        // (values that are the same in every lane are told so: the compiler cannot see it
        // through LDS and the shuffles, and would keep the range arithmetic in vector registers)
        T = __builtin_amdgcn_readfirstlane(prefix[B]);
        log2_least = __builtin_amdgcn_readfirstlane(least_share(longest >> log2_whole)) + log2_whole;
    }
    const long long total = (long long)HC * T;
    if (x < 0) {
        const long long wanted = (total + (1 << log2_least) - 1) >> log2_least;
        if (wanted < P) {
            P = __builtin_amdgcn_readfirstlane(max(1, (int)wanted));
            if (share >= P) {
                empty_share(share);
                return;
            }
        } else if (a.share_gcd > 0) {
            // rank = (share * HC mod P) + share / (P / gcd) orders the shares by where they
            // start inside a head's stretch; this wave takes the share of rank
            // (XCD, index inside the XCD), found by inverting that
            const int rank = (blockIdx.x & 7) * (P >> 3) + (blockIdx.x >> 3) * kOwnShares + sub;
            const unsigned turn = (unsigned)rank / (unsigned)a.share_gcd, tie = (unsigned)rank - turn * (unsigned)a.share_gcd;
            share = (int)(turn * (unsigned)a.share_inv % (unsigned)a.share_period + tie * (unsigned)a.share_period);   // < kMaxShares^2
        }
        x = share_begin(share, total, P);
        x_end = share_begin(share + 1, total, P);
        if (x >= x_end) {
            empty_share(share);
            return;
        }
        // request that holds position x of its head: the last r that begins at or before it
        hc = __builtin_amdgcn_readfirstlane(fits32(total) ? (int)((unsigned)x / (unsigned)T) : (int)(x / T));
        const int first_pos = (int)(x - (long long)hc * T);
        if (B <= 4 * kLaneBatch) {
            r = __popcll(__ballot(seq.upto <= first_pos));
            if (B > kLaneBatch) {                     // of four
                const int *of = prefix + 8 * r;
                r = 4 * r + __builtin_amdgcn_readfirstlane((of[2] <= first_pos) + (of[4] <= first_pos) + (of[6] <= first_pos));
            }
        } else {
            int lo = 0, hi = B;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (prefix[mid] <= first_pos) lo = mid; else hi = mid;
            }
            r = __builtin_amdgcn_readfirstlane(lo);
        }
    }
    // What the merge kernel needs to know about this share: whether it is empty,
    // and the (request, head) range it starts but does not finish, if any (only
    // its last range can be one): request, head/pass, last share of the range,
    // and the slot this share's piece went to.
    int4 owned = make_int4(0, 0, 0, 0);
    const bool wide = ((uintptr_t)a.out & 15) == 0;
    Request at = seq[r];
    for (const long long x_begin = x; x < x_end;) {
        const int base = at.before, nr = at.count, C = at.ctx;   // nr > 0 here
        const int c0 = (int)(x - (long long)hc * T) - base;
        const int len = (int)min((long long)(nr - c0), x_end - x);
        int g = hc, h0 = hc * GH;                     // (GH == G, or a pass over part of the group)
        if (passes > 1) g = hc / passes;
        const bool whole = (c0 == 0 && len == nr);
        // a share's first range goes to slot 0, a later partial one (its last) to slot 1
        float *slot = a.partials + ((size_t)share * 2 + (x == x_begin ? 0 : 1)) * GH * (D + 2);
        const size_t rh0 = (size_t)r * a.num_q_heads + h0;
        if constexpr (TOGETHER) {
            float *part = reinterpret_cast<float *>(prefix) + balanced_ints(B);
            const int each = (len + kWaves - 1) / kWaves, from = min(len, each * wv);
            float *mine = part + (size_t)wv * GH * (D + 2);
            R::run(a, r, (size_t)r, g, h0, GH, (c0 + from) * GT, min(C, (c0 + min(len, from + each)) * GT),
                   [&](int h, int d, float M, float L, const auto &A) { store_partial(mine + h * (D + 2), D, d, M, L, A); });
            __syncthreads();
            for (int i = 2 * tid; i < GH * D; i += 2 * kThreads) {
                const int h = i / D, d = i % D;
                const float *x = part + h * (D + 2);
                float M = kLowest, L = 0.0f, A[2] = {0.0f, 0.0f};
                float2 ml[kWaves];
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    ml[w] = *reinterpret_cast<const float2 *>(x + w * GH * (D + 2) + D);
                    M = fmaxf(M, ml[w].x);
                }
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const float f = fast_exp2(ml[w].x - M);
                    const float2 o = *reinterpret_cast<const float2 *>(x + w * GH * (D + 2) + d);
                    L += ml[w].y * f;
                    A[0] += o.x * f;
                    A[1] += o.y * f;
                }
                if (whole)
                    store_out<R::kBF16>(a.out, (rh0 + h) * D + d, wide, L, A);
                else
                    store_partial(slot + (size_t)h * (D + 2), D, d, M, L, A);
            }
            __syncthreads();                          // before the next range's parts
        } else {
            R::run(a, r, (size_t)r, g, h0, GH, c0 * GT, min(C, (c0 + len) * GT),
                   [&](int h, int d, float M, float L, const auto &A) {
                       if (whole)
                           store_out<R::kBF16>(a.out, (rh0 + h) * D + d, wide, L, A);
                       else
                           store_partial(slot + (size_t)h * (D + 2), D, d, M, L, A);
                   });
        }
        if (c0 == 0 && len < nr)
            owned = make_int4(r, hc, last_share >= 0 ? last_share : share_of(x + nr - 1, total, P),
                              kShareOwner | (x == x_begin ? 0 : kShareSlot1));
        x += len;
        if (c0 + len == nr && x < x_end) {            // request finished: next one with work,
            do {                                      // after the last one the next head's first
                if (++r == B) {
                    r = 0;
                    ++hc;
                }
                at = seq[r];
            } while (at.count == 0);
        }
    }
    if (TOGETHER ? tid == 0 : lane == 0) a.share_info[share] = owned;
}

// ---------------------------------------------------------------- whole ranges

// Chunks c0 .. c1 - 1 of a range by W waves of a workgroup, a stretch each, whose states are added up through x0 ([wave][head][D + 2], LDS)
// and given to out(first head's row, head, dim, M, L, two outputs).  A barrier: by all waves of the workgroup.
template <typename R, int W, typename Out>
__device__ __forceinline__ void stretches(const DecodeArgs &a, float *x0, int sub, int r, int hc, int c0, int c1, int C, Out out)
{
    constexpr int D = R::D;
    constexpr bool kCut = R::CT != R::GT;
    const int lane = threadIdx.x & 63, GH = a.heads_per_pass, passes = a.passes;
    const int g = passes > 1 ? hc / passes : hc, h0 = hc * GH, n = c1 - c0;
    int each = (n + W - 1) / W;
    if (kCut && each >= 2) each = (each + 1) & ~1;    // (by whole chunks)
    const int from = min(n, each * sub);
    const size_t rh0 = (size_t)r * a.num_q_heads + h0;
    R::run(a, r, (size_t)r, g, h0, GH, (c0 + from) * R::GT, min(C, (c0 + min(n, from + each)) * R::GT),
           [&](int h, int d, float M, float L, const auto &A) { store_partial(x0 + (size_t)(sub * GH + h) * (D + 2), D, d, M, L, A); });
    __syncthreads();
    for (int i = 2 * (64 * sub + lane); i < GH * D; i += 128 * W) {
        const int h = i / D, d = i % D;
        const float *x = x0 + h * (D + 2);
        float M = kLowest, L = 0.0f, A[2] = {0.0f, 0.0f};
        float2 ml[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            ml[w] = *reinterpret_cast<const float2 *>(x + w * GH * (D + 2) + D);
            M = fmaxf(M, ml[w].x);
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = fast_exp2(ml[w].x - M);
            const float2 o = *reinterpret_cast<const float2 *>(x + w * GH * (D + 2) + d);
            L += ml[w].y * f;
            A[0] += o.x * f;
            A[1] += o.y * f;
        }
        out(rh0, h, d, M, L, A);
    }
}

// W waves of a workgroup take a whole range, one (request, kv head / pass), each a stretch of its chunks, and add their states up in LDS:
// no plan, no pieces and no second launch.  For launches of ranges that are short, or short against the work of the chip; lengths are on the
// device, so the host goes by the bound of a table row (decode_rules.h).  Bound by latency -- length, table entries, K / V, and at the end the
// sum -- where the launch is small, otherwise by memory as decode_balanced is.  Both ways, us: one request of 200 tokens, 32 / 8 heads of 128,
// 7.0 / 4.4; 64 of 50 to 300 on 32 / 8 14.8 / 8.9; 40 of 16 to 130 on 40 plain heads 14.1 / 9.6; 200 of 20 to 250 on 32 / 8 20.6 / 12.9.
// By two waves a workgroup has two ranges, half of the launch apart, and where one of them waits all four waves take the other: where few of thousands of
// ranges run they are walks on an empty chip.  Time over the plan's, mean and slowest, 4 096 ranges and more of 2 and 3 rounds, of 2 to 25 % of the requests: by
// two waves always 0.63, 1.84, so 0.58, 1.33, four 0.57, 1.27; all others 0.90, 1.34 / 0.89, 1.49 / 0.98, 1.73.
template <typename R, int W>
__global__ __launch_bounds__(64 * (W > kWaves ? W : kWaves), R::kLeastPerCu) void decode_whole(const DecodeArgs a)
{
    constexpr int D = R::D;
    extern __shared__ __align__(16) float parts[];    // [range][wave][head][D + 2]
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int GH = a.heads_per_pass, HC = a.num_kv_heads * a.passes;
    const auto take = [&](auto waves, float *x0, int sub, int r, int hc, int C) {
        stretches<R, decltype(waves)::value>(a, x0, sub, r, hc, 0, chunks_of(1, C, R::GT), C, [&](size_t rh, int h, int d, float M, float L, const float (&A)[2]) {
            store_out<R::kBF16>(a.out, (rh + h) * D + d, ((uintptr_t)a.out & 15) == 0, L, A);
        });
    };
    const int item = blockIdx.x, r = __builtin_amdgcn_readfirstlane(item / HC);
    const int2 q = request_of(a, r);
    const bool on = __builtin_amdgcn_readfirstlane(q.x) != 0;
    if constexpr (W >= kWaves) {
        if (on) take(std::integral_constant<int, W>{}, parts, wv, r, item - r * HC, __builtin_amdgcn_readfirstlane(q.y));
    } else {
        const int item2 = item + gridDim.x, r2 = __builtin_amdgcn_readfirstlane(item2 / HC);
        const int2 q2 = request_of(a, r2);            // (past the batch: does not run)
        const bool on2 = __builtin_amdgcn_readfirstlane(q2.x) != 0;
        if (!on && !on2) return;
        const bool second = on && on2 ? wv / W != 0 : on2;
        const int rr = second ? r2 : r, hc = (second ? item2 : item) - rr * HC, C = __builtin_amdgcn_readfirstlane(second ? q2.y : q.y);
        if (on && on2) take(std::integral_constant<int, W>{}, parts + (size_t)(wv / W) * W * GH * (D + 2), wv % W, rr, hc, C);
        else take(std::integral_constant<int, kWaves>{}, parts, wv, rr, hc, C);
    }
}

// Ranges that may be long, in one launch that looks at the lengths itself: those of about the size of an even share go whole to a workgroup, the
// longest first, and longer ones are cut, each part a workgroup's, in front of them; the last part of a range to arrive adds them up.  No walk
// is longer than one and a half even shares (or three rounds of chunks), however skewed the batch is and however few of it run; the workgroups that are not needed
// (`spare` more than there are ranges are launched) leave.  Bound by the memory where the launch is large, else by one walk: request, table entry, two
// rounds, the sum.  By the plan's two launches / whole ranges by eight waves / so, us, 40 plain heads: 16 requests of 60 to 1 500 tokens 32.5 / 30.3 / 27.3,
// 15 of 30 and one of 1 500 14.9 / 22.7 / 12.8, 2 of 16 running 15.8 / 23.4 / 14.6; 54 of 144 running, 180 tokens and one of 2 863, 32 heads, 37.2 / 48.4 / 34;
// 64 of 1 500, 32 / 8 heads, 65.6 / 60.8 / 59.5.  Every wave finds its place: where ranges are less than a round that is most of what it does,
// and they go as they come (180 requests, 43 tokens and one of 1 231: 55 us sorted, 43 so; 40 by the plan, 94 by eight waves).
struct CutArgs {
    uint64_t tag;
    int spare;
};
// What a workgroup of it takes: chunks c0 .. c1 - 1 of a range, which is one of `runs` parts of it (the at'th, `first` the item of the first).
struct CutItem {
    int r, hc, C, c0, c1, runs, at, first;
};
// Found by every wave for itself, K consecutive requests per lane.  False: nothing.
template <typename R, int K>
__device__ __forceinline__ bool cut_item(const DecodeArgs &a, const CutArgs &c, int item, CutItem &it)
{
    constexpr int kChunk = R::CT / R::GT, kUnit = kWaves * kChunk;
    const int lane = threadIdx.x & 63, HC = a.num_kv_heads * a.passes;
    int2 q[K];
    requests_of(a, K * lane, q);
    int n[K], np[K], sum = 0, longest = 0, running = 0, cuts = 0, upto = 0, own = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        n[k] = chunks_of(q[k].x, q[k].y, R::GT);
        np[k] = 0;
        sum += n[k];
        longest = max(longest, n[k]);
        running += __popcll(__ballot(n[k] > 0));
    }
    longest = __builtin_amdgcn_readlane(wave_max_to(longest), 63);
    const unsigned all = (unsigned)__builtin_amdgcn_readlane(wave_scan(sum), 63) * (unsigned)HC;
    const rules::CutSize size = rules::cut_size(all, c.spare, kUnit);
    if (longest > size.worth) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            np[k] = rules::cut_parts(n[k], size);
            own += np[k];
            running -= __popcll(__ballot(np[k] > 0));
        }
        upto = wave_scan(own);
        cuts = __builtin_amdgcn_readlane(upto, 63) * HC;
    }
    const int total = cuts + running * HC;
    // Every other 256 of them, one to a CU, the other way round: where the chip holds all at once a CU else has the longest of each
    // 256 (as they come / so, us: 4 layers of 32 requests of 60 to 1 500 tokens, 32 heads, 202 / 195; 128 of those on 32 / 8 heads 45.1 / 43.2).
    if ((item & 256) && (item | 255) < total) item ^= 255;
    if (item >= total) return false;
    if (item < cuts) {
        int at = split::small_div(item, HC);
        it.hc = item - at * HC;
        const int l = __popcll(__ballot(upto <= at));
        at -= __builtin_amdgcn_readlane(upto - own, l);
        int k = 0, of = __builtin_amdgcn_readlane(np[0], l), nr = __builtin_amdgcn_readlane(n[0], l);
        it.C = __builtin_amdgcn_readlane(q[0].y, l);
#pragma unroll
        for (int j = 1; j < K; ++j)
            if (k == j - 1 && at >= of) {
                at -= of;
                k = j;
                of = __builtin_amdgcn_readlane(np[j], l);
                nr = __builtin_amdgcn_readlane(n[j], l);
                it.C = __builtin_amdgcn_readlane(q[j].y, l);
            }
        it.r = K * l + k;
        const int each = rules::cut_each(nr, of, kChunk);
        it.runs = split::small_div(nr + each - 1, each);
        it.at = at;
        it.first = item - at * HC;
        it.c0 = at * each;
        it.c1 = min(nr, it.c0 + each);
        return it.at < it.runs;
    }
    // the request with the nth longest context (of those that run and are not cut; ties by place): its bits from the highest on
    int nth = split::small_div(item - cuts, HC);
    it.hc = item - cuts - nth * HC;
    unsigned key[K], top = 0;
    unsigned long long in[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        key[k] = np[k] == 0 ? (unsigned)n[k] : 0;
        top = max(top, key[k]);
        in[k] = __ballot(key[k] > 0);
    }
    if (all >= (unsigned)total * kUnit) {
        top = (unsigned)min(longest, size.worth);
        for (int bit = 31 - __builtin_clz(top); bit >= 0; --bit) {
            unsigned long long set[K];
            int m = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                set[k] = in[k] & __ballot(key[k] >> bit & 1);
                m += __popcll(set[k]);
            }
            const bool have = nth < m;
            if (!have) nth -= m;
#pragma unroll
            for (int k = 0; k < K; ++k) in[k] = have ? set[k] : in[k] & ~set[k];
        }
    }
    it.r = it.C = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int m = __popcll(in[k]);
        if (nth >= 0 && nth < m) {
            // (the lane with nth of them in front of it)
            const unsigned long long mine = __ballot((in[k] >> lane & 1) && __builtin_amdgcn_mbcnt_hi((unsigned)(in[k] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in[k], 0)) == (unsigned)nth);
            const int l = __ffsll((long long)mine) - 1;
            it.r = K * l + k;
            it.C = __builtin_amdgcn_readlane(q[k].y, l);
            nth = -1;
        } else if (nth >= 0) {
            nth -= m;
        }
    }
    it.c0 = 0;
    it.c1 = chunks_of(1, it.C, R::GT);
    it.runs = 1;
    it.at = it.first = 0;
    return true;
}

template <typename R>
__global__ __launch_bounds__(kThreads, R::kLeastPerCu) void decode_cut(const DecodeArgs a, const CutArgs c)
{
    constexpr int D = R::D;
    extern __shared__ __align__(16) float parts[];    // [wave][head][D + 2]
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int GH = a.heads_per_pass, HC = a.num_kv_heads * a.passes;
    CutItem it;
    if (a.batch <= kLaneBatch ? !cut_item<R, 1>(a, c, blockIdx.x, it) : !cut_item<R, 4>(a, c, blockIdx.x, it)) return;
    const size_t slot = (size_t)GH * (D + 2);
    const bool wide = ((uintptr_t)a.out & 15) == 0;
    float *mine = a.partials + (size_t)(it.first + it.at * HC) * slot;
    stretches<R, kWaves>(a, parts, wv, it.r, it.hc, it.c0, it.c1, it.C, [&](size_t rh, int h, int d, float M, float L, const float (&A)[2]) {
        if (it.runs == 1) {
            store_out<R::kBF16>(a.out, (rh + h) * D + d, wide, L, A);
        } else {
            put_shared(mine + h * (D + 2) + d, A[0], A[1]);
            if (d == 0) put_shared(mine + h * (D + 2) + D, M, L);
        }
    });
    if (it.runs == 1) return;
    uint64_t *flags = reinterpret_cast<uint64_t *>(a.partials + gridDim.x * slot);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    int *is_last = reinterpret_cast<int *>(parts);
    if (wv == 0) {
        const bool last = report_run<true>(flags + it.first, HC, it.at, it.runs, c.tag);
        if (lane == 0) *is_last = last;
    }
    __syncthreads();
    if (!*is_last) return;
    for (int i = 2 * (64 * wv + lane); i < GH * D; i += 128 * kWaves) {
        const int h = i / D, d = i % D;
        const float *x = a.partials + (size_t)it.first * slot + h * (D + 2);
        float M = kLowest, L = 0.0f, A[2] = {0.0f, 0.0f};
        for (int p0 = 0; p0 < it.runs; p0 += 8) {
            float2 ml[8], o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float *y = x + (size_t)min(p0 + j, it.runs - 1) * HC * slot;
                ml[j] = get_shared(y + D);
                o[j] = get_shared(y + d);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (p0 + j >= it.runs) break;
                const float Mn = fmaxf(M, ml[j].x), f0 = fast_exp2(M - Mn), f = fast_exp2(ml[j].x - Mn);
                L = L * f0 + ml[j].y * f;
                A[0] = A[0] * f0 + o[j].x * f;
                A[1] = A[1] * f0 + o[j].y * f;
                M = Mn;
            }
        }
        store_out<R::kBF16>(a.out, ((size_t)it.r * a.num_q_heads + it.hc * GH + h) * D + d, wide, L, A);
    }
}

// Few ranges, all of them in parts of one size, a workgroup each; the parts of a range are added up by a second launch, which works them out from the
// lengths as this one does, so neither launch has records of shares in front of its first byte: one request of 1 999 tokens, 32 / 8 heads, 9.3 -> 7.2 us
// (5.2 + 3.7 -> 4.3 + 2.8), one of 4 000 on 8 plain heads of 64 9.0 -> 7.8.
struct PartArgs {
    int even;                                         // parts of a range if all are alike: the launch's workgroups by the ranges there can be
    int most;                                         // ... at most: there is room for so many
};
struct Parts {
    int n, own, upto, size;                           // of the lane's request: chunks, parts, those of all up to it; chunks of a part at most
};
__device__ __forceinline__ Parts parts_of(const DecodeArgs &a, const PartArgs &c, int2 q, int GT, int chunk)
{
    Parts p;
    p.n = chunks_of(q.x, q.y, GT);
    p.size = rules::part_size(__builtin_amdgcn_readlane(wave_scan(p.n), 63), __builtin_amdgcn_readlane(wave_max_to(p.n), 63), a.batch, c.even, c.most, kWaves, chunk);
    for (int tries = rules::kPartTries;; --tries) {
        p.own = split::small_div(p.n + p.size - 1, p.size);
        p.upto = wave_scan(p.own);
        if (tries == 0 || __builtin_amdgcn_readlane(p.upto, 63) <= c.even * a.batch) return p;
        p.size += chunk;
    }
}
template <typename R>
__global__ __launch_bounds__(kThreads, R::kLeastPerCu) void decode_parts(const DecodeArgs a, const PartArgs c)
{
    constexpr int D = R::D, kChunk = R::CT / R::GT;
    extern __shared__ __align__(16) float parts[];    // [wave][head][D + 2]
    const int lane = threadIdx.x & 63, GH = a.heads_per_pass, HC = a.num_kv_heads * a.passes;
    const int2 q = request_of(a, lane);
    const Parts p = parts_of(a, c, q, R::GT, kChunk);
    int at = split::small_div(blockIdx.x, HC);
    const int hc = blockIdx.x - at * HC;
    const int r = __popcll(__ballot(p.upto <= at));   // the first whose parts end behind `at`
    if (r == 64) return;
    at -= __builtin_amdgcn_readlane(p.upto - p.own, r);
    const int of = __builtin_amdgcn_readlane(p.own, r), n = __builtin_amdgcn_readlane(p.n, r), C = __builtin_amdgcn_readlane(q.y, r);
    const int c0 = at * p.size;
    float *slot = a.partials + ((size_t)(r * HC + hc) * c.most + at) * GH * (D + 2);
    stretches<R, kWaves>(a, parts, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r, hc, c0, min(n, c0 + p.size), C,
                         [&](size_t rh, int h, int d, float M, float L, const float (&A)[2]) {
                             if (of == 1)
                                 store_out<R::kBF16>(a.out, (rh + h) * D + d, ((uintptr_t)a.out & 15) == 0, L, A);
                             else
                                 store_partial(slot + (size_t)h * (D + 2), D, d, M, L, A);
                         });
}

// Adds the parts of a range up: 128 (head, dim) outputs a workgroup, two per lane, its waves every eighth part.  One round trip where ranges are about
// alike: as many parts as they then have are asked for together with the lengths that say how many there are; a second one for those of longer ranges.
constexpr int kPartWaves = 8;
template <bool BF16>
__global__ __launch_bounds__(64 * kPartWaves) void decode_merge_parts(const DecodeArgs a, const PartArgs c, const int GT, const int chunk)
{
    constexpr int N = rules::kMostCuts / kPartWaves;
    __shared__ float4 sums[kPartWaves][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int D = a.head_dim, log2_D = __builtin_ctz(D);   // (a power of two)
    const int GH = a.heads_per_pass, HC = a.num_kv_heads * a.passes;
    const int range = blockIdx.x, r = range / HC, hc = range - r * HC;
    const int idx = min((int)blockIdx.y * 128 + 2 * lane, GH * D - 2), h = idx >> log2_D, d = idx & (D - 1);
    const int2 q = request_of(a, lane);
    float2 ml[N], ao[N];
    const auto ask = [&](int k) {
        const float2 *x = reinterpret_cast<const float2 *>(a.partials + (((size_t)range * c.most + wv + kPartWaves * k) * GH + h) * (D + 2));
        ml[k] = x[D / 2];
        ao[k] = x[d / 2];
    };
#pragma unroll
    for (int k = 0; k < N; ++k) {
        ml[k] = make_float2(kLowest, 0.0f);
        ao[k] = make_float2(0.0f, 0.0f);
        if (wv + kPartWaves * k < c.even) ask(k);     // uniform
    }
    const Parts p = parts_of(a, c, q, GT, chunk);
    const int runs = __builtin_amdgcn_readlane(p.own, r);
    if (runs <= 1) return;                            // does not run, or written already
    if (runs > c.even) {
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (wv + kPartWaves * k >= c.even && wv + kPartWaves * k < runs) ask(k);
    }
    float M = kLowest, L = 0.0f, A[2] = {0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (wv + kPartWaves * k >= runs) break;
        const float Mn = fmaxf(M, ml[k].x), f0 = fast_exp2(M - Mn), f = fast_exp2(ml[k].x - Mn);
        L = L * f0 + ml[k].y * f;
        A[0] = A[0] * f0 + ao[k].x * f;
        A[1] = A[1] * f0 + ao[k].y * f;
        M = Mn;
    }
    sums[wv][lane] = make_float4(M, L, A[0], A[1]);
    __syncthreads();
    if (wv > 0) return;
#pragma unroll
    for (int k = 1; k < kPartWaves; ++k) {
        const float4 o = sums[k][lane];
        const float Mn = fmaxf(M, o.x), f0 = fast_exp2(M - Mn), f = fast_exp2(o.x - Mn);
        L = L * f0 + o.y * f;
        A[0] = A[0] * f0 + o.z * f;
        A[1] = A[1] * f0 + o.w * f;
        M = Mn;
    }
    if (blockIdx.y * 128 + 2 * lane < GH * D)
        store_out<BF16>(a.out, ((size_t)r * a.num_q_heads + hc * GH + h) * D + d, ((uintptr_t)a.out & 15) == 0, L, A);
}

// N pieces of a split range (first, first + 1, ... in slot order; at most cnt of them), their loads
// in flight together, folded into the running (M, L, A0, A1) of the lane's two outputs.
template <int N>
__device__ __forceinline__ void merge_pieces(const float *partials, int w, int w_first, int first_slot, int cnt, int GH, int h,
                                             int D, int d, float &M, float &L, float &A0, float &A1)
{
    float2 ml[N], ao[N];                               // rows of the partials are 8-byte aligned
#pragma unroll
    for (int k = 0; k < N; ++k) {
        // the range's first share knows its slot; later ones start inside the range: slot 0
        ml[k] = make_float2(kLowest, 0.0f);
        ao[k] = make_float2(0.0f, 0.0f);
        if (k < cnt) {                                 // uniform
            const int slot = 2 * (w + k) + (w + k == w_first ? first_slot : 0);
            const float2 *x = reinterpret_cast<const float2 *>(partials + ((size_t)slot * GH + h) * (D + 2));
            ml[k] = x[D / 2];
            ao[k] = x[d / 2];
        }
    }
    float Mn = M;
#pragma unroll
    for (int k = 0; k < N; ++k) Mn = fmaxf(Mn, ml[k].x);
    const float f0 = fast_exp2(M - Mn);
    L *= f0;
    A0 *= f0;
    A1 *= f0;
    M = Mn;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float f = fast_exp2(ml[k].x - M);
        L += ml[k].y * f;
        A0 += ao[k].x * f;
        A1 += ao[k].y * f;
    }
}

// Merges the pieces of every (request, kv head / pass) that was split over several shares, in
// share order (= token order).  A workgroup looks at kMergeShares consecutive shares -- one wavefront
// each, and a slice of 128 (head, dim) outputs, two per lane -- and merges the ranges that start in
// them.  The wavefronts divide those ranges evenly: with one range per share each has one and
// works alone; with few and therefore long ranges (a small batch of long contexts: hundreds of
// pieces each) several wavefronts take a stretch of the same range's pieces and the first of them
// adds the stretches up, in order, through LDS.  Two round trips to memory, the share records and the
// pieces, whatever the lengths: up to 128 pieces are asked for at once.  (What the kernel costs is its
// launch and those round trips: 4.2-5.5 us on batches of 1 to 256 requests.  Before, a wave walked
// each range alone, eight pieces and a list of their slots at a time: the fp32 batch above, 21 pieces
// per range, 13.2 us, 12.2 with the waves sharing, 4.3 with a quarter of the pieces.)
constexpr int kMergeShares = 16;

template <bool BF16>
__global__ __launch_bounds__(64 * kMergeShares) void decode_merge_balanced(const DecodeArgs a, const int shares)
{
    __shared__ float4 stretch[kMergeShares][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = blockIdx.x * kMergeShares;
    int4 rec = make_int4(0, 0, 0, 0);                  // lane i: the record of share base + i
    if (lane < kMergeShares && base + lane < shares) rec = a.share_info[base + lane];
    const unsigned owners = (unsigned)__ballot(rec.w & kShareOwner);
    if (owners == 0) return;                           // uniform over the workgroup, like everything but `own` and `part`
    // Ranges of up to 8 pieces, one round of loads, are the work of the wave of their first share; nothing is
    // divided for them (the divisions below are 1 of the 6 us of a launch that has no use for them).
    const bool any_long = __any((rec.w & kShareOwner) && rec.z - (base + lane) >= 8);
    int own = wv, n = 1, parts = 1, part = 0;
    if (any_long) {
        n = __popc(owners);                            // ranges that start here
        parts = kMergeShares / n;
        part = wv / n;
        unsigned left = owners;
        for (int k = wv % n; k > 0; --k) left &= left - 1;
        own = __ffs((int)left) - 1;                    // this wave's range: the (wv % n)th of them
    } else if (!(owners >> wv & 1)) {
        return;
    }
    const int r = __builtin_amdgcn_readlane(rec.x, own), hc = __builtin_amdgcn_readlane(rec.y, own);
    const int w_first = base + own, w_last = __builtin_amdgcn_readlane(rec.z, own);
    const int first_slot = (__builtin_amdgcn_readlane(rec.w, own) & kShareSlot1) ? 1 : 0;
    const int D = a.head_dim, log2_D = __builtin_ctz(D);   // (a power of two)
    const int GH = a.heads_per_pass;
    const int idx = blockIdx.y * 128 + 2 * lane;       // the lane's two outputs: same head, d even
    const bool live = idx < GH * D;
    const int h = live ? idx >> log2_D : 0, d = live ? idx & (D - 1) : 0;
    float M = kLowest, L = 0.0f, A0 = 0.0f, A1 = 0.0f;
    const int each = any_long ? (w_last - w_first + parts) / parts : 8;
    const int w_end = min(w_last + 1, w_first + (part + 1) * each);
    if (part < parts)
        for (int w = w_first + part * each; w < w_end; w += 8)
            merge_pieces<8>(a.partials, w, w_first, first_slot, min(8, w_end - w), GH, h, D, d, M, L, A0, A1);
    if (parts > 1) {
        stretch[wv][lane] = make_float4(M, L, A0, A1);
        __syncthreads();
    }
    if (part > 0) return;
    if (parts > 1) {
        for (int k = 1; k < parts; ++k) {
            const float4 o = stretch[wv + k * n][lane];
            const float Mn = fmaxf(M, o.x), f0 = fast_exp2(M - Mn), f1 = fast_exp2(o.x - Mn);
            L = L * f0 + o.y * f1;
            A0 = A0 * f0 + o.z * f1;
            A1 = A1 * f0 + o.w * f1;
            M = Mn;
        }
    }
    if (live) {
        // (a group's heads follow each other, pass by pass: kv head and pass times GH is the first of this one)
        const size_t at = ((size_t)r * a.num_q_heads + hc * GH + h) * D + d;
        store_out<BF16>(a.out, at, L > 0.0f ? A0 / L : 0.0f);
        store_out<BF16>(a.out, at + 1, L > 0.0f ? A1 / L : 0.0f);
    }
}

// ---------------------------------------------------------------- launchers

// Bytes of partial states in the library's own scratch memory.  The form of a launch goes by the smaller of that and what a workspace has for the geometry,
// so that a call has the same results from either.
constexpr size_t kStaticPartialBytes = (size_t)LAMPS_STATIC_SCRATCH_BYTES - ((size_t)1 << 20);

// LDS of a decode_balanced launch.
template <typename R, bool TOGETHER>
size_t balanced_lds(int batch, int heads_per_pass)
{
    return balanced_ints(batch) * sizeof(int) + (TOGETHER ? (size_t)kWaves * heads_per_pass * (R::D + 2) * sizeof(float) : 0);
}

// Workgroups the chip holds at once for a decode_balanced<R, TOGETHER> launch: what the kernel's registers allow,
// asked once per device and instantiation (a later call may be under capture; every thread that asks gets the
// same), and what the launch's own LDS does.
template <typename R, bool TOGETHER>
hipError_t resident_workgroups(const DecodeArgs &a, int *out)
{
    static std::atomic<int> by_registers[kMaxDevices], cus_of[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int cus = cus_of[dev].load(std::memory_order_relaxed), per_cu = by_registers[dev].load(std::memory_order_relaxed);
    if (cus == 0 || per_cu == 0) {
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_balanced<R, TOGETHER>, kThreads, 0);
        if (e != hipSuccess) return e;
        if (cus < 1 || per_cu < 1) return hipErrorInvalidValue;
        cus_of[dev].store(cus, std::memory_order_relaxed);
        by_registers[dev].store(per_cu, std::memory_order_relaxed);
    }
    constexpr size_t kLds = (size_t)160 << 10, kStep = 2048;   // of a gfx950 CU; no allocation step is larger
    const size_t lds = (balanced_lds<R, TOGETHER>(a.batch, a.heads_per_pass) + 256 + kStep - 1) / kStep * kStep;
    *out = cus * min(min(per_cu, R::kMostPerCu), (int)(kLds / lds));      // (never none: 32 KiB for 8 192 requests, 66 for 16 heads of 256 together)
    return hipSuccess;
}

// The two launches of the balanced scheme over `wgs` workgroups.
template <typename R, bool TOGETHER>
hipError_t launch_balanced(const DecodeArgs &a, int wgs, hipStream_t s)
{
    const int HC = a.num_q_heads / a.heads_per_pass;
    const int P = wgs * (TOGETHER ? 1 : kWaves);
    DecodeArgs b = a;
    b.share_gcd = b.share_inv = b.share_period = 0;                    // shares in launch order
    if (wgs % 8 == 0) {                               // whole rounds over the XCDs: ranked shares
        int g = HC, t = P;
        while (t) { const int m = g % t; g = t; t = m; }
        // inverse of HC / g modulo P / g (the two are coprime), by the extended Euclidean algorithm
        const int period = P / g;
        long long r0 = period, r1 = HC / g % period, t0 = 0, t1 = 1;
        while (r1 > 1) {
            const long long q = r0 / r1, r2 = r0 - q * r1, t2 = t0 - q * t1;
            r0 = r1; r1 = r2; t0 = t1; t1 = t2;
        }
        b.share_gcd = g;
        b.share_period = period;
        b.share_inv = period > 1 ? (int)((t1 % period + period) % period) : 0;
    }
    hipLaunchKernelGGL((decode_balanced<R, TOGETHER>), dim3(wgs), dim3(kThreads), (balanced_lds<R, TOGETHER>(a.batch, a.heads_per_pass)),
                       s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int slices = (a.heads_per_pass * a.head_dim + 127) / 128;
    hipLaunchKernelGGL(decode_merge_balanced<R::kBF16>, dim3((P + kMergeShares - 1) / kMergeShares, slices), dim3(64 * kMergeShares), 0,
                       s, a, P);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_parts(const DecodeArgs &a, int HC, int even, int most, hipStream_t s)
{
    const PartArgs c = {even, most};
    hipLaunchKernelGGL(decode_parts<R>, dim3(a.batch * HC * (even + 1)), dim3(kThreads), (size_t)kWaves * a.heads_per_pass * (R::D + 2) * sizeof(float), s, a, c);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_merge_parts<R::kBF16>, dim3(a.batch * HC, (a.heads_per_pass * a.head_dim + 127) / 128), dim3(64 * kPartWaves), 0, s, a, c,
                       R::GT, R::CT / R::GT);
    return hipGetLastError();
}
template <typename R, int W>
hipError_t launch_whole(const DecodeArgs &a, int HC, hipStream_t s)
{
    constexpr int kPer = W > kWaves ? 1 : kWaves / W, kAll = kPer * W;   // ranges and waves of a workgroup
    hipLaunchKernelGGL((decode_whole<R, W>), dim3((unsigned)(((long long)a.batch * HC + kPer - 1) / kPer)), dim3(64 * kAll),
                       (size_t)kAll * a.heads_per_pass * (R::D + 2) * sizeof(float), s, a);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_cut(const DecodeArgs &a, int HC, bool matrix, hipStream_t s)
{
    const CutArgs c = {next_launch_tag(), rules::cut_spare(matrix)};
    hipLaunchKernelGGL(decode_cut<R>, dim3((unsigned)(a.batch * HC + c.spare)), dim3(kThreads), (size_t)kWaves * a.heads_per_pass * (R::D + 2) * sizeof(float), s, a, c);
    return hipGetLastError();
}

// demand != nullptr: nothing is launched; *demand receives the bytes of partial slots the
// balanced launch would use with every resident wavefront taking a share.
template <typename R>
hipError_t launch_one(const DecodeArgs &a, hipStream_t s, size_t *demand)
{
    const int G = a.num_q_heads / a.num_kv_heads;
    const int HC = a.num_kv_heads * (G / a.heads_per_pass);
    if (a.part_tokens > 0) {
        if (demand) return hipErrorInvalidValue;
        const long long items = (long long)a.max_parts * HC * a.batch;
        dim3 grid((unsigned)((items + kWaves - 1) / kWaves));
        hipLaunchKernelGGL(decode_partial<R>, grid, dim3(kThreads), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || a.max_parts == 1) return e;
        hipLaunchKernelGGL(decode_merge<R::kBF16>, dim3(a.num_q_heads, a.batch), dim3(a.head_dim), 0,
                           s, a);
        return hipGetLastError();
    }
    // balanced: as many workgroups as the chip holds at once for this kernel (fewer
    // if the partial slots of that many wave shares would not fit behind a.partials)
    int resident = 0, together = 0;                   // (both asked for at once, for the calls under capture)
    hipError_t e = resident_workgroups<R, false>(a, &resident);
    if (e == hipSuccess) e = resident_workgroups<R, true>(a, &together);
    if (e != hipSuccess) return e;
    const size_t per_share = decode_share_bytes(a.heads_per_pass, a.head_dim);
    if (demand) {
        *demand = (size_t)min(resident, kMaxShares / kWaves) * kWaves * per_share;
        return hipSuccess;
    }
    const size_t fit = min((size_t)kMaxShares, a.partial_capacity / per_share);
    const int wgs = min(resident, (int)(fit / kWaves));
    if (wgs < 1) return hipErrorInvalidValue;
    const bool matrix = decode_uses_tiled_layout(a.bf16, G);
    const rules::DecodeLaunch launch = {(long long)a.batch * HC, a.batch, a.head_dim, (long long)a.max_blocks * a.block_size, kWaves * R::CT, matrix,
                                        a.max_blocks <= a.num_blocks, (size_t)a.heads_per_pass * (R::D + 2) * sizeof(float),
                                        std::min({a.partial_capacity, (size_t)decode_max_shares(a.heads_per_pass, R::D) * per_share, kStaticPartialBytes})};
    switch (rules::decode_form(launch)) {
    case rules::kWholeTwo: return launch_whole<R, 2>(a, HC, s);
    case rules::kWholeFour: return launch_whole<R, kWaves>(a, HC, s);
    case rules::kWholeEight: return launch_whole<R, 8>(a, HC, s);
    case rules::kCut: return launch_cut<R>(a, HC, matrix, s);
    case rules::kParts: return launch_parts<R>(a, HC, rules::decode_cuts(launch), rules::decode_most_cuts(launch), s);
    case rules::kPlan: break;
    }
    // With eight waves and more to a range (if every request runs) they are better off together; with
    // six (16 requests of 60 to 1 500 tokens, 40 heads) the barriers cost 4 % more than they save.
    constexpr int kTogetherWaves = 8;
    if ((long long)a.batch * HC * kTogetherWaves <= (long long)wgs * kWaves)
        return launch_balanced<R, true>(a, min(together, wgs), s);
    return launch_balanced<R, false>(a, wgs, s);
}

template <bool BF16, int LPT>
hipError_t launch_valu(const DecodeArgs &a, hipStream_t s, size_t *demand)
{
    switch (a.heads_per_pass) {
    case 1: return launch_one<ValuReducer<BF16, LPT, 1, kHalves>>(a, s, demand);
    case 2:
        if constexpr (!BF16) return launch_one<ValuReducer<BF16, LPT, 2, kHalves>>(a, s, demand);
        break;                                 // grouped bf16 heads take the MFMA path
    case 4:
        if constexpr (!BF16) return launch_one<ValuReducer<BF16, LPT, 4, 1>>(a, s, demand);
        break;
    }
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_mfma(const DecodeArgs &a, hipStream_t s, size_t *demand)
{
    if (a.heads_per_pass > 16) return hipErrorInvalidValue;
    return launch_one<MfmaReducer<D>>(a, s, demand);
}

// Picks the instantiation for the geometry; launches, or (demand != nullptr) only asks.
hipError_t dispatch_impl(const DecodeArgs &a, hipStream_t stream, size_t *demand)
{
    const int G = a.num_q_heads / a.num_kv_heads;
    if (a.heads_per_pass != decode_heads_per_pass(a.bf16, a.head_dim, G) || a.heads_per_pass == 0)
        return hipErrorInvalidValue;
    const int lpt = a.head_dim * (a.bf16 ? 2 : 4) / 16;
    if (decode_uses_tiled_layout(a.bf16, G)) {
        if (a.head_dim == 64) return launch_mfma<64>(a, stream, demand);
        if (a.head_dim == 128) return launch_mfma<128>(a, stream, demand);
        if (a.head_dim == 256) return launch_mfma<256>(a, stream, demand);
    } else if (a.bf16) {
        if (lpt == 8) return launch_valu<true, 8>(a, stream, demand);
        if (lpt == 16) return launch_valu<true, 16>(a, stream, demand);
        if (lpt == 32) return launch_valu<true, 32>(a, stream, demand);
    } else {
        if (lpt == 8) return launch_valu<false, 8>(a, stream, demand);
        if (lpt == 16) return launch_valu<false, 16>(a, stream, demand);
        if (lpt == 32) return launch_valu<false, 32>(a, stream, demand);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t dispatch(const DecodeArgs &a, hipStream_t stream, size_t *demand) { return dispatch_impl(a, stream, demand); }

int decode_uses_tiled_layout(int bf16, int group) { return bf16 && group >= 2; }

int decode_heads_per_pass(int bf16, int head_dim, int group)
{
    const int lpt = head_dim * (bf16 ? 2 : 4) / 16;
    if (head_dim * (bf16 ? 2 : 4) % 16 != 0 || (lpt != 8 && lpt != 16 && lpt != 32)) return 0;
    if (group <= 0) return 0;
    if (decode_uses_tiled_layout(bf16, group)) {      // MFMA path: the largest divisor <= 16
        for (int gh = 16; gh >= 1; --gh)
            if (group % gh == 0) return gh;
    }
    if (group % 4 == 0) return 4;
    if (group % 2 == 0) return 2;
    return 1;
}

size_t decode_share_bytes(int heads_per_pass, int head_dim)
{
    return (size_t)2 * heads_per_pass * (head_dim + 2) * sizeof(float);
}

int decode_max_shares(int heads_per_pass, int head_dim)
{
    size_t n = kPartialBudget / decode_share_bytes(heads_per_pass, head_dim);
    if (n > (size_t)kMaxShares) n = kMaxShares;
    return (int)(n / kWaves) * kWaves;
}

hipError_t launch_decode(const DecodeArgs &a, hipStream_t stream)
{
    if (a.batch == 0) return hipSuccess;
    return dispatch(a, stream, nullptr);
}

}  // namespace lamps

// ---------------------------------------------------------------- decode without a workspace
//
// The balanced scheme's scratch memory -- the partial slots of split ranges and one int4 per
// share -- in a file-scope device array instead of the caller's workspace.  Every device the
// library runs on holds its own copy of the array, at its own address, until the process ends.
namespace {

constexpr size_t kStaticInfoBytes = (size_t)(lamps::kMaxShares + 1) * sizeof(int4);
static_assert(kStaticInfoBytes <= ((size_t)1 << 20), "share records must fit the last MiB");
static_assert(lamps::kStaticPartialBytes % 256 == 0, "the share records start 256-byte aligned");

static __device__ __align__(256) unsigned char scratch[LAMPS_STATIC_SCRATCH_BYTES];

// Device address of `scratch` on the current device.  The array's name is only a handle in host
// code: the address comes from hipGetSymbolAddress, once per device, with that device current.
hipError_t static_scratch(unsigned char **base)
{
    static std::atomic<unsigned char *> scratch_on[lamps::kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= lamps::kMaxDevices) return hipErrorInvalidDevice;
    unsigned char *ptr = scratch_on[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        scratch_on[dev].store(ptr, std::memory_order_release);   // every thread finds the same address
    }
    *base = ptr;
    return hipSuccess;
}

int static_fail(int code, const char *text)
{
    lamps::set_thread_error(text);
    return code;
}

}  // namespace

extern "C" int lamps_decode_attn_static(const lamps_config *cfg, void *compute_stream, int32_t layer,
                                        int32_t batch, const void *q, const void *k_pool, const void *v_pool,
                                        const int32_t *block_table, const int32_t *ctx_lens,
                                        const uint8_t *running_mask, void *out)
{
    lamps::DecodeArgs a;
    if (const char *why = lamps::decode_geometry(cfg, &a)) return static_fail(LAMPS_ERR_INVALID, why);
    if (cfg->part_tokens != 0)
        return static_fail(LAMPS_ERR_INVALID, "lamps_decode_attn_static: part_tokens must be 0 (balanced shares only)");
    if (!q || !k_pool || !v_pool || !block_table || !ctx_lens || !running_mask || !out)
        return static_fail(LAMPS_ERR_INVALID, "lamps_decode_attn_static: null argument");
    if (((uintptr_t)k_pool | (uintptr_t)v_pool | (uintptr_t)q | (uintptr_t)out) & 15)
        return static_fail(LAMPS_ERR_INVALID, "lamps_decode_attn_static: pools, q and out must be 16-byte aligned");
    if (layer < 0 || layer >= cfg->num_layers)
        return static_fail(LAMPS_ERR_RANGE, "lamps_decode_attn_static: layer out of range");
    if (batch < 0 || batch > cfg->max_batch)
        return static_fail(LAMPS_ERR_RANGE, "lamps_decode_attn_static: batch out of range");
    if (batch == 0) return LAMPS_OK;
    unsigned char *base = nullptr;
    hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return static_fail(LAMPS_ERR_HIP, hipGetErrorString(e));
    a.q = q;
    a.k_pool = k_pool;
    a.v_pool = v_pool;
    a.block_table = block_table;
    a.ctx_lens = ctx_lens;
    a.running = running_mask;
    a.out = out;
    a.batch = batch;
    a.layer = layer;
    a.partials = reinterpret_cast<float *>(base);
    a.partial_capacity = lamps::kStaticPartialBytes;
    a.share_info = reinterpret_cast<int4 *>(base + lamps::kStaticPartialBytes);
    size_t demand = 0;
    if ((e = lamps::dispatch(a, nullptr, &demand)) != hipSuccess)
        return static_fail(LAMPS_ERR_HIP, hipGetErrorString(e));
    if (demand > lamps::kStaticPartialBytes)
        return static_fail(LAMPS_ERR_RANGE,
                           "lamps_decode_attn_static: this geometry's partial slots (two records of heads per "
                           "pass x (head_dim + 2) floats per resident wavefront) exceed the static scratch buffer");
    // a launch of shares writes the record of every wavefront it starts and reads only those and the slots they name; the merge of parts may load a
    // slot that no part has written, and does not use it; parts that are handed over count by a tag of the call: nothing has to start at zero
    if ((e = lamps::dispatch(a, static_cast<hipStream_t>(compute_stream), nullptr)) != hipSuccess)
        return static_fail(LAMPS_ERR_HIP, hipGetErrorString(e));
    return LAMPS_OK;
}
