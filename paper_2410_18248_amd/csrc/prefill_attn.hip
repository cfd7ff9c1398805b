// Attention for several new tokens per request over the paged cache: what the
// Discard strategy's recompute, a new request's prompt and the processing of
// an API response need (arXiv 2410.18248, Section 1, Section 4.2: "Discard and
// Recompute"; Section 2.2 equation per token, each token over the cached
// positions up to and including its own).  The keys and values of the new
// tokens are already in the cache (lamps_kv_append_tokens).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "attn_reducers.h"
#include "handover.h"
#include "internal.h"
#include "prefill_rules.h"
#include "prefill_split.h"
#include "requests.h"

namespace lamps {
namespace {

// Last request r with q_start[r] <= n.
__device__ __forceinline__ int request_of(const int32_t *q_start, int batch, int n)
{
    int lo = 0, hi = batch;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (q_start[mid] <= n) lo = mid; else hi = mid;
    }
    return lo;
}

// One wavefront per (new token, kv head / pass): the decode reducer over the
// token's own prefix.  Every K/V byte is read once per new token, so this form
// is for the geometries the matrix-core kernels do not cover, and on request.
// (Head size 256, grouped heads: 262 registers, one workgroup to a CU.  Two, at 256 registers with the loads of a chunk behind the one
// before it, are slower: 8 requests of 200 to 300 new on 2 000 to 4 000, 16 / 4 heads, 2 090 us and 2 440; with loads in flight and 256 registers
// the loop spills: 2 896.)
template <typename R>
__global__ __launch_bounds__(kThreads) void prefill_rows(const PrefillArgs p)
{
    constexpr int D = R::D;
    const DecodeArgs &a = p.d;
    const int G = a.num_q_heads / a.num_kv_heads;
    const int GH = a.heads_per_pass;
    const int passes = G / GH;
    const int hc_count = a.num_kv_heads * passes;
    const long long item = (long long)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (item >= (long long)p.total_tokens * hc_count) return;
    const int hc = (int)(item % hc_count);
    const int n = (int)(item / hc_count);
    const int r = __builtin_amdgcn_readfirstlane(request_of(p.q_start, a.batch, n));
    const int first = p.q_start[r], count = p.q_start[r + 1] - first;
    if (n >= first + count) return;
    const int C = a.ctx_lens[r];
    // a context shorter than its new tokens, or longer than the block-table row, is the caller's
    // mistake: nothing is read or written for it
    if (C - count < 0 || C > a.max_blocks * a.block_size) return;
    const int t_end = C - count + (n - first) + 1;    // its own position included
    const int g = hc / passes;
    const int h0 = g * G + (hc % passes) * GH;
    const size_t row0 = (size_t)n * a.num_q_heads + h0;
    const bool wide = ((uintptr_t)a.out & 15) == 0;
    R::run(a, r, (size_t)n, g, h0, GH, 0, max(t_end, 0), [&](int h, int d, float, float L, const auto &A) {
        store_out<R::kBF16>(a.out, (row0 + h) * D + d, wide, L, A);
    });
}

// Which request, kv head (or pass) of `heads` and tile of new tokens a workgroup takes, and the
// request's first row, new rows and context length; false: none.
//
// full_groups >= 0: a grid of (request, head) pairs x tiles, tiles being the most any request has.
// All tiles of one pair run on one XCD (workgroups are dealt to the 8 XCDs round-robin in launch
// order), so its K/V stream is fetched into one L2 and shared there; consecutive heads go to
// different XCDs; the longest tiles of a pair, or of the pairs that go abreast (p.slots of them, or
// as the contexts say), start first.  That holds for the pairs that fill whole
// groups of 8; the (pair, tile) items of the remaining 1..7 pairs are dealt round-robin over all
// XCDs instead of leaving some of them empty.
//
// full_groups < 0, for ragged batches: only the tiles there are, (tile, request, head) with the last
// tiles first, found by every wave from q_start, a few requests per lane.  A workgroup without a
// tile holds its slot (LDS and registers) for 2 us, and workgroups start in order: 24 prompts of 16 to
// 700 tokens on 40 heads kept 300 to 440 of 512 slots busy with 5 760 workgroups for 1 560 tiles, and
// 400 to 512 this way: 55 -> 48 us for the kernel.  With the number of heads a multiple of 8 a pair's
// tiles stay on one XCD here too.  More requests than a wave keeps (kByStart): numbered by request, each
// getting the tiles it can have at most, its start in tiles plus one per request before it.
constexpr int kRagged = 4;               // requests per lane
constexpr int kByStart = -2;
struct Place {
    int r, head, tile, first, n_new, ctx;
};
template <bool BY_START>
__device__ __forceinline__ bool place(const PrefillArgs &p, int heads, int tiles, int full_groups, int WT, bool two_per_cu, Place &at)
{
    const DecodeArgs &a = p.d;
    if (full_groups >= 0) {
        const int pairs = heads * a.batch;
        int abreast = p.slots;
        if (abreast == 0) {
            const int lane = threadIdx.x & 63;
            const int longest = __builtin_amdgcn_readlane(wave_max_to(lane < a.batch ? a.ctx_lens[lane] : 0), 63);
            abreast = __builtin_amdgcn_readfirstlane(rules::pairs_abreast({p.longest, p.part}, longest, full_groups));
        }
        const rules::Turn turn = rules::deal(blockIdx.x, pairs, full_groups, tiles, abreast);
        const int pair = turn.pair;
        int t = turn.t;
        // Where all run at once, two to a CU (the 32 CUs of an XCD are dealt to in turn), and the
        // second turn begins with a pair, its pairs start with their short tiles, so that a CU has
        // a long and a short one: 4 prompts of 512 on 16 heads of 256, append included, 41.2 -> 37.6
        // us, 2 of 1 000 54.6 -> 49.3; fp32, 2 of 512 on 8 heads of 64, 17.0 -> 12.8, 2 of 256 on 16 of 128,
        // 19.6 -> 15.2.  (Beginning inside a pair's tiles: 2 % slower than without.)  Not where a CU holds
        // one workgroup: the second turn then waits for the first, and has to begin with its long tiles
        // (4 prompts of 512, 32 / 4 heads of 256: 55.3 us, 42.3 in order).
        if (two_per_cu && gridDim.x <= 512 && 32 % tiles == 0 && turn.slot >= 0 && (turn.slot & 32)) t = tiles - 1 - t;
        if (t >= tiles) return false;
        at.tile = tiles - 1 - t;
        at.r = pair / heads;
        at.head = pair - at.r * heads;
        at.first = p.q_start[at.r];
        at.n_new = p.q_start[at.r + 1] - at.first;
        if (at.tile * WT >= at.n_new) return false;
        at.ctx = a.ctx_lens[at.r];
    } else if (BY_START && full_groups == kByStart) {
        const int item = blockIdx.x / heads;
        at.head = blockIdx.x - item * heads;
        at.r = last_request(p.q_start, a.batch, item, [WT](int start, int r) { return start / WT + r; });
        at.first = p.q_start[at.r];
        at.n_new = p.q_start[at.r + 1] - at.first;
        at.ctx = a.ctx_lens[at.r];
        at.tile = item - (at.first / WT + at.r);
        if (at.tile >= tiles || at.tile * WT >= at.n_new) return false;
    } else {
        const int lane = threadIdx.x & 63;
        int first[kRagged], n_new[kRagged], ctx[kRagged], n_tiles[kRagged], most = 0;
#pragma unroll
        for (int k = 0; k < kRagged; ++k) {
            const int r = 64 * k + lane;
            first[k] = n_new[k] = ctx[k] = n_tiles[k] = 0;
            if (64 * k < a.batch && r < a.batch) {
                first[k] = p.q_start[r];
                n_new[k] = p.q_start[r + 1] - first[k];
                ctx[k] = a.ctx_lens[r];
                n_tiles[k] = n_new[k] > 0 ? min((n_new[k] + WT - 1) / WT, tiles) : 0;
            }
            most = max(most, n_tiles[k]);
        }
        // tiles of index t and above, of one head; decreasing in t
        auto above = [&](int t) {
            int n = 0;
#pragma unroll
            for (int k = 0; k < kRagged; ++k) n += max(0, n_tiles[k] - t);
            return __builtin_amdgcn_readlane(wave_scan(n), 63);
        };
        int left = blockIdx.x / heads;                    // requests' tiles before this one
        at.head = blockIdx.x - left * heads;
        at.r = -1;
        // the level: above(lo) > left >= above(hi).  (One level after the other, 45 of them on prompts of
        // up to 1 413 tokens with 4 heads per kv head, was 2 us and made that launch 5 % slower than the
        // full grid.)
        int lo = 0, hi = __builtin_amdgcn_readlane(wave_max_to(most), 63);
        if (above(0) <= left) return false;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (above(mid) > left) lo = mid; else hi = mid;
        }
        left -= above(lo + 1);
        at.tile = lo;
#pragma unroll
        for (int k = 0; k < kRagged; ++k)
            if (64 * k < a.batch && at.r < 0) {
                const unsigned long long have = __ballot(n_tiles[k] > lo);
                const int n = __popcll(have);
                if (left < n) {
                    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(have >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)have, 0));
                    const int l = __ffsll((long long)__ballot(n_tiles[k] > lo && before == left)) - 1;
                    at.r = 64 * k + l;
                    at.first = __builtin_amdgcn_readlane(first[k], l);
                    at.n_new = __builtin_amdgcn_readlane(n_new[k], l);
                    at.ctx = __builtin_amdgcn_readlane(ctx[k], l);
                } else {
                    left -= n;
                }
            }
        if (at.r < 0) return false;
    }
    // a context shorter than its new tokens, or longer than the block-table row, is the caller's
    // mistake: nothing is read or written for it
    return at.ctx >= at.n_new && at.ctx <= a.max_blocks * a.block_size;
}
// The grid for it and what place() needs to know; 0: too large.  `spare`: workgroups without a tile that
// cost less than finding one's place among the tiles there are.  `chip`: workgroups it holds at once.
unsigned place_grid(PrefillArgs &p, long long heads, long long tiles, int WT, bool by_start, int spare, int chip, int *full_groups)
{
    const long long pairs = heads * p.d.batch, full = pairs / 8, rest = pairs % 8;
    long long grid = full * tiles * 8 + (rest * tiles + 7) / 8 * 8;
    *full_groups = (int)full;
    // the tiles of all requests are at most this many; a quarter fewer workgroups pay for finding them
    const long long most = heads * ((long long)p.total_tokens / WT + p.d.batch);
    // With a number of heads that is no multiple of 8 a pair's tiles, numbered so, lie on several XCDs and each
    // fetches the pair's K / V.  That does not pay where the chip holds the full grid at once, nor for short
    // walks, which leave no long tail to fill (2 kv heads of 128, 8 heads, append + attention: 16 prompts of 45 to
    // 278 tokens 17.7 us together, 18.9 apart; 100 of 10 to 200 32.4 and 34.7; but 24 of 16 to 700 49 and 38, and
    // with 40 of 45 to 278 on 1 000 cached it is 54.4 and 53.8, with heads of 64 45 and 39).
    const bool short_walks = p.max_new_tokens < 320 && (long long)p.d.max_blocks * p.d.block_size < 640;
    const bool together = !by_start && p.d.head_dim < 256 && heads % 8 != 0 && (grid <= chip || short_walks);
    if (!together && (by_start || p.d.batch <= 64 * kRagged) && most + most / 4 + spare < grid) {
        grid = most;
        *full_groups = p.d.batch <= 64 * kRagged ? -1 : kByStart;
    }
    const rules::Launch launch = {(int)heads, p.d.num_q_heads / p.d.num_kv_heads, p.d.head_dim, p.d.batch, p.total_tokens,
                                  p.max_new_tokens, (long long)p.d.max_blocks * p.d.block_size};
    p.slots = 1;
    if (*full_groups >= 0) {
        const rules::Together w = rules::together(launch, p.d.bf16 ? 4 : 8, tiles, grid, most, (int)full, chip);
        p.longest = w.longest;
        p.part = w.part;
        if (w.longest > 0) p.slots = launch.row <= w.longest ? rules::pairs_abreast(w, (int)launch.row, (int)full) : p.d.batch <= 64 && launch.most >= 128 ? 0 : 1;
    }
    return tiles < 1 || grid > 0x7fffffffLL ? 0u : (unsigned)grid;
}

// ---------------------------------------------------------------- matrix cores, 32 bits

// fp32.  A workgroup takes one tile of 16 columns -- (new token, head of the pass) pairs of one kv
// head -- and its four waves every fourth chunk of 16 positions each; their states are added up
// through LDS.  Bound by the fp32 matrix rate on long prompts (each K / V byte from L2 serves 16
// columns) and by the walk over the positions on short ones, which is why the waves share it:
// six prompts of 17 to 700 tokens, 8 heads of 64: 27 us with a wavefront per token on the vector ALUs
// (every K / V byte read once per token), 14 now.  At head_dim 128 the register bound is what keeps two
// workgroups on a CU: one register more than 256 and one CU holds one, for 25 to 75 % of the time.
// Heads of a group that share a tile: the largest divisor up to 16.
__host__ __device__ __forceinline__ int f32_tile_heads(int group)
{
    int gh = group < 16 ? group : 16;
    while (group % gh) --gh;
    return gh;
}

template <int D>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 1) void prefill_tiles_f32(const PrefillArgs p, const int tiles, const int full_groups)
{
    typedef MfmaF32Tile<D> R;
    constexpr int ROW = D + 4;                        // floats; 16-byte aligned, rows in different banks
    __shared__ __align__(16) float part[kWaves][16][ROW];
    __shared__ float2 stat[kWaves][16];
    const DecodeArgs &a = p.d;
    const int G = a.num_q_heads / a.num_kv_heads, GH = f32_tile_heads(G), passes = G / GH, HC = a.num_kv_heads * passes;
    const int TW = 16 / GH;                           // new tokens per tile
    Place at;
    if (!place<true>(p, HC, tiles, full_groups, TW, true, at)) return;
    const int r = at.r, tile = at.tile, first = at.first, n_new = at.n_new, base_pos = at.ctx - n_new;
    const int g = at.head / passes, h0 = at.head * GH;
    const int lane = threadIdx.x & 63, j = lane & 15, qd = lane >> 4, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int toks = min(TW, n_new - tile * TW);
    const int tok = j / GH;                           // this lane's column: token tile * TW + tok, head h0 + j % GH
    const bool ok = tok < toks;
    const float *q = static_cast<const float *>(a.q) + ((size_t)(first + tile * TW + tok) * a.num_q_heads + h0 + j % GH) * D;
    const int seen = base_pos + tile * TW + 1;        // positions the tile's first token attends to
    typename R::State st;
    R::reduce(a, r, g, ok ? q : nullptr, ok ? seen + tok : 0, seen, 16 * wv, seen + toks - 1, kWaves, st);
    if (qd == 0) stat[wv][j] = make_float2(st.m, st.l);
#pragma unroll
    for (int c = 0; c < R::NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < R::VW; ++v) part[wv][j][16 * R::VW * c + R::VW * (4 * qd + e) + v] = st.o[c][v][e];
    __syncthreads();
    const int col = threadIdx.x >> 4, x = threadIdx.x & 15, t = col / GH;
    if (t >= toks) return;
    float M = kLowest, L = 0.0f, f[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, stat[w][col].x);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        f[w] = fast_exp2(stat[w][col].x - M);
        L += stat[w][col].y * f[w];
    }
    float *out = static_cast<float *>(a.out) + ((size_t)(first + tile * TW + t) * a.num_q_heads + h0 + col % GH) * D;
    for (int d = 4 * x; d < D; d += 64) {
        f32x4 A = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const f32x4 o = *reinterpret_cast<const f32x4 *>(&part[w][col][d]);
#pragma unroll
            for (int e = 0; e < 4; ++e) A[e] += o[e] * f[w];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) A[e] = L > 0.0f ? A[e] / L : 0.0f;
        *reinterpret_cast<f32x4 *>(out + d) = A;
    }
}

template <int D>
hipError_t launch_tiles_f32(PrefillArgs p, hipStream_t s)
{
    const int GH = f32_tile_heads(p.d.num_q_heads / p.d.num_kv_heads), TW = 16 / GH;
    const long long tiles = (p.max_new_tokens + TW - 1) / TW;
    int full = 0;
    // Up to 1 024 workgroups for nothing cost less than finding the tiles there are: 3 prompts of 100 to 500 tokens,
    // 8 heads of 64 (768 workgroups, 400 tiles), 10.2 us on the full grid, 11.8 ragged; 12 of 8 to 300, 16 / 2
    // heads (3 600 and 1 000), 25.5 and 15.4.  The full grid alone grew with requests x tokens where the most
    // new tokens are not known: 64 prompts of 100, 32 / 8 heads of 128, 1 200 us, 203 so.
    const unsigned grid = place_grid(p, p.d.num_q_heads / GH, tiles, TW, true, 1024, 512, &full);
    if (grid == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prefill_tiles_f32<D>, dim3(grid), dim3(kThreads), 0, s, p, (int)tiles, full);
    return hipGetLastError();
}

// ---------------------------------------------------------------- matrix cores, bf16

// bf16, up to 32 query heads per kv head.  With many new tokens per request both
// products of the Section 2.2 equation are real contractions: for one kv head,
// the (token, head-of-group) pairs are the columns of a query matrix, and every
// 32 cached positions cost 2 D/32 + D/16 + 1 MFMAs (16x16x32) per 16 columns.
//
// One workgroup = one (request, kv head, tile of new tokens); its four waves each
// own kCols = 32 columns (16 in launches of few rounds, and at head_dim 256; kCols / G tokens x G heads) as blocks of 16.  K and V
// are streamed 32 positions at a time through LDS: while stage s is consumed,
// stage s + 1 arrives in the other of two LDS buffers, straight from the pools (loads
// that write LDS directly: no registers, no LDS-write instructions), one barrier
// per stage -- or per two stages, loaded and published together, when a request has
// several tiles of new tokens and two such groups fit the 64 KiB of a workgroup.  Every wave reads each K / V operand from LDS
// once per stage and uses it for both column blocks.  Scores come out transposed
// (lane: four consecutive positions of one column), which is the operand layout
// the second product wants for the weights, so nothing is shuffled between the
// two; the positions of a stage's two 16-position halves share one 32-deep MFMA
// (the contraction index may be permuted as long as both operands agree).
//
// The loop is software-pipelined around its one barrier: a stage's V operands are
// read from LDS before its scores are computed and used after the barrier, the
// next stage's K operands are read right after the barrier and used at the top of
// the next iteration, so LDS latency is behind MFMA or softmax work both times.
//
// The vector ALUs are the scarce unit (an exponential costs as much issue time as
// a quarter of an MFMA), so everything that is not the softmax itself is kept off
// them: block-table entries are looked up one stage ahead through the scalar
// unit, the causal mask is applied only in the stages that straddle a column's own
// position, the weights' sums come from one more MFMA against a vector of ones
// (they accumulate, like the outputs, in registers and need no cross-lane sum at
// the end), and V reaches the second product without any shuffling in registers.
//
// LDS layouts of a stage: the pools' tiles as they are.  Tiled pool layout: a K unit
// is an operand already, a V operand is the first or the second 8 bytes of the same
// unit of the stage's two sub-tiles.  Plain layout: K and V row-major; rows cannot
// be padded on the way in, so the 16-byte units of a row are permuted instead (unit
// s of row r sits in slot s ^ r, or s ^ 2 r for V) and the rows an operand read
// touches fall in different banks; V^T operands come out of the transposing LDS
// read of gfx950 (ds_read_b64_tr_b16: the 16 lanes of a group read four rows of 16
// dims, lane j receives dim j of the four rows).
constexpr int kMaxCols = 32;             // columns per wave: two blocks of 16 keep a wave under 256 registers,
                                         // so two workgroups share a CU and cover each other's stalls
constexpr int kStage = 32;               // cached positions per LDS stage
constexpr float kSlack = 8.0f;           // log2 of the largest weight before the reference moves

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(4))) const int32_t *table_ptr;   // read-only: scalar loads

// s_waitcnt immediate: wait until at most n of the wave's vector memory operations are outstanding
constexpr int vmcnt(int n) { return 0x0F70 | (n & 15) | (n >> 4) << 14; }

// Splitting a tile's cached positions.  One workgroup per (request, kv head, tile) leaves most of
// the chip idle when few requests bring few new tokens -- the API responses of a dozen requests
// are 100 to 200 workgroups, each a serial walk over a whole context.  Then the stages of the tiles
// are cut into runs (prefill_split.h), each a workgroup of its own that leaves its columns'
// (reference, sum, unnormalised output) in the workspace; the last of a tile to do so adds them up
// in order.  The references of the runs differ from that of an uncut walk, and so do the roundings of
// the bf16 weights: a request's output depends on how it is cut, that is on the other requests of the
// call, by what another order of the same sums gives.
// Bound by the walk over K / V and the hand-over: a dozen requests with 6 to 58 new tokens on 345 to
// 2 490 cached, 32 / 8 heads of 128 (50 MB): 63 us for this kernel before, 24 now; one request with 16
// new on 3 000: 75 us before, 20 now.  (Adding the runs up in a second launch instead is 1-8 us faster
// on such a call and 4 us slower on every one that has nothing to add up.)
constexpr int kSplitSlots = 512;         // two workgroups per CU
constexpr int kSplitRequests = 64;       // one per lane
constexpr int kWhole = 1 << 26;          // stages per run of a request that is not cut: more than any context has
constexpr int kSplitStages = 32;         // a block-table row of fewer (1024 positions) is not split

struct Run {
    int r, g, tile;                      // request, kv head, tile of new tokens (r < 0: nothing to do)
    int first, n_new, ctx;               // of the request: first new row, new rows, context length
    int item, first_item, stride;        // the workgroup's item (= partial slot); those of the tile's runs
    int index, per;                      // which of the tile's runs, and stages per run
};

// What a workgroup of a split launch is to do.  Every wave works it out for itself from q_start and
// ctx_lens, one request per lane: one round trip to memory, no barrier.  (The launcher has checked that
// the sums fit 32 bits.)
template <int D, bool WIDE, int GRP>
__device__ __forceinline__ Run locate(const PrefillArgs &p, int tiles, int WT)
{
    const DecodeArgs &a = p.d;
    const int lane = threadIdx.x & 63;
    int first = 0, n_new = 0, ctx = 0, stages = 0, n_tiles = 0;
    if (lane < a.batch) {
        first = p.q_start[lane];
        n_new = p.q_start[lane + 1] - first;
        ctx = a.ctx_lens[lane];
        // a context shorter than its new tokens, or longer than the block-table row, is the
        // caller's mistake: nothing is read or written for it
        if (n_new > 0 && ctx >= n_new && ctx <= a.max_blocks * a.block_size) {
            n_tiles = split::tiles_of(n_new, WT, tiles);
            stages = (ctx - 1) / kStage + 1;          // of the last tile; no tile has more
        }
    }
    split::Sums sums;
    sums.stages = __builtin_amdgcn_readlane(wave_scan(stages * n_tiles), 63);
    sums.tiles = __builtin_amdgcn_readlane(wave_scan(n_tiles), 63);
    sums.most = WIDE ? __builtin_amdgcn_readlane(wave_max_to(stages), 63) : 0;
    const split::Cut cut = split::cut_of(sums, p.head_slots, a.num_kv_heads, GRP, D, WIDE);
    int runs = 1;
    if (__any(stages > cut.worth)) runs = split::runs_of(stages, cut, p.slots);
    const int items = n_tiles * runs * a.num_kv_heads, upto = wave_scan(items);
    Run run;
    run.item = split::item_of(blockIdx.x, __builtin_amdgcn_readlane(upto, 63), p.slots);
    run.r = __ffsll((long long)__ballot(run.item >= upto - items && run.item < upto)) - 1;
    if (run.r < 0) return run;                        // (no items: those of -1, too)
    const int nt = __builtin_amdgcn_readlane(n_tiles, run.r), nr = __builtin_amdgcn_readlane(runs, run.r);
    const split::Piece at = split::piece_of(run.item - __builtin_amdgcn_readlane(upto - items, run.r), nt, nr);
    run.g = at.head;
    run.tile = at.tile;
    run.first = __builtin_amdgcn_readlane(first, run.r);
    run.n_new = __builtin_amdgcn_readlane(n_new, run.r);
    run.ctx = __builtin_amdgcn_readlane(ctx, run.r);
    run.stride = nt;
    run.first_item = run.item - at.run * nt;
    run.index = at.run;
    run.per = nr > 1 ? cut.per : kWhole;
    return run;
}

// Memory of a split launch behind DecodeArgs::partials, per item: the unnormalised outputs of each
// block of 16 columns as its wave holds them, [pair of registers][lane] -- whole lines, written and
// read by 512 contiguous bytes per instruction (by column, in pieces of 8 bytes, the hand-over of a
// tile took 25 us) --, the columns' (reference, sum), and a flag that they are there.
constexpr size_t split_item_bytes(int D, int columns) { return (size_t)columns * (D + 2) * sizeof(float) + sizeof(uint64_t); }

// Stores a column's N slabs of 16 outputs, those of quarter qd being 4 qd .. of each.  Odd and even quarters exchange halves of
// two slabs, so that a lane stores 16 bytes and an instruction 64 of a row: by 8 and 32, 24 prompts of 16 to 700 tokens on 40 heads took
// 42.0 us, 39.2 so; 12 of 100 to 700 on 32 / 8 heads 30.4 and 27.5.  By a whole wave, which leaves where none of its columns is a row (8 tokens, 16 / 8
// heads of 256: 6.2 us with all blocks exchanged, 5.7 so).
template <int N, typename Slabs>
__device__ __forceinline__ void store_column(uint16_t *dst, int qd, bool mine, float inv, const Slabs &o)
{
    static_assert(N % 2 == 0, "slabs go in pairs");
    if (!__any(mine)) return;
#pragma unroll
    for (int s = 0; s < N; s += 2) {
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = pack_bf16(o[s + (k >> 1)][2 * (k & 1)] * inv, o[s + (k >> 1)][2 * (k & 1) + 1] * inv);
        const auto x0 = __builtin_amdgcn_permlane16_swap(w[0], w[2], false, false);
        const auto x1 = __builtin_amdgcn_permlane16_swap(w[1], w[3], false, false);
        if (mine) *reinterpret_cast<uint4 *>(dst + 16 * (s + (qd & 1)) + 8 * (qd >> 1)) = make_uint4(x0[0], x1[0], x0[1], x1[1]);
    }
}

// The kernels of narrow tiles: more than two workgroups to a CU.
template <int D, int kCols, int GRP, bool SPLIT>
constexpr bool kSmall = D <= 128 && kCols <= 16 && GRP == 1 && !SPLIT;

template <int D, bool TILED, int kCols, int GRP, bool SPLIT>
__global__ __launch_bounds__(kThreads, (D >= 256 && kCols <= 16) ? 2 : (kSmall<D, kCols, GRP, SPLIT>) ? (D == 128 && TILED ? 3 : 4) : 1) void prefill_mfma(const PrefillArgs p, const int tiles, const int full_groups)
{
    constexpr int kColBlocks = kCols / 16;
    constexpr int NK = D / 32;                       // score MFMAs per 16 positions
    constexpr int NS = D / 16;                       // 16-dim slabs of the output
    constexpr int U = D * 2;                         // 16-byte units of one 16-position sub-tile
    constexpr int LPT = (2 * U) / kThreads;          // units per thread, pool and stage
    // The pool's tiles go to LDS as they are, by loads that write LDS directly
    // (global_load_lds_dwordx4: lane l of a wave writes 16 bytes at base + 16 l, read from any
    // address); two stage buffers (64 KiB at head_dim 256).
    constexpr int NB = SPLIT && D <= 128 && GRP == 1 ? 4 : 2;   // group buffers
    constexpr int NU = D / 8;                        // 16-byte units of one row (plain layout)
    constexpr int SUBB = 16 * D * 2;                 // one 16-position sub-tile of K or V
    constexpr int VOFF = 2 * SUBB;                   // V follows the two K sub-tiles
    constexpr int STAGE = 4 * SUBB;
    // Stages are loaded, and published by a barrier, GRP at a time: with two, half as many
    // barriers and waits for loads, and a group's loads have twice as long to arrive.
    constexpr int GSTAGE = GRP * STAGE;
    static_assert(NB * GSTAGE <= 65536, "LDS of one workgroup");
    static_assert(LPT >= 1 && (2 * U) % kThreads == 0, "head_dim");
    __shared__ __align__(16) char lds[NB * GSTAGE];

    const DecodeArgs &a = p.d;
    const int TW = kCols / (a.num_q_heads / a.num_kv_heads);   // new tokens per wave (G <= kCols)
    const int WT = kWaves * TW;                      // ... per workgroup
    int r, g, tile, first, n_new, C;
    int item = 0, st0 = 0, per = 0x7fffffff;         // SPLIT: the workgroup's item, first stage, most stages,
    int first_item = 0, item_stride = 0;             // ... and the items of its tile's runs
    if constexpr (SPLIT) {
        const Run run = locate<D, (D >= 256 || kCols > 16), GRP>(p, tiles, WT);
        if (run.r < 0) return;
        item = run.item;
        r = run.r;
        g = run.g;
        tile = run.tile;
        first = run.first;
        n_new = run.n_new;
        C = run.ctx;
        per = run.per;
        first_item = run.first_item;
        item_stride = run.stride;
        st0 = run.index * per;
    } else {
        Place at;
        if (!place<false>(p, a.num_kv_heads, tiles, full_groups, WT, !(D >= 256 && kCols > 16), at)) return;
        r = at.r;
        g = at.head;
        tile = at.tile;
        first = at.first;
        n_new = at.n_new;
        C = at.ctx;
    }
    const int G = a.num_q_heads / a.num_kv_heads;
    const int base_pos = C - n_new;                  // position of the request's first new token
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, qd = lane >> 4;

    // the wave's columns see the positions up to wave_maxpos, every one of them those up to wave_minpos
    const int wave_tok = tile * WT + wv * TW;        // the wave's first new token
    const int wave_maxpos = __builtin_amdgcn_readfirstlane(wave_tok < n_new ? base_pos + min(n_new, wave_tok + TW) - 1 : -1);
    const int wave_minpos = __builtin_amdgcn_readfirstlane(wave_tok < n_new ? base_pos + wave_tok : 0x7fffffff);
    int wg_maxpos = base_pos + min(n_new, (tile + 1) * WT) - 1;
    int n_stages = wg_maxpos / kStage + 1;
    int n_runs = 1;                                   // workgroups that share the tile
    if constexpr (SPLIT) {
        if (st0 >= n_stages) return;                  // a tile before the request's last one has fewer
        if (n_stages > per) {
            n_runs = (int)((unsigned)(n_stages + per - 1) / (unsigned)per);
            n_stages = min(n_stages, st0 + per);
        }
        wg_maxpos = min(wg_maxpos, n_stages * kStage - 1);
    }

    const table_ptr table = (table_ptr)(uintptr_t)(a.block_table + (size_t)r * a.max_blocks);
    const uint32_t tile_bytes = (uint32_t)a.block_size * D * 2;
    // bytes from one block to the next; the launcher has checked that they fit 32 bits
    const uint32_t block_stride = (uint32_t)a.num_layers * a.num_kv_heads * tile_bytes;
    const size_t head_off = ((size_t)a.layer * a.num_kv_heads + g) * tile_bytes;
    const char *kp = static_cast<const char *>(a.k_pool) + head_off;
    const char *vp = static_cast<const char *>(a.v_pool) + head_off;

    // Block-table entries of a group's sub-tiles: wave-uniform, through the scalar unit, and
    // looked up one iteration before the loads that use them so that nobody waits for them.
    uint32_t ent[2 * GRP];
    const uint32_t last_entry = (uint32_t)wg_maxpos >> a.log2_block_size;   // nothing past it is looked up
    const uint32_t last_block = (uint32_t)a.num_blocks - 1;
    auto lookup = [&](int grp, uint32_t (&ent)[2 * GRP]) {
        const uint32_t t0 = (uint32_t)(grp * GRP * kStage);
#pragma unroll
        for (int i = 0; i < 2 * GRP; ++i)               // (an entry that names no block of the pool is the caller's
            ent[i] = min((uint32_t)table[min((t0 + 16 * i) >> a.log2_block_size, last_entry)], last_block);   // mistake: it reads the last block instead of memory outside the pools)
    };
    // This lane's part of a load's address: unit x of a sub-tile as it lies in the pool goes to
    // LDS slot x (tiled layout), or, plain layout (rows of NU units, which cannot be padded on the
    // way in), slot s of row r takes unit s ^ (r mod NU) of a K row and s ^ (2 r mod NU) of a V
    // row, so that the rows an operand read touches fall in different banks.
    uint32_t lane_k[LPT], lane_v[LPT];
#pragma unroll
    for (int k = 0; k < LPT; ++k) {
        const int x = (kThreads * k + 64 * wv) % U + lane;   // the lane's LDS slot within the sub-tile
        const int row = x / NU, sl = x % NU;
        lane_k[k] = (uint32_t)(TILED ? x : row * NU + (sl ^ (row & (NU - 1)))) * 16;
        lane_v[k] = (uint32_t)(TILED ? x : row * NU + (sl ^ ((2 * row) & (NU - 1)))) * 16;
    }
    // The stage's tiles from the pools straight into LDS buffer `buf`, each wave instruction one
    // run of 64 units (1 KiB).  Sub-tiles past the workgroup's last position are not loaded.  Nothing
    // waits here: the caller waits for vmcnt before the barrier that publishes the stage.
    // The address is a scalar base (pool + block + sub-tile, all on the scalar unit, 32 x 32 -> 64
    // bit) plus the lane's constant 32-bit offset: no vector arithmetic per load.
    auto dma = [&](int st, char *buf, uint32_t e0, uint32_t e1) {
#pragma unroll
        for (int k = 0; k < LPT; ++k) {
            const int x0 = kThreads * k + 64 * wv;    // the wave's first unit: sub-tile x0 / U, unit x0 % U
            // (known at compile time where a sub-tile is at least as large as a pass of the workgroup)
            const int sub = U >= kThreads ? (kThreads * k) / U : x0 / U;
            const int t = st * kStage + 16 * sub;
            if (t <= wg_maxpos) {
                const uint64_t off = (uint64_t)(sub ? e1 : e0) * block_stride +
                                     (uint32_t)(((t & (a.block_size - 1)) >> 4) * (16 * D * 2));
                // (written as assembly: the compiler would make every later LDS read wait for these loads;
                // m0, the LDS base of such a load, is a register the compiler reserves and sets itself
                // before any instruction of its own that reads it)
                typedef __attribute__((address_space(3))) char *lptr;
                const uint32_t lk = (uint32_t)(uintptr_t)(lptr)(buf + x0 * 16), lv = lk + VOFF;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lk), "v"(lane_k[k]),
                             "s"(kp + off) : "memory");
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lv), "v"(lane_v[k]),
                             "s"(vp + off) : "memory");
            }
        }
    };
    auto dma_group = [&](int grp, char *buf, const uint32_t (&ent)[2 * GRP]) {
#pragma unroll
        for (int h = 0; h < GRP; ++h) dma(grp * GRP + h, buf + h * STAGE, ent[2 * h], ent[2 * h + 1]);
    };
    const int grp0 = SPLIT ? st0 / GRP : 0;           // (a run begins with a group)
    constexpr int kGroupLoads = GRP * 2 * LPT;        // of one wave
    // The first tiles are asked for in front of the queries, which nothing depends on until the tiles are
    // there, by the kernels that load two stages at a time (24 prompts of 16 to 700 tokens on 40 heads, with
    // the append: 71.3 -> 70.2 us); behind them by the others, which are slower that way: 20 responses
    // of up to 30 tokens, 32 / 8 heads of 128, 69.3 us and 71.1; 4 of 16 on 1 500, 16 / 8 heads of 256, 26.1 and
    // 31.5 (registers).
    constexpr bool kTilesFirst = GRP > 1;            // (written twice: in a lambda it costs the wider kernels registers)
    if constexpr (kTilesFirst) {
        uint32_t first_ent[NB][2 * GRP];
#pragma unroll
        for (int i = 0; i < NB; ++i) lookup(grp0 + i, first_ent[i]);
#pragma unroll
        for (int i = 0; i < NB; ++i) dma_group(grp0 + i, lds + i * GSTAGE, first_ent[i]);
    }

    // this lane's column in each block: (token, head), its position, its q slices
    int pos[kColBlocks];                             // -1: no such column
    size_t orow[kColBlocks];                         // element offset of its output row
    bf16x8 qb[kColBlocks][NK];
#pragma unroll
    for (int b = 0; b < kColBlocks; ++b) {
        const int c = b * 16 + j;
        const int tl = c / G, hd = c - tl * G;
        const int tok = wave_tok + tl;
        const bool ok = c < TW * G && tok < n_new;
        pos[b] = ok ? base_pos + tok : -1;
        orow[b] = ((size_t)(first + (ok ? tok : 0)) * a.num_q_heads + g * G + hd) * D;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            uint4 t = make_uint4(0, 0, 0, 0);
            if (ok) t = *reinterpret_cast<const uint4 *>(static_cast<const char *>(a.q) + (orow[b] + 32 * i + 8 * qd) * 2);
            qb[b][i] = __builtin_bit_cast(bf16x8, t);
        }
    }
    if constexpr (!kTilesFirst) {
        uint32_t first_ent[NB][2 * GRP];
#pragma unroll
        for (int i = 0; i < NB; ++i) lookup(grp0 + i, first_ent[i]);
#pragma unroll
        for (int i = 0; i < NB; ++i) dma_group(grp0 + i, lds + i * GSTAGE, first_ent[i]);
    }

    float m[kColBlocks];
    f32x4 o[kColBlocks][NS];                          // out^T: dims 16 s + 4 qd + e, this lane's column
    f32x4 l[kColBlocks];                              // the column's sum of weights, four copies
#pragma unroll
    for (int b = 0; b < kColBlocks; ++b) {
        m[b] = kLowest;
        l[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) o[b][s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));

    // Value slots at or past the context's end, and those of a sub-tile that was not loaded, are
    // zeroed once the stage is in LDS (they may hold anything, and a zero weight does not silence
    // a NaN; the scores of such positions are masked whatever the keys are).
    const int valid_end = min(C, (wg_maxpos | 15) + 1);
    auto zero_tail = [&](int st, char *buf) {
        int me = tid;
        // Worked out here at head size 256: kept in registers over the loop, what follows made tiles of 64 columns
        // in the tiled layout spill into it, with a wait for every load on its way (4 x 16 new on 1 500, 16 / 8 heads:
        // 26.1 us, 22.7 so).  At smaller head sizes there are registers, and it is 1-2 % slower so.
        if constexpr (D >= 256) asm volatile("" : "+v"(me));
#pragma unroll
        for (int k = 0; k < LPT; ++k) {
            const int x = me + kThreads * k, u = x / U, unit = x % U;
            if (!TILED) {                             // a slot is part of one row: position 16 u + unit / NU
                if (st * kStage + 16 * u + unit / NU >= valid_end)
                    *reinterpret_cast<uint4 *>(buf + VOFF + x * 16) = make_uint4(0, 0, 0, 0);
                continue;
            }
            const int valid = valid_end - (st * kStage + 16 * u + 4 * ((unit >> 4) & 3));
            if (valid < 4) {
                uint4 *slot = reinterpret_cast<uint4 *>(buf + VOFF + x * 16);
                uint4 v = *slot;
                const uint32_t m01 = valid >= 2 ? 0xFFFFFFFFu : (valid == 1 ? 0x0000FFFFu : 0u);
                const uint32_t m23 = valid == 3 ? 0x0000FFFFu : 0u;
                v.x &= m01; v.z &= m01;
                v.y &= m23; v.w &= m23;
                *slot = v;
            }
        }
    };

    // per-lane operand offsets in a stage buffer, tiled layout
    const int koff = qd * 256 + j * 16;               // + i * 1024, + SUBB for the second half
    const int voff = VOFF + (qd * 16 + j) * 16;       // + (s / 2) * 1024 + (s % 2) * 8, + SUBB for the second half
    // plain layout, tiles as they are: the swizzled slots of this lane's operands
    int kslot[NK], vslot[NS];
#pragma unroll
    for (int i = 0; i < NK; ++i) kslot[i] = (j * NU + ((4 * i + qd) ^ (j & (NU - 1)))) * 16;   // row j, dims 32 i + 8 qd ..
#pragma unroll
    for (int s2 = 0; s2 < NS; ++s2) {                 // row 4 qd + j / 4, dims 16 s + 4 (j % 4) ..
        const int rv = 4 * qd + (j >> 2);
        vslot[s2] = VOFF + (rv * NU + ((2 * s2 + ((j & 3) >> 1)) ^ ((2 * rv) & (NU - 1)))) * 16 + (j & 1) * 8;
    }

    bf16x8 kop[NK][2];                                // K rows: position (16 h +) j, dims 32 i + 8 qd ..
    bf16x8 vop[NS];                                   // V^T rows: dim 16 s + j, positions 4 qd .. of both halves
    auto read_k = [&](const char *buf) {
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                kop[i][h] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(
                    buf + (TILED ? koff + i * 1024 : kslot[i]) + h * SUBB));
    };
    auto read_v = [&](const char *buf) {
        if constexpr (TILED) {
            // the two sub-tiles' units as they lie in the pool: dims 32 i + j in bytes 0..7, 32 i + 16 + j in 8..15
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const char *at = buf + voff + (s >> 1) * 1024 + (s & 1) * 8;
                const uint2 h0 = *reinterpret_cast<const uint2 *>(at), h1 = *reinterpret_cast<const uint2 *>(at + SUBB);
                vop[s] = __builtin_bit_cast(bf16x8, make_uint4(h0.x, h0.y, h1.x, h1.y));
            }
        } else {
#pragma unroll
            for (int s = 0; s < NS; ++s) {            // four rows of 16 dims, transposed on the way
                typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
                const s16x4 h0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(buf + vslot[s]));
                const s16x4 h1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(buf + vslot[s] + SUBB));
                vop[s] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
    };

    f32x4 sc0[kColBlocks], sc1[kColBlocks];            // scores: positions t0 (+16) + 4 qd + e of the lane's column
    bf16x8 pw[kColBlocks];                             // weights, transposed: the second product's operand
    // Operand-major order: every K / V operand is used at once for both column blocks
    // (independent MFMAs back to back).
    auto scores = [&]() {
#pragma unroll
        for (int b = 0; b < kColBlocks; ++b) sc0[b] = sc1[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
            for (int b = 0; b < kColBlocks; ++b) {
                sc0[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[i][0], qb[b][i], sc0[b], 0, 0, 0);
                sc1[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[i][1], qb[b][i], sc1[b], 0, 0, 0);
            }
    };
    auto softmax = [&](int t0) {
        const bool masked = t0 + kStage - 1 > wave_minpos;   // wave-uniform: some column does not see the whole stage
#pragma unroll
        for (int b = 0; b < kColBlocks; ++b) {
            float sc[8];                              // raw scores; scale_log2e > 0 is applied in the exponent
#pragma unroll
            for (int e = 0; e < 8; ++e) sc[e] = e < 4 ? sc0[b][e] : sc1[b][e - 4];
            if (masked) {                             // a token sees the positions up to its own
                const int lim = pos[b] - t0 - 4 * qd;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (16 * (e >> 2) + (e & 3) > lim) sc[e] = -INFINITY;
            }
            float mx = sc[0];                         // median with +inf = maximum, without fmaxf's NaN quieting moves
#pragma unroll
            for (int e = 1; e < 8; ++e) mx = __builtin_amdgcn_fmed3f(mx, sc[e], INFINITY);
            mx *= a.scale_log2e;
            // The reference point of the exponentials follows the running maximum lazily:
            // it moves only when a score exceeds it by more than kSlack, so weights stay
            // below 2^kSlack, the four lanes that share a column compare notes only then,
            // and the accumulators are rescaled a handful of times per column.
            if (__any(mx - m[b] > kSlack)) {          // wave-uniform, rare after the first stages
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float mn = mx - m[b] > kSlack ? mx : m[b];
                const float f = fast_exp2(m[b] - mn);
                m[b] = mn;
#pragma unroll
                for (int e = 0; e < 4; ++e) l[b][e] *= f;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[b][s][e] *= f;
            }
            const float mn = m[b];
#pragma unroll
            for (int e = 0; e < 8; ++e) pw[b][e] = (__bf16)fast_exp2(fmaf(sc[e], a.scale_log2e, -mn));
        }
    };
    auto accumulate = [&]() {
#pragma unroll
        for (int b = 0; b < kColBlocks; ++b) l[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pw[b], l[b], 0, 0, 0);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int b = 0; b < kColBlocks; ++b) o[b][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[s], pw[b], o[b][s], 0, 0, 0);
    };

    lookup(grp0 + NB, ent);
    // Waits for group grp with the loads of `ahead` groups behind it on their way.  (Where the last
    // of those loads less than a whole group, or nothing, the count says nothing: all are waited for.)
    auto landed = [&](int grp, auto ahead) {
        if (ahead > 0 && (grp + ahead + 1) * GRP * kStage <= wg_maxpos + 1)
            __builtin_amdgcn_s_waitcnt(vmcnt(ahead * kGroupLoads));
        else
            __builtin_amdgcn_s_waitcnt(vmcnt(0));
        __syncthreads();
    };
    // (two buffers: with group 0 alone waited for here, the two workgroups of a CU fall into a
    // rhythm that is 14 % slower at head_dim 256)
    landed(grp0, std::integral_constant<int, NB == 2 ? 0 : NB - 1>{});
    // At head_dim 256 the K and V operands of a stage are 64 registers each.  With 16 columns per
    // wave they are read one after the other, K right before the scores and V behind them: the
    // wave then stays under 256 registers and two workgroups share a CU here as well.  At 128 it stays
    // under 128 (168 with the tiled layout) that way, for four workgroups (three).
    constexpr bool kLean = (D >= 256 && kCols <= 16) || (kSmall<D, kCols, GRP, SPLIT> && D == 128);
    if (!kLean) read_k(lds);
    const int n_groups = (n_stages + GRP - 1) / GRP;
    // Instructions are fetched by 32 bytes.  Where in such a line the loops of narrow tiles of heads of 64 begin (16 bytes behind this,
    // grouped ones 28) is up to 6 % of their time, least at 4: 10 requests' 16 to 64 on 300 to 1 000 cached, 32 / 8 heads, 13.1 us to
    // 14.1; one prompt of 2 000 on 8 plain heads 27.2 to 29.3.
    if constexpr (D == 64 && kCols == 16 && GRP == 1 && !SPLIT) asm volatile(".p2align 5\n\t.fill %0, 4, 0xbf800000" ::"n"(TILED ? 2 : 5));
    for (int grp = grp0; grp < n_groups; ++grp) {
        char *cur = lds + ((grp - grp0) & (NB - 1)) * GSTAGE, *nxt = lds + ((grp - grp0 + 1) & (NB - 1)) * GSTAGE;
        if ((grp + 1) * GRP * kStage > valid_end) {   // the group holds the last stage: uniform
#pragma unroll
            for (int h = 0; h < GRP; ++h)
                if ((grp * GRP + h) * kStage + kStage > valid_end) zero_tail(grp * GRP + h, cur + h * STAGE);
            __syncthreads();
        }
#pragma unroll
        for (int h = 0; h < GRP; ++h) {
            const int st = grp * GRP + h;
            char *at = cur + h * STAGE;
            const bool live = st * kStage <= wave_maxpos;   // wave-uniform: this wave's columns see the stage
            if (live) {
                if (kLean) read_k(at);
                else read_v(at);                      // needed after the next K operands are asked for
                scores();
                if (kLean) read_v(at);
                softmax(st * kStage);
            }
            if (h == GRP - 1) {
                landed(grp + 1, std::integral_constant<int, NB - 2>{});                    // in LDS for everyone; this group's operands are in registers
                dma_group(grp + NB, cur, ent);        // NB == 2: in flight until the next barrier (a third buffer and
                lookup(grp + NB + 1, ent);            // loads two barriers ahead were measured: slower)
            }
            if (!kLean && st + 1 < n_stages) read_k(h == GRP - 1 ? nxt : at + STAGE);   // needed at the top of the next stage
            if (live) accumulate();
        }
    }

    if (SPLIT && n_runs > 1) {
        constexpr int kAll = kWaves * kCols;          // columns of an item
        float *out = a.partials, *stats = out + (size_t)p.slots * kAll * D;
        uint64_t *flags = reinterpret_cast<uint64_t *>(stats + (size_t)p.slots * kAll * 2);
        if (wave_maxpos >= 0) {                       // uniform: the wave has columns
#pragma unroll
            for (int b = 0; b < kColBlocks; ++b) {
                const size_t at = (size_t)item * (kAll / 16) + wv * kColBlocks + b;
#pragma unroll
                for (int s = 0; s < 2 * NS; ++s)
                    put_shared(out + at * 16 * D + s * 128 + 2 * lane, o[b][s >> 1][2 * (s & 1)], o[b][s >> 1][2 * (s & 1) + 1]);
                if (qd == 0) put_shared(stats + (at * 16 + j) * 2, m[b], l[b][0]);
            }
        }
        __builtin_amdgcn_s_waitcnt(vmcnt(0));
        __syncthreads();                              // the workgroup's stores have arrived, and its LDS is free
        int *is_last = reinterpret_cast<int *>(lds);
        if (wv == 0) {
            const bool all = report_run<(kCols <= 16)>(flags + first_item, item_stride, (item - first_item) / item_stride, n_runs, p.tag);
            if (lane == 0) *is_last = all;
        }
        __syncthreads();
        if (!*is_last) return;
        // The runs in order, whichever workgroup this is: bit-reproducible.  The waves share the blocks of 16 columns that
        // the tile has: at head size 128 by halves of their dims, eight runs at a time, if that leaves no wave two units of work (an
        // API response's few tokens fill one or two blocks, and a wave alone on each took two trips of 50 KB and more at the rate one wave
        // gets); otherwise whole and four at a time.  Attention alone, a wave to a block / by halves always / so: 12 requests' 4 to 64 on
        // 300 to 3 000, 32 / 8 heads of 128, 24.4 / 23.8 / 23.2 us; one of 300 on 2 000 43.3 / 35.9 / 35.2; 3 of 17 to 69 on 74 to 1 529 17.8 / 18.3 /
        // 17.3; 2 of 100 on 1 500, 40 heads, 33.4 / 33.3 / 30.6.
        int me = lane;
        if constexpr (D >= 256) asm volatile("" : "+v"(me));   // (worked out here, not kept over the loop: it spills as it is)
        const int j = me & 15, qd = me >> 4;
        const int blocks = (min(WT, n_new - tile * WT) + TW - 1) / TW * kColBlocks;
        const auto add_up = [&](auto parts, auto runs) {   // parts of a block's dims; runs whose loads are in flight together
            constexpr int PARTS = parts, HS = NS / PARTS, N = runs;
#pragma unroll 1
            for (int u = wv; u < PARTS * blocks; u += kWaves) {
                const int block = u / PARTS, half = u % PARTS;
                const size_t at0 = (size_t)first_item * (kAll / 16) + block, step = (size_t)item_stride * (kAll / 16);
                float M = kLowest, L = 0.0f;
                f32x4 A[HS];
#pragma unroll
                for (int s = 0; s < HS; ++s) A[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int k0 = 0; k0 < n_runs; k0 += N) {
                    float2 ml[N], x[N][2 * HS];
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const size_t at = at0 + min(k0 + k, n_runs - 1) * step;
                        if (k > 0 && k0 + k >= n_runs) {  // uniform
                            ml[k] = make_float2(kLowest, 0.0f);
#pragma unroll
                            for (int s = 0; s < 2 * HS; ++s) x[k][s] = make_float2(0.0f, 0.0f);
                            continue;
                        }
                        ml[k] = get_shared(stats + (at * 16 + j) * 2);
#pragma unroll
                        for (int s = 0; s < 2 * HS; ++s) x[k][s] = get_shared(out + at * 16 * D + (half * 2 * HS + s) * 128 + 2 * me);
                    }
                    float Mn = M;
#pragma unroll
                    for (int k = 0; k < N; ++k) Mn = fmaxf(Mn, ml[k].x);
                    const float f0 = fast_exp2(M - Mn);
                    M = Mn;
                    L *= f0;
#pragma unroll
                    for (int s = 0; s < HS; ++s)
#pragma unroll
                        for (int e = 0; e < 4; ++e) A[s][e] *= f0;
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const float f = fast_exp2(ml[k].x - M);
                        L += ml[k].y * f;
#pragma unroll
                        for (int s = 0; s < 2 * HS; ++s) {
                            A[s >> 1][2 * (s & 1)] += x[k][s].x * f;
                            A[s >> 1][2 * (s & 1) + 1] += x[k][s].y * f;
                        }
                    }
                }
                // column j of the block: as above, for the wave whose block it was
                const int c = block % kColBlocks * 16 + j, t = c / G, tok = tile * WT + block / kColBlocks * TW + t;
                const bool mine = c < TW * G && tok < n_new;
                const float inv = L > 0.0f ? 1.0f / L : 0.0f;
                store_column<HS>(static_cast<uint16_t *>(a.out) + ((size_t)(first + (mine ? tok : 0)) * a.num_q_heads + g * G + (mine ? c - t * G : 0)) * D + 16 * half * HS,
                                 qd, mine, inv, A);
            }
        };
        using one = std::integral_constant<int, 1>;
        using two = std::integral_constant<int, 2>;
        using four = std::integral_constant<int, 4>;
        using eight = std::integral_constant<int, 8>;
        if constexpr (D >= 256)
            add_up(two{}, two{});
        else if constexpr (D < 128)
            add_up(one{}, four{});
        else if (2 * blocks <= kWaves)
            add_up(two{}, eight{});
        else
            add_up(one{}, four{});
        return;
    }
#pragma unroll
    for (int b = 0; b < kColBlocks; ++b) {
        const float lt = l[b][0];
        store_column<NS>(static_cast<uint16_t *>(a.out) + orow[b], qd, pos[b] >= 0, lt > 0.0f ? 1.0f / lt : 0.0f, o[b]);
    }
}

#include "prefill_teams.h"

// The split launch if it is the right one for the sizes; *done says whether it was.
template <int D, bool TILED, int kCols>
hipError_t launch_split_prefill(PrefillArgs p, hipStream_t s, bool *done)
{
    *done = false;
    const int G = p.d.num_q_heads / p.d.num_kv_heads, Hkv = p.d.num_kv_heads;
    if (G > kCols || p.d.batch > kSplitRequests) return hipSuccess;
    const int WT = kWaves * (kCols / G);
    const long long tiles = (p.max_new_tokens + WT - 1) / WT;          // of one request, at most
    const long long all = Hkv * min(tiles * p.d.batch, (long long)p.total_tokens / WT + p.d.batch);
    const long long stages = ((long long)p.d.max_blocks * p.d.block_size - 1) / kStage + 1;   // of one request, at most
    p.slots = (int)min((size_t)kSplitSlots, p.d.partial_capacity / split_item_bytes(D, kWaves * kCols)) / 8 * 8;
    // Half the slots must be left to cut into: with more tiles than that the chip is busy anyhow.
    // (Tiles of 128: a quarter.  They come with many new tokens, and what such a launch can gain is less: half
    // a turn of the chip at most.  By a quarter / a half of the slots, 32 / 8 heads of 128: one prompt of 1 000
    // 29.7 / 30.1 us, 2 of 400 on 1 500 50.1 / 50.8; against it 600 on 1 500, 54 / 47.)
    if (all > p.slots / (kCols == 16 ? 2 : 4) || stages < kSplitStages || all * stages > 0x7fffffff) return hipSuccess;
    p.head_slots = p.slots / Hkv;
    // Two stages per barrier for tiles of 128 as on the plain grid, so that a launch that cuts nothing is as
    // fast as there (one stage and four buffers: 900 new, 16 / 1 heads of 128, 30.3 us against 27.3); one
    // stage and four buffers for tiles of 64, which wait for memory.
    hipLaunchKernelGGL((prefill_mfma<D, TILED, kCols, (D <= 128 && kCols > 16 ? 2 : 1), true>), dim3(p.slots), dim3(kThreads), 0, s, p, (int)tiles, 0);
    *done = true;
    return hipGetLastError();
}

template <int D, bool TILED, int kCB>
hipError_t launch_teams(PrefillArgs p, hipStream_t s)
{
    constexpr int kLds = 128 << 10;
    const int WT = 8 * (16 * kCB / (p.d.num_q_heads / p.d.num_kv_heads));
    const long long tiles = (p.max_new_tokens + WT - 1) / WT;
    int full = 0;
    const unsigned grid = place_grid(p, p.d.num_kv_heads, tiles, WT, false, 0, 256, &full);
    if (grid == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((prefill_teams<D, TILED, kCB>), dim3(grid), dim3(512), kLds, s, p, (int)tiles, full);
    return hipGetLastError();
}

template <int D, bool TILED, int kCols = kMaxCols>
hipError_t launch_mfma_prefill(PrefillArgs p, hipStream_t s)
{
    const int G = p.d.num_q_heads / p.d.num_kv_heads;
    // Split launches: tiles of 64 columns leave no wave without work when a request brings a few
    // tokens (append + attention, 32 / 8 heads: 16 new on 3 000 cached 23 us against 26 with tiles of 128; 40 on
    // 1 000, 8 requests, 30 against 35); from 16 such tiles per request on each K / V byte is read 16 times
    // and more, and tiles of 128 are the better ones (512 new on 3 000: 53 us against 77; where the line lies
    // they are not yet: 256 on 3 000 41 and 39, 300 on 2 000 46 and 37).
    bool done = false;
    hipError_t e;
    if (G <= 16 && (kCols == 16 || (long long)p.max_new_tokens * G < 1024))
        e = launch_split_prefill<D, TILED, 16>(p, s, &done);
    else
        e = launch_split_prefill<D, TILED, kCols>(p, s, &done);
    if (e != hipSuccess || done) return e;
    const int WT = kWaves * (kCols / G);
    const long long tiles = (p.max_new_tokens + WT - 1) / WT;
    int full = 0;
    if constexpr (D >= 128) {
        const rules::Launch launch = {p.d.num_kv_heads, G, D, p.d.batch, p.total_tokens, p.max_new_tokens, (long long)p.d.max_blocks * p.d.block_size};
        if (rules::teams(launch)) return launch_teams<D, TILED, D == 128 ? 2 : 1>(p, s);
    }
    const unsigned grid = place_grid(p, p.d.num_kv_heads, tiles, WT, false, 0, 512, &full);
    if (grid == 0) return hipErrorInvalidValue;
    if constexpr (kCols == kMaxCols && D <= 128) {
        const long long row = (long long)p.d.max_blocks * p.d.block_size;
        if (rules::narrow_tiles({p.d.num_kv_heads, G, D, p.d.batch, p.total_tokens, p.max_new_tokens, row}, TILED)) {
            const int WT16 = kWaves * (16 / G);
            const long long tiles16 = (p.max_new_tokens + WT16 - 1) / WT16;
            const unsigned grid16 = place_grid(p, p.d.num_kv_heads, tiles16, WT16, false, 0, 512, &full);
            if (grid16 == 0) return hipErrorInvalidValue;
            hipLaunchKernelGGL((prefill_mfma<D, TILED, 16, 1, false>), dim3(grid16), dim3(kThreads), 0, s, p, (int)tiles16, full);
            return hipGetLastError();
        }
    }
    // Two stages per barrier where they fit and a request has many new tokens (the matrix cores
    // bind: +2-5 %); with one tile per request the kernel is a stream over the cache, and the
    // finer grain is the faster one (+3 %).
    constexpr bool kFits = 2 * 2 * (4 * 16 * D * 2) <= 65536;
    if (kFits && tiles > 1)
        hipLaunchKernelGGL((prefill_mfma<D, TILED, kCols, kFits ? 2 : 1, false>), dim3(grid), dim3(kThreads), 0, s, p, (int)tiles, full);
    else
        hipLaunchKernelGGL((prefill_mfma<D, TILED, kCols, 1, false>), dim3(grid), dim3(kThreads), 0, s, p, (int)tiles, full);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_rows(const PrefillArgs &p, hipStream_t s)
{
    const int G = p.d.num_q_heads / p.d.num_kv_heads;
    const long long items = (long long)p.total_tokens * p.d.num_kv_heads * (G / p.d.heads_per_pass);
    if (items > 0x7fffffffLL * kWaves) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prefill_rows<R>, dim3((unsigned)((items + kWaves - 1) / kWaves)), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

template <int LPT>
hipError_t launch_rows_f32(const PrefillArgs &p, hipStream_t s)
{
    switch (p.d.heads_per_pass) {
    case 1: return launch_rows<ValuReducer<false, LPT, 1, kHalves>>(p, s);
    case 2: return launch_rows<ValuReducer<false, LPT, 2, kHalves>>(p, s);
    case 4: return launch_rows<ValuReducer<false, LPT, 4, 1>>(p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_prefill(const PrefillArgs &p, hipStream_t stream)
{
    const DecodeArgs &a = p.d;
    if (a.batch == 0 || p.total_tokens == 0) return hipSuccess;
    const int G = a.num_q_heads / a.num_kv_heads;
    if (a.heads_per_pass != decode_heads_per_pass(a.bf16, a.head_dim, G) || a.heads_per_pass == 0)
        return hipErrorInvalidValue;
    const int lpt = a.head_dim * (a.bf16 ? 2 : 4) / 16;
    // (the matrix-core kernel keeps the distance between two blocks of a pool in 32 bits)
    const unsigned long long stride = 2ull * a.num_layers * a.num_kv_heads * a.block_size * a.head_dim;
    if (a.bf16 && G <= kMaxCols && !p.force_rows && stride <= 0xffffffffull) {     // matrix cores
        const bool tiled = decode_uses_tiled_layout(a.bf16, G);
        if (a.head_dim == 64) return tiled ? launch_mfma_prefill<64, true>(p, stream) : launch_mfma_prefill<64, false>(p, stream);
        if (a.head_dim == 128) return tiled ? launch_mfma_prefill<128, true>(p, stream) : launch_mfma_prefill<128, false>(p, stream);
        // head_dim 256: 32 columns per wave need more than 256 registers (one workgroup per CU); without
        // head groups 16 columns and two workgroups per CU are faster (measured: +9 %), with groups not
        if (a.head_dim == 256) return tiled ? launch_mfma_prefill<256, true>(p, stream) : launch_mfma_prefill<256, false, 16>(p, stream);
    }
    if (decode_uses_tiled_layout(a.bf16, G)) {
        if (a.heads_per_pass > 16) return hipErrorInvalidValue;
        if (a.head_dim == 64) return launch_rows<MfmaReducer<64>>(p, stream);
        if (a.head_dim == 128) return launch_rows<MfmaReducer<128>>(p, stream);
        if (a.head_dim == 256) return launch_rows<MfmaReducer<256>>(p, stream);
    } else if (a.bf16) {
        if (lpt == 8) return launch_rows<ValuReducer<true, 8, 1, kHalves>>(p, stream);
        if (lpt == 16) return launch_rows<ValuReducer<true, 16, 1, kHalves>>(p, stream);
        if (lpt == 32) return launch_rows<ValuReducer<true, 32, 1, kHalves>>(p, stream);
    } else if (!p.force_rows) {
        if (a.head_dim == 32) return launch_tiles_f32<32>(p, stream);
        if (a.head_dim == 64) return launch_tiles_f32<64>(p, stream);
        if (a.head_dim == 128) return launch_tiles_f32<128>(p, stream);
    } else {
        if (lpt == 8) return launch_rows_f32<8>(p, stream);
        if (lpt == 16) return launch_rows_f32<16>(p, stream);
        if (lpt == 32) return launch_rows_f32<32>(p, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace lamps
