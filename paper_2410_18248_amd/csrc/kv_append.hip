// KV append: the step before attention in every decode iteration.
//
// arXiv 2410.18248, Section 2.2 / 2.2.1: each iteration produces one key and
// one value vector per layer (and kv head) for the token being generated and
// adds them to the request's cache, which is why the cache -- the M bytes per
// token of equations (1)-(3) -- grows with every iteration.  Here the new
// vectors of all running requests are written into the paged pools at cached
// position ctx_lens[r], i.e. slot ctx_lens[r] % block_size of physical block
// block_table[r][ctx_lens[r] / block_size], in the tile layout the decode
// kernels read (plain or tiled, see lamps.h).  Requests outside the running
// batch (Algorithm 1) append nothing.
//
// One workgroup per request (decode; several of a long row) or per token (many tokens at once).  In
// the decode form all threads read the request's context length, meet at a
// barrier, then scatter; with `advance` thread 0 stores length + 1 after the
// barrier, so nobody can read the new value.  A position outside the
// block-table row, or a block id outside the pool, writes nothing.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "requests.h"

namespace lamps {
namespace {

constexpr int kAppendThreads = 256;

// Writes the key and value vectors kn, vn ([H_kv][D]) of one token at cached position t of request r.
// Called by the workgroups of a token, of which this is number `slice` of `slices`; EARLY: k0 and v0 are what this thread
// takes of them first, asked for before anything is known of where they go.  A position outside the block-table row, or a block id
// outside the pool, writes nothing.
template <typename T>
__device__ __forceinline__ uint4 first_unit(const AppendArgs &a, const T *x, int slice)
{
    const int i = (slice * kAppendThreads + threadIdx.x) * (16 / (int)sizeof(T));
    return i < a.num_kv_heads * a.head_dim ? *reinterpret_cast<const uint4 *>(x + i) : make_uint4(0, 0, 0, 0);
}
template <typename T, bool TILED, bool EARLY>
__device__ __forceinline__ bool scatter_token(const AppendArgs &a, int r, int t, const T *kn, const T *vn, uint4 k0, uint4 v0, int slice, int slices)
{
    const int D = a.head_dim, Hkv = a.num_kv_heads, bs = a.block_size;
    const int lb = t >> a.log2_block_size, slot = t & (bs - 1);
    if (t < 0 || lb >= a.max_blocks) return false;
    const int block = a.block_table[(size_t)r * a.max_blocks + lb];
    if (block < 0 || block >= a.num_blocks) return false;
    const size_t tile = (size_t)bs * D;
    T *kt = static_cast<T *>(a.k_pool) + (((size_t)block * a.num_layers + a.layer) * Hkv) * tile;
    T *vt = static_cast<T *>(a.v_pool) + (((size_t)block * a.num_layers + a.layer) * Hkv) * tile;
    // 16 bytes at a time wherever 16 bytes of a vector stay together in the tile: keys in
    // both layouts (8 dims of a key are contiguous), values in the plain layout
    constexpr int V16 = 16 / (int)sizeof(T);
    const int step = slices * kAppendThreads * V16;
    for (int i = (slice * kAppendThreads + threadIdx.x) * V16; i < Hkv * D; i += step) {
        if (!EARLY || i >= step) {
            k0 = *reinterpret_cast<const uint4 *>(kn + i);
            v0 = *reinterpret_cast<const uint4 *>(vn + i);
        }
        const int g = i / D, d = i - g * D;           // d is a multiple of V16, and V16 divides D
        const size_t ko = TILED ? (size_t)(slot >> 4) * 16 * D + (size_t)((d >> 3) * 16 + (slot & 15)) * 8
                                : (size_t)slot * D + d;
        *reinterpret_cast<uint4 *>(kt + g * tile + ko) = k0;
        if constexpr (!TILED) {
            *reinterpret_cast<uint4 *>(vt + g * tile + ko) = v0;
        } else {
            const size_t base = (size_t)(slot >> 4) * 16 * D;
            const int s16 = slot & 15;
            const uint32_t w[4] = {v0.x, v0.y, v0.z, v0.w};
#pragma unroll
            for (int e = 0; e < V16; ++e) {
                const int dd = d + e;
                const size_t vo = base +
                                  (size_t)(((((dd >> 5) * 4 + (s16 >> 2)) * 16 + (dd & 15)) * 2 + ((dd & 31) >> 4)) * 4) +
                                  (s16 & 3);
                vt[g * tile + vo] = (T)(w[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
    return true;
}

// Bound by the round trips in front of the stores: mask, length and the vectors are asked for
// together, then the table entry.  4 layers of append + decode for 16 requests on 40 heads of 128:
// 116.7 us with each asked for when the one before had come, 113.8 then; with a unit per thread in place of two and a half one
// after the other (4 layers of 16 requests, ranges cut: 106.4 -> 104.2; of 16 up to 600 tokens, 87.0 -> 85.3; where a workgroup takes a request level).
template <typename T, bool TILED>
__global__ __launch_bounds__(kAppendThreads) void kv_append(const AppendArgs a)
{
    const int r = blockIdx.x;
    const size_t row = (size_t)r * a.num_kv_heads * a.head_dim;
    const T *kn = static_cast<const T *>(a.k_new) + row, *vn = static_cast<const T *>(a.v_new) + row;
    const int slice = blockIdx.y, slices = a.slices;
    const uint4 k0 = first_unit(a, kn, slice), v0 = first_unit(a, vn, slice);
    const int t = a.ctx_lens[r];
    if (!a.running[r]) return;                        // uniform over the workgroup
    __syncthreads();
    const bool ok = scatter_token<T, TILED, true>(a, r, t, kn, vn, k0, v0, slice, slices);
    if (ok && a.advance && threadIdx.x == 0) a.ctx_lens[r] = t + 1;
}

// Several new tokens per request (a prompt, a recomputed context, an API
// response): token row n of k_new / v_new belongs to the request r with
// q_start[r] <= n < q_start[r + 1] and goes to position
// ctx_lens[r] - (q_start[r + 1] - q_start[r]) + (n - q_start[r]), ctx_lens
// already counting the new tokens.  One workgroup per token.
// EARLY, the vectors asked for before the request is found, is for rows of more than a unit per thread:
// 4 prompts of 200, 40 heads of 128, 5.6 us, 5.9 late; with smaller rows most of the threads only wait
// (4 prompts of 2 000, 8 heads of 64, 8.5 us, 7.9 late; fp32, 8 heads of 128, the largest such row: 5.4 and 5.3).
// The request, the place of its first token and its length come in one round trip (one for the request and one for those: 4 prompts
// of 2 000 as above 8.6 us, 7.8 so; 6 of 17 to 700, fp32, 3.05 and 2.88; 24 of 16 to 700, 40 heads, level).
template <typename T, bool EARLY>
__global__ __launch_bounds__(kAppendThreads) void kv_append_tokens(const AppendArgs a)
{
    const int n = blockIdx.x;
    const size_t row = (size_t)n * a.num_kv_heads * a.head_dim;
    const T *kn = static_cast<const T *>(a.k_new) + row, *vn = static_cast<const T *>(a.v_new) + row;
    const uint4 none = make_uint4(0, 0, 0, 0), k0 = EARLY ? first_unit(a, kn, 0) : none, v0 = EARLY ? first_unit(a, vn, 0) : none;
    const auto [r, first, count, ctx] = new_tokens_at(a.q_start, a.ctx_lens, a.batch, n, [](int q, int) { return q; });
    if (n >= first + count) return;                   // q_start[batch] is less than the grid
    const int t = ctx - count + (n - first);
    scatter_token<T, false, EARLY>(a, r, t, kn, vn, k0, v0, 0, 1);
}

// The same for the tiled layout (bf16), where the 16-byte unit of a value tile is four
// consecutive positions of two dims: one token alone can only write it 16 bits at a time.
// One workgroup per (request, 16-position sub-tile that holds new tokens, kv head): keys are
// copied 16 bytes at a time as above; for values a thread takes four consecutive positions
// and 2 x 2 dims, transposes them in registers and stores two whole units; only the
// positions of a quad that is not entirely new -- at most one at each end of a request's
// range -- fall back to 16-bit stores.
// Workgroup w belongs to the last request r with (q_start[r] >> 4) + 2 r <= w: request r
// touches at most (count >> 4) + 2 sub-tiles, and the keys of consecutive requests are at
// at least that far apart.
// A long prompt is bound by memory (5.6 TB/s read + written), short ones by the round trips to it: the request, the table entry, keys and values, all
// of them asked for before the first is stored.  (Values asked for behind the stores of keys, and a ragged quad's positions one by one behind one
// another's stores: 12 requests of 6 to 58 tokens, 8 heads of 128, 5.3 us, 3.6 so; 64 prompts of 20 to 200 11.0 and 8.5; 4 of 4 096 28.6 and 28.4.
// Keys and values asked for together with the table entry were up to 5 % slower: 4 prompts of 200, 16 / 8 heads of 256, 4.3 us as it is, 4.5 so.
// A few requests are told apart one by one, by scalar loads: 4 prompts of 4 096 28.6, in one trip by lanes 29.5; 12 requests of 6 to 58 0.1 the other way.)
__global__ __launch_bounds__(kAppendThreads) void kv_append_tokens_tiled(const AppendArgs a)
{
    typedef uint16_t T;
    const int w = blockIdx.x;
    const auto sub_start = [](int q, int i) { return (q >> 4) + 2 * i; };
    const int few = a.batch < kFew ? last_of_few(a.q_start, a.batch, w, sub_start) : 0;
    const auto [r, first, count, ctx] = a.batch < kFew ? NewTokens{few, a.q_start[few], a.q_start[few + 1] - a.q_start[few], a.ctx_lens[few]}
                                                       : new_tokens_at(a.q_start, a.ctx_lens, a.batch, w, sub_start);
    const int p0 = ctx - count;                       // position of the request's first new token
    if (count <= 0 || p0 < 0) return;
    const int sub = (p0 >> 4) + (w - ((first >> 4) + 2 * r));     // sub-tile of the request's context
    const int t_lo = max(p0, sub * 16), t_hi = min(p0 + count, sub * 16 + 16);
    if (t_lo >= t_hi) return;
    const int D = a.head_dim, Hkv = a.num_kv_heads, bs = a.block_size;
    const int lb = (sub * 16) >> a.log2_block_size;
    if (lb >= a.max_blocks) return;
    const int block = a.block_table[(size_t)r * a.max_blocks + lb];
    if (block < 0 || block >= a.num_blocks) return;
    const size_t tile = (size_t)bs * D;
    const size_t at = (((size_t)block * a.num_layers + a.layer) * Hkv) * tile + (size_t)(((sub * 16) & (bs - 1)) >> 4) * 16 * D;
    T *kt = static_cast<T *>(a.k_pool) + at;
    T *vt = static_cast<T *>(a.v_pool) + at;
    const T *kn = static_cast<const T *>(a.k_new), *vn = static_cast<const T *>(a.v_new);
    const int row = Hkv * D;                          // elements of one token's keys (or values)

    const int g = blockIdx.y;                         // kv head
    kt += g * tile; vt += g * tile;
    kn += g * D; vn += g * D;

    // Everything is asked for before the first of it is stored.
    const auto src = [&](const T *x, int t) { return x + (size_t)(first + (t - p0)) * row; };
    // keys: (position, 8 dims) -> one 16-byte unit, at most two to a thread (heads are 64, 128 or 256 here); eight positions by eight units to
    // a wave: 128 bytes of a row on one side and of a tile on the other
    const auto unit = [](int i) { return (i >> 3 & 7) | (i >> 7) << 3; };
    const auto slot = [](int i) { return (i & 7) | (i >> 3 & 8); };
    const int i1 = threadIdx.x + kAppendThreads, c0 = unit(threadIdx.x), c1 = unit(i1), s0 = sub * 16 + slot(threadIdx.x), s1 = sub * 16 + slot(i1);
    const bool key0 = c0 < D / 8 && s0 >= t_lo && s0 < t_hi, key1 = c1 < D / 8 && s1 >= t_lo && s1 < t_hi;
    uint4 k0 = make_uint4(0, 0, 0, 0), k1 = k0;
    if (key0) k0 = *reinterpret_cast<const uint4 *>(src(kn, s0) + c0 * 8);
    if (key1) k1 = *reinterpret_cast<const uint4 *>(src(kn, s1) + c1 * 8);
    // values: (quad of positions, 32-dim group, dims 2 j, 2 j + 1 of its first 16 and of its last 16), one to a thread at most
    const int j = threadIdx.x & 7, i32 = (threadIdx.x >> 3) % (D / 32), q = threadIdx.x / (D / 4);
    const int t0 = sub * 16 + 4 * q;                  // the quad's first position
    const int d0 = 32 * i32 + 2 * j;
    const bool some = q < 4 && t0 + 4 > t_lo && t0 < t_hi;
    uint32_t lo2[4], hi2[4];                          // [position]: dims d0, d0 + 1 and d0 + 16, d0 + 17
    if (some) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {                 // (positions that are not new: the nearest that is)
            const T *x = src(vn, min(max(t0 + k, t_lo), t_hi - 1)) + d0;
            lo2[k] = *reinterpret_cast<const uint32_t *>(x);
            hi2[k] = *reinterpret_cast<const uint32_t *>(x + 16);
        }
    }
    if (key0) *reinterpret_cast<uint4 *>(kt + (size_t)(c0 * 16 + (s0 & 15)) * 8) = k0;
    if (key1) *reinterpret_cast<uint4 *>(kt + (size_t)(c1 * 16 + (s1 & 15)) * 8) = k1;
    if (!some) return;
    T *dst = vt + (size_t)((i32 * 4 + q) * 16 + 2 * j) * 8;       // unit of dim d0; dim d0 + 1's follows
    if (t0 >= t_lo && t0 + 4 <= t_hi) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int sh = 16 * e;
            uint4 u;
            u.x = ((lo2[0] >> sh) & 0xFFFFu) | ((lo2[1] >> sh) << 16);
            u.y = ((lo2[2] >> sh) & 0xFFFFu) | ((lo2[3] >> sh) << 16);
            u.z = ((hi2[0] >> sh) & 0xFFFFu) | ((hi2[1] >> sh) << 16);
            u.w = ((hi2[2] >> sh) & 0xFFFFu) | ((hi2[3] >> sh) << 16);
            *reinterpret_cast<uint4 *>(dst + e * 8) = u;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (t0 + k < t_lo || t0 + k >= t_hi) continue;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                dst[e * 8 + k] = (T)(lo2[k] >> (16 * e));
                dst[e * 8 + 4 + k] = (T)(hi2[k] >> (16 * e));
            }
        }
    }
}

}  // namespace

hipError_t launch_kv_append(AppendArgs a, int tiled, hipStream_t stream)
{
    if (a.batch == 0) return hipSuccess;
    // A unit per thread, by as many workgroups as that takes of a request -- except where the call advances the lengths, which the
    // request's other workgroups may have yet to read.
    const int unit = 16 / (a.bf16 ? 2 : 4);
    a.slices = a.advance ? 1 : (a.num_kv_heads * a.head_dim + kAppendThreads * unit - 1) / (kAppendThreads * unit);
    dim3 grid((unsigned)a.batch, (unsigned)a.slices), block(kAppendThreads);
    if (a.bf16) {
        if (tiled)
            hipLaunchKernelGGL((kv_append<uint16_t, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((kv_append<uint16_t, false>), grid, block, 0, stream, a);
    } else {
        hipLaunchKernelGGL((kv_append<float, false>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_kv_append_tokens(const AppendArgs &a, int total_tokens, int tiled, hipStream_t stream)
{
    if (a.batch == 0 || total_tokens == 0) return hipSuccess;
    dim3 grid((unsigned)total_tokens), block(kAppendThreads);
    const bool early = (size_t)a.num_kv_heads * a.head_dim * (a.bf16 ? 2 : 4) > 16 * kAppendThreads;
    if (a.bf16) {
        if (tiled)
            hipLaunchKernelGGL(kv_append_tokens_tiled, dim3((unsigned)((total_tokens >> 4) + 2 * a.batch), (unsigned)a.num_kv_heads),
                               block, 0, stream, a);
        else if (early)
            hipLaunchKernelGGL((kv_append_tokens<uint16_t, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((kv_append_tokens<uint16_t, false>), grid, block, 0, stream, a);
    } else if (early) {
        hipLaunchKernelGGL((kv_append_tokens<float, true>), grid, block, 0, stream, a);
    } else {
        hipLaunchKernelGGL((kv_append_tokens<float, false>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace lamps
