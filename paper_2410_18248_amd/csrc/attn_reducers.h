// Per-wavefront attention reducers shared by the decode and the prefill kernels:
// the online-softmax pass of one wavefront over a token range of one request's
// paged K/V (arXiv 2410.18248, Section 2.2 equation; paging as in Section 7),
// on the vector ALUs (ValuReducer) or on the matrix cores (MfmaReducer: bf16,
// MfmaF32Tile: fp32, many new tokens).
// Device code; include from a .hip file only.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.h"

namespace lamps {
namespace {

constexpr int kWaves = 4;               // wavefronts per workgroup
constexpr int kThreads = 64 * kWaves;
// wave-wide 16-byte loads per half-chunk and pool; a half-chunk (loads * tokens
// per load) must fit in the smallest block (16 tokens)
constexpr int loads_per_chunk(int lpt) { return lpt == 8 ? 2 : 4; }
constexpr int kHalves = 2;              // half-chunks per chunk on the 1-2 head vector-ALU paths
constexpr float kLowest = -3.0e38f;     // finite stand-in for "no score seen yet"
constexpr int kMaxShares = 16384;       // most wave shares the balanced scheme ever uses
constexpr size_t kPartialBudget = (size_t)64 << 20;   // bytes of partial slots it may need
// The context length of request r as the kernels use it: never beyond the block-table row (a
// longer value is the caller's mistake; clamped, it cannot send a lookup past the row).
__device__ __forceinline__ int ctx_len(const DecodeArgs &a, int r)
{
    return min(a.ctx_lens[r], a.max_blocks * a.block_size);
}

constexpr int kShareOwner = 1, kShareSlot1 = 2, kShareEmpty = 4;   // flags in share_info[].w

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// K and V are read exactly once per launch: a non-temporal 16-byte load keeps
// the stream from displacing anything in the caches (measurably faster here).
__device__ __forceinline__ uint4 load_stream16(const char *p)
{
    u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x)
{
    int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true);
    return x + __int_as_float(y);
}

// Inclusive sum (or, for values that are not negative, maximum) over the lanes of a wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_shifted(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int wave_scan(int x)
{
    x += dpp_shifted<0x111, 0xF>(x);                  // row_shr 1, 2, 4, 8: inside each row of 16
    x += dpp_shifted<0x112, 0xF>(x);
    x += dpp_shifted<0x114, 0xF>(x);
    x += dpp_shifted<0x118, 0xF>(x);
    x += dpp_shifted<0x142, 0xA>(x);                  // row_bcast 15: into rows 1 and 3
    x += dpp_shifted<0x143, 0xC>(x);                  // row_bcast 31: into rows 2 and 3
    return x;
}
__device__ __forceinline__ int wave_max_to(int x)
{
    x = max(x, dpp_shifted<0x111, 0xF>(x));
    x = max(x, dpp_shifted<0x112, 0xF>(x));
    x = max(x, dpp_shifted<0x114, 0xF>(x));
    x = max(x, dpp_shifted<0x118, 0xF>(x));
    x = max(x, dpp_shifted<0x142, 0xA>(x));
    return max(x, dpp_shifted<0x143, 0xC>(x));
}

// Sum over the LPT consecutive lanes that hold one token; every lane gets the
// same bits (each step adds the same two numbers on both sides).
template <int LPT>
__device__ __forceinline__ float sum_token_lanes(float x)
{
    x = dpp_add<0xB1>(x);                       // quad_perm [1,0,3,2]
    x = dpp_add<0x4E>(x);                       // quad_perm [2,3,0,1]
    if (LPT >= 8) x = dpp_add<0x141>(x);        // row_half_mirror
    if (LPT >= 16) x = dpp_add<0x140>(x);       // row_mirror
    if (LPT >= 32) x += __shfl_xor(x, 16);
    if (LPT >= 64) x += __shfl_xor(x, 32);
    return x;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp32 -> bf16 bits, round to nearest even.
__device__ __forceinline__ uint16_t to_bf16_rne(float f)
{
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
    return (uint16_t)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}

// Two of them by the conversion instruction (RNE too; a NaN stays one).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

template <bool BF16>
__device__ __forceinline__ void store_out(void *out, size_t i, float o)
{
    if (BF16)
        static_cast<uint16_t *>(out)[i] = to_bf16_rne(o);
    else
        static_cast<float *>(out)[i] = o;
}

// N consecutive dims, d and up, of one head's row.  Rows of partials are 8-byte aligned.
template <int N>
__device__ __forceinline__ void store_partial(float *pp, int D, int d, float M, float L, const float (&A)[N])
{
#pragma unroll
    for (int e = 0; e < N; e += 2) *reinterpret_cast<float2 *>(pp + d + e) = make_float2(A[e], A[e + 1]);
    if (d == 0) *reinterpret_cast<float2 *>(pp + D) = make_float2(M, L);
}
// Element i and up of `out`, divided by L (zeros if that is none).  wide: out is 16-byte aligned (i is a multiple
// of N).
template <bool BF16, int N>
__device__ __forceinline__ void store_out(void *out, size_t i, bool wide, float L, const float (&A)[N])
{
    float o[N];
#pragma unroll
    for (int e = 0; e < N; ++e) o[e] = L > 0.0f ? A[e] / L : 0.0f;
    if (!wide) {
#pragma unroll
        for (int e = 0; e < N; ++e) store_out<BF16>(out, i + e, o[e]);
    } else if constexpr (BF16) {
        uint32_t w[N / 2];
#pragma unroll
        for (int e = 0; e < N; e += 2) w[e / 2] = pack_bf16(o[e], o[e + 1]);
        uint16_t *at = static_cast<uint16_t *>(out) + i;
        if constexpr (N == 2) *reinterpret_cast<uint32_t *>(at) = w[0];
        if constexpr (N == 4) *reinterpret_cast<uint2 *>(at) = make_uint2(w[0], w[1]);
        if constexpr (N == 8) *reinterpret_cast<uint4 *>(at) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
        for (int e = 0; e < N; e += 2) *reinterpret_cast<float2 *>(static_cast<float *>(out) + i + e) = make_float2(o[e], o[e + 1]);
    }
}

// Partial dot product of a lane's 16 bytes of q and K.
template <bool BF16>
__device__ __forceinline__ float dot16(const uint4 &q, const uint4 &k)
{
    if (BF16) {
        float s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.x),
                                                  __builtin_bit_cast(bf16x2, k.x), 0.0f, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.y),
                                            __builtin_bit_cast(bf16x2, k.y), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.z),
                                            __builtin_bit_cast(bf16x2, k.z), s, false);
        s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.w),
                                            __builtin_bit_cast(bf16x2, k.w), s, false);
        return s;
    } else {
        float s = __uint_as_float(q.x) * __uint_as_float(k.x);
        s = fmaf(__uint_as_float(q.y), __uint_as_float(k.y), s);
        s = fmaf(__uint_as_float(q.z), __uint_as_float(k.z), s);
        s = fmaf(__uint_as_float(q.w), __uint_as_float(k.w), s);
        return s;
    }
}

// A lane's 16 bytes of V as floats.
template <bool BF16, int VEC>
__device__ __forceinline__ void unpack(const uint4 &v, float (&f)[VEC])
{
    if constexpr (BF16) {
        f[0] = bf16_lo(v.x); f[1] = bf16_hi(v.x);
        f[2] = bf16_lo(v.y); f[3] = bf16_hi(v.y);
        f[4] = bf16_lo(v.z); f[5] = bf16_hi(v.z);
        f[6] = bf16_lo(v.w); f[7] = bf16_hi(v.w);
    } else {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
        f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
}

// (m, l, acc) <- merge of (m, l, acc) and (mo, lo, acco), both in exp2 domain.
template <int VEC>
__device__ __forceinline__ void merge_state(float &m, float &l, float (&acc)[VEC], float mo,
                                            float lo, const float (&acco)[VEC])
{
    float mn = fmaxf(m, mo);
    float fa = fast_exp2(m - mn), fb = fast_exp2(mo - mn);
    l = l * fa + lo * fb;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = acc[e] * fa + acco[e] * fb;
    m = mn;
}

// ---------------------------------------------------------------- vector-ALU reducer

// Plain pool layout, GH query heads of the group per pass (GH == 1 for bf16).
template <bool BF16, int LPT, int GH, int NH>
struct ValuReducer {
    static constexpr int kLeastPerCu = 4, kMostPerCu = 8;   // workgroups of a decode launch: as many as fit
    static constexpr bool kBF16 = BF16;
    static constexpr int VEC = BF16 ? 8 : 4;          // elements per 16-byte load
    static constexpr int D = LPT * VEC;
    static constexpr int ES = BF16 ? 2 : 4;           // element bytes
    static constexpr int TPW = 64 / LPT;              // tokens per wave-wide load
    static constexpr int kLoads = loads_per_chunk(LPT);
    static constexpr int HT = TPW * kLoads;           // tokens per half-chunk (<= 16 <= block_size)
    static constexpr int NL = NH * kLoads;            // wave-wide loads per chunk and pool
    static constexpr int CT = HT * NH;                // tokens per chunk
    static constexpr int GT = HT;                     // a range may begin at, and be cut by, any half-chunk

    // One wavefront reduces cached positions [t_begin, t_end) of request r (kv
    // head g, query heads h0 .. h0+GH-1), chunk after chunk, then calls
    // sink(h, d, M, L, A) for every head and run of VEC dims: M = running max (log2
    // domain), L = sum of weights, A[] = weighted sums of V[:, d ..].  t_begin is a
    // multiple of GT.  No barrier, no LDS: waves of a workgroup are independent.
    // q is row `qrow` of a.q ([rows][H][D]); the block table row is r (decode: the same).
    template <typename Sink>
    static __device__ __forceinline__ void run(const DecodeArgs &a, int r, size_t qrow, int g, int h0, int,
                                               int t_begin, int t_end, Sink sink)
    {
        const int lane = threadIdx.x & 63;
        const int row = lane / LPT;                // which of the TPW tokens of a load
        const int col = lane % LPT;                // which 16-byte slice of the head vector

        // q slices of the GH heads, kept in registers for the whole range
        uint4 qv[GH];
#pragma unroll
        for (int h = 0; h < GH; ++h)
            qv[h] = *reinterpret_cast<const uint4 *>(
                static_cast<const char *>(a.q) +
                ((qrow * a.num_q_heads + h0 + h) * D + col * VEC) * ES);

        float m[GH], l[GH], acc[GH][VEC];
#pragma unroll
        for (int h = 0; h < GH; ++h) {
            m[h] = kLowest;
            l[h] = 0.0f;
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[h][e] = 0.0f;
        }

        const int n_chunks = (t_end - t_begin + CT - 1) / CT;
        const int32_t *table = a.block_table + (size_t)r * a.max_blocks;
        const size_t tile_bytes = (size_t)a.block_size * D * ES;
        const size_t block_stride = (size_t)a.num_layers * a.num_kv_heads * tile_bytes;
        const size_t head_off = ((size_t)a.layer * a.num_kv_heads + g) * tile_bytes;
        const char *kp = static_cast<const char *>(a.k_pool) + head_off + lane * 16;
        const char *vp = static_cast<const char *>(a.v_pool) + head_off + lane * 16;

        // A chunk is NH half-chunks of HT tokens; a half-chunk never straddles a
        // block (HT <= 16 <= block_size), so it needs one block-table entry.  All
        // NH * kLoads K loads and as many V loads of a chunk are issued before
        // any is consumed (a deeper software pipeline brought nothing here: with
        // up to eight waves per SIMD the other waves' loads fill the gaps).
        int ch = 0;
        int pb[NH], pbn[NH];
#pragma unroll
        for (int f = 0; f < NH; ++f) {
            const int th = t_begin + ch * CT + f * HT;
            pb[f] = (ch < n_chunks && th < t_end) ? table[th >> a.log2_block_size] : -1;
        }
        while (ch < n_chunks) {
            const int t0 = t_begin + ch * CT;
            uint4 kx[NL], vx[NL];
#pragma unroll
            for (int f = 0; f < NH; ++f) {
                // wave-uniform: half-chunks past the context are skipped, and so is a table entry
                // that does not name a block of the pool (the caller's mistake must not become a
                // wild read; the row it belongs to is then meaningless)
                if ((unsigned)pb[f] < (unsigned)a.num_blocks) {
                    const size_t off = (size_t)pb[f] * block_stride +
                                       (size_t)((t0 + f * HT) & (a.block_size - 1)) * D * ES;
                    if (t0 + (f + 1) * HT <= t_end) {
#pragma unroll
                        for (int i = 0; i < kLoads; ++i)
                            kx[f * kLoads + i] = load_stream16(kp + off + i * 1024);
#pragma unroll
                        for (int i = 0; i < kLoads; ++i)
                            vx[f * kLoads + i] = load_stream16(vp + off + i * 1024);
                    } else {                   // the context ends inside: loads wholly past it are skipped too
#pragma unroll
                        for (int i = 0; i < kLoads; ++i) {
                            const bool in = t0 + f * HT + i * TPW < t_end;
                            kx[f * kLoads + i] = in ? load_stream16(kp + off + i * 1024) : make_uint4(0, 0, 0, 0);
                            vx[f * kLoads + i] = in ? load_stream16(vp + off + i * 1024) : make_uint4(0, 0, 0, 0);
                        }
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < kLoads; ++i) {
                        kx[f * kLoads + i] = make_uint4(0, 0, 0, 0);
                        vx[f * kLoads + i] = make_uint4(0, 0, 0, 0);
                    }
                }
            }

            // physical blocks of the next chunk, fetched while the tiles arrive
            const int chn = ch + 1;
#pragma unroll
            for (int f = 0; f < NH; ++f) {
                const int th = t_begin + chn * CT + f * HT;
                pbn[f] = (chn < n_chunks && th < t_end) ? table[th >> a.log2_block_size] : -1;
            }

            float s[GH][NL];
#pragma unroll
            for (int h = 0; h < GH; ++h)
#pragma unroll
                for (int i = 0; i < NL; ++i)
                    s[h][i] = sum_token_lanes<LPT>(dot16<BF16>(qv[h], kx[i])) * a.scale_log2e;

            if (t0 + CT > t_end) {             // ragged tail: slots at or past ctx_len never count
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    if (t0 + i * TPW + row >= t_end) {
#pragma unroll
                        for (int h = 0; h < GH; ++h) s[h][i] = -INFINITY;
                        vx[i] = make_uint4(0, 0, 0, 0);
                    }
                }
            }

#pragma unroll
            for (int h = 0; h < GH; ++h) {
                float mn = m[h];
#pragma unroll
                for (int i = 0; i < NL; ++i) mn = fmaxf(mn, s[h][i]);
                const float sc = fast_exp2(m[h] - mn);
                float ps = 0.0f;
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    s[h][i] = fast_exp2(s[h][i] - mn);   // now the weight p
                    ps += s[h][i];
                }
                l[h] = l[h] * sc + ps;
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[h][e] *= sc;
                m[h] = mn;
            }
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                float vf[VEC];
                unpack<BF16, VEC>(vx[i], vf);
#pragma unroll
                for (int h = 0; h < GH; ++h)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[h][e] = fmaf(s[h][i], vf[e], acc[h][e]);
            }
            ch = chn;
#pragma unroll
            for (int f = 0; f < NH; ++f) pb[f] = pbn[f];
        }

        // rows of a wave -> one state per wave
#pragma unroll
        for (int h = 0; h < GH; ++h) {
#pragma unroll
            for (int stride = LPT; stride < 64; stride *= 2) {
                float mo = __shfl_xor(m[h], stride), lo = __shfl_xor(l[h], stride);
                float ao[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) ao[e] = __shfl_xor(acc[h][e], stride);
                merge_state<VEC>(m[h], l[h], acc[h], mo, lo, ao);
            }
        }

        if (row == 0) {
#pragma unroll
            for (int h = 0; h < GH; ++h) sink(h, col * VEC, m[h], l[h], acc[h]);
        }
    }
};

// ---------------------------------------------------------------- MFMA reducer

// bf16, tiled pool layout, up to 16 query heads of one kv group per pass.
// Per 16-token sub-tile (a chunk): scores^T[token][head] = K . q^T with D/32
// 16x16x32 MFMAs (A = a coalesced K load as it arrives, B = q slices held in
// registers); the result leaves each lane with 4 consecutive tokens of head
// lane%16, which after the softmax step is, converted to bf16, already the B
// operand p^T[token][head] of the 16x16x16 MFMAs that accumulate
// out^T[dim][head] += V^T . p^T (A = a coalesced V load).  So every statistic of
// head j lives in the lanes with lane%16 == j, and the only cross-lane step per
// sub-tile is the max over the four token groups (two shuffles).
template <int DIM>
struct MfmaReducer {
    // Workgroups of a decode launch on a CU.  At head_dim 128 three fit, and two are the better ones: fewer shares, so
    // fewer pieces and shorter merges, for a stream that two keep at the memory's rate, and a plan that two waves of a
    // SIMD issue in front of the first byte, not three (three / two, 32 / 8 heads: 230 requests of 32 to 8 192 tokens 212.6 / 206.7 us;
    // 256 of 16 to 80 20.2 / 16.6; 64 of 50 to 300 17.6 / 14.9; one of 30 000 28.2 / 27.5; of 59 batches tried, 3 are up to 7 % faster with three).
    static constexpr int kLeastPerCu = DIM >= 256 ? 1 : DIM == 128 ? 2 : 4, kMostPerCu = DIM == 128 ? 2 : 8;
    static constexpr bool kBF16 = true;
    static constexpr int D = DIM;
    static constexpr int CT = 16, GT = 16;            // tokens per chunk = one sub-tile
    static constexpr int NK = D / 32;                 // K loads = score MFMAs per sub-tile
    static constexpr int NS = D / 32;                 // V loads per sub-tile (two 16-dim slabs each)

    template <typename Sink>
    static __device__ __forceinline__ void run(const DecodeArgs &a, int r, size_t qrow, int g, int h0, int heads,
                                               int t_begin, int t_end, Sink sink)
    {
        const int lane = threadIdx.x & 63;
        const int j = lane & 15;                   // head (B / result column); dim in slab (V rows)
        const int qd = lane >> 4;                  // token group of 4 (results) / k slice (operands)

        // B operands of the score MFMAs: q[h0 + j][32 i + 8 qd .. + 8]; zero rows pad to 16 heads
        bf16x8 qb[NK];
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            uint4 t = make_uint4(0, 0, 0, 0);
            if (j < heads)
                t = *reinterpret_cast<const uint4 *>(
                    static_cast<const char *>(a.q) +
                    ((qrow * a.num_q_heads + h0 + j) * D + 32 * i + 8 * qd) * 2);
            qb[i] = __builtin_bit_cast(bf16x8, t);
        }

        float m = kLowest, l = 0.0f;               // m is the same in the 4 lanes of a head
        f32x4 o[2 * NS];                           // out^T: dims 16 s + 4 qd + e, head j
#pragma unroll
        for (int s = 0; s < 2 * NS; ++s) o[s] = f32x4{0.f, 0.f, 0.f, 0.f};

        const int n_chunks = (t_end - t_begin + CT - 1) / CT;
        const int32_t *table = a.block_table + (size_t)r * a.max_blocks;
        const size_t tile_bytes = (size_t)a.block_size * D * 2;
        const size_t block_stride = (size_t)a.num_layers * a.num_kv_heads * tile_bytes;
        const size_t head_off = ((size_t)a.layer * a.num_kv_heads + g) * tile_bytes;
        const char *kp = static_cast<const char *>(a.k_pool) + head_off + lane * 16;
        const char *vp = static_cast<const char *>(a.v_pool) + head_off + lane * 16;

        // Software pipeline: the loads of chunk ch + 1 are issued before chunk ch is
        // consumed, and the block-table entries of the two chunks behind it with them,
        // so a wave always has a sub-tile of K and V in flight while it computes.  Nothing on
        // the way is conditional: behind a load that may or may not have been issued the compiler
        // waits for the loads of the next chunk before it touches the present one.  (So it did: 200 requests of 100 to
        // 4 000 tokens, 8 / 2 heads of 64, 28.0 -> 26.8 us; 32 of 100 to 4 000, 16 / 4 heads of 256, 31.3 -> 28.4, with
        // the accumulators in ordinary registers; 19 of 4 096 to 32 768, 32 / 8 of 128, 202.7 -> 199.7.)
        auto entry = [&](int c) -> int { return table[(t_begin + min(c, n_chunks - 1) * CT) >> a.log2_block_size]; };
        auto issue = [&](int c, int block, uint4 (&kx)[NK], uint4 (&vx)[NS]) {
            // sub-tile (t % block_size) / 16 of the block's tile: 16 * D elements each.  A table entry
            // that does not name a block of the pool is the caller's mistake; it must not become a wild
            // read: the pool's last block is read instead, and the row it belongs to is meaningless
            const int t = t_begin + c * CT;
            const size_t off = (size_t)min((unsigned)block, (unsigned)a.num_blocks - 1) * block_stride +
                               (size_t)((t & (a.block_size - 1)) >> 4) * (16 * D * 2);
#pragma unroll
            for (int i = 0; i < NK; ++i) kx[i] = load_stream16(kp + off + i * 1024);
#pragma unroll
            for (int i = 0; i < NS; ++i) vx[i] = load_stream16(vp + off + i * 1024);
        };
        auto consume = [&](int t0, uint4 (&kx)[NK], uint4 (&vx)[NS], auto last) {
            __builtin_amdgcn_sched_barrier(0);     // (the loads above stay above what waits for the ones before them)
            f32x4 s = {0.f, 0.f, 0.f, 0.f};        // tokens t0 + 4 qd + e, head j
#pragma unroll
            for (int i = 0; i < NK; ++i)
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kx[i]), qb[i],
                                                            s, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] *= a.scale_log2e;

            if (last && t0 + CT > t_end) {         // ragged tail: slots at or past ctx_len never count
                const int valid = min(4, max(0, t_end - (t0 + 4 * qd)));   // of this lane's 4 tokens
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e >= valid) s[e] = -INFINITY;
                // a V load holds tokens 4 qd + {0,1} in .x/.z and + {2,3} in .y/.w (16 bits each)
                const uint32_t m01 = valid >= 2 ? 0xFFFFFFFFu : (valid == 1 ? 0x0000FFFFu : 0u);
                const uint32_t m23 = valid >= 4 ? 0xFFFFFFFFu : (valid == 3 ? 0x0000FFFFu : 0u);
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    vx[i].x &= m01; vx[i].z &= m01;
                    vx[i].y &= m23; vx[i].w &= m23;
                }
            }

            float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mn = fmaxf(m, mx);
            const float sc = fast_exp2(m - mn);
            m = mn;
            float p[4], ps = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[e] = fast_exp2(s[e] - mn);
                ps += p[e];
            }
            l = l * sc + ps;
            // p as a bf16 pair: high part and (exactly computed) remainder
            union { s16x4 v; uint16_t u[4]; } ph, pl;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ph.u[e] = to_bf16_rne(p[e]);
                pl.u[e] = to_bf16_rne(p[e] - __uint_as_float((uint32_t)ph.u[e] << 16));
            }
#pragma unroll
            for (int sidx = 0; sidx < 2 * NS; ++sidx) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[sidx][e] *= sc;
            }
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                union { uint2 u; s16x4 v; } a0, a1;    // V^T rows: dim 32 i + j, and 32 i + 16 + j
                a0.u = make_uint2(vx[i].x, vx[i].y);
                a1.u = make_uint2(vx[i].z, vx[i].w);
                o[2 * i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0.v, ph.v, o[2 * i], 0, 0, 0);
                o[2 * i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0.v, pl.v, o[2 * i], 0, 0, 0);
                o[2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1.v, ph.v, o[2 * i + 1], 0, 0, 0);
                o[2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1.v, pl.v, o[2 * i + 1], 0, 0, 0);
            }
        };
        if (n_chunks > 0) {
            uint4 ka[NK], va[NS], kb[NK], vb[NS];
            int ch = 0, e1, e2;
            if ((n_chunks & 1) == 0) {             // the last chunk is to be one that `ka` holds
                const int e0 = entry(0);
                e1 = entry(1);
                issue(0, e0, kb, vb);
                issue(1, e1, ka, va);
                e1 = entry(2);
                e2 = entry(3);
                consume(t_begin, kb, vb, std::false_type{});
                ch = 1;
            } else {
                issue(0, entry(0), ka, va);
                e1 = entry(1);
                e2 = entry(2);
            }
            for (; ch + 1 < n_chunks; ch += 2) {
                issue(ch + 1, e1, kb, vb);
                e1 = entry(ch + 3);
                consume(t_begin + ch * CT, ka, va, std::false_type{});
                issue(ch + 2, e2, ka, va);
                e2 = entry(ch + 4);
                consume(t_begin + (ch + 1) * CT, kb, vb, std::false_type{});
            }
            consume(t_begin + ch * CT, ka, va, std::true_type{});
        }

        // the weight sum was kept per token group: add the four groups of a head
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);

        if (j < heads) {
#pragma unroll
            for (int sidx = 0; sidx < 2 * NS; ++sidx) {
                const float A[4] = {o[sidx][0], o[sidx][1], o[sidx][2], o[sidx][3]};
                sink(j, 16 * sidx + 4 * qd, m, l, A);
            }
        }
    }
};

// ---------------------------------------------------------------- MFMA tile reducer, 32 bits

// fp32, plain pool layout, up to 16 columns -- (query row, limit) pairs -- of one kv head, on the fp32
// matrix instruction (16x16x4: full fp32 products and sums).  Both operands come out of memory as
// they are, 16 bytes per lane.  Scores^T[token][column] = K . q^T: the contraction index may be
// permuted, so a lane's 16 bytes of row lane % 16 feed four MFMAs.  The result leaves a lane with
// four consecutive tokens of its column; its register e is, unchanged, the operand p^T[token][column]
// of the MFMAs that take tokens 4 (lane / 16) + e, and the V operand of those is what the lane gets
// from 16 bytes (8 at head_dim 32) of that token's row: four dims, one for each of four MFMAs.
// (Decode with grouped heads keeps the vector ALUs: there, 24 requests of 17 to 2 500 tokens, 32 / 8
// heads of 128, this reducer took 34 us against 27, two waves per SIMD against four.)
template <int DIM>
struct MfmaF32Tile {
    static constexpr int D = DIM;
    static constexpr int CT = 16;                     // tokens per chunk
    static constexpr int NK = D / 16;                 // K loads per chunk, four score MFMAs each
    static constexpr int VW = D >= 64 ? 4 : 2;        // dims of one V load
    static constexpr int NC = D / (16 * VW);          // V loads per token group
    typedef __attribute__((ext_vector_type(VW))) float vvec;

    struct State {                                    // of column lane % 16: the same m and l in its four lanes
        float m, l;
        f32x4 o[NC][VW];                              // [c][v][e]: dim 16 VW c + VW (4 (lane / 16) + e) + v
    };

    // Reduces cached positions [t_begin, t_end) of request r, kv head g, taking every `stride`-th
    // chunk of 16 (two at least: then only a wave's last chunk can hold positions that some column does not
    // see, limits being at most 15 apart); t_begin is a multiple of 16.  q: the lane's column's row (nullptr: no column), of
    // which positions at or past `limit` do not count; every column sees the positions before min_limit.
    static __device__ __forceinline__ void reduce(const DecodeArgs &a, int r, int g, const float *q, int limit, int min_limit,
                                                  int t_begin, int t_end, int stride, State &st)
    {
        const int lane = threadIdx.x & 63, j = lane & 15, qd = lane >> 4;
        f32x4 qb[NK];
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            qb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (q) qb[i] = *reinterpret_cast<const f32x4 *>(q + 16 * i + 4 * qd);
        }
        float m = kLowest, l = 0.0f;                  // l: of this lane's tokens, until the end
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < VW; ++v) st.o[c][v] = f32x4{0.f, 0.f, 0.f, 0.f};

        const int n_chunks = (t_end - t_begin + CT * stride - 1) / (CT * stride);
        const int32_t *table = a.block_table + (size_t)r * a.max_blocks;
        const size_t tile = (size_t)a.block_size * D, block_stride = (size_t)a.num_layers * a.num_kv_heads * tile;
        const size_t head_off = ((size_t)a.layer * a.num_kv_heads + g) * tile;
        const float *kp = static_cast<const float *>(a.k_pool) + head_off + j * D + 4 * qd;
        const float *vp = static_cast<const float *>(a.v_pool) + head_off + 4 * qd * D + VW * j;

        // As in MfmaReducer: chunk c + 1 is asked for before chunk c is consumed, the table entries of the
        // two behind it with it, and nothing on the way is conditional.  (With conditional loads each chunk
        // waited for the loads of the next: one prompt of 1 000 tokens, 8 heads of 64, append included, 28.2 -> 24.6 us;
        // 4 x 8 to 32 new on 1 000 to 3 000 cached 41.4 -> 30.7; 3 of 600 on 32 / 8 heads of 128 152.6 -> 125, in the order of now.)
        auto entry = [&](int c) -> int { return table[(t_begin + min(c, n_chunks - 1) * CT * stride) >> a.log2_block_size]; };
        auto issue = [&](int c, int block, f32x4 (&kx)[NK], vvec (&vx)[4][NC]) {
            const int t = t_begin + c * CT * stride;
            // (an entry that names no block of the pool is the caller's mistake: it reads the last block)
            const size_t off = (size_t)min((unsigned)block, (unsigned)a.num_blocks - 1) * block_stride +
                               (size_t)(t & (a.block_size - 1)) * D;
#pragma unroll
            for (int i = 0; i < NK; ++i) kx[i] = *reinterpret_cast<const f32x4 *>(kp + off + 16 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c2 = 0; c2 < NC; ++c2) vx[e][c2] = *reinterpret_cast<const vvec *>(vp + off + e * D + 16 * VW * c2);
        };
        auto consume = [&](int t0, f32x4 (&kx)[NK], vvec (&vx)[4][NC], auto last) {
            __builtin_amdgcn_sched_barrier(0);        // (the loads above stay above what waits for the ones before them)
            // tokens t0 + 4 qd + e of the lane's column; eight chains: no MFMA waits for the one before
            // it, and the sums are short (their error stays that of the vector ALUs' pairwise ones)
            f32x4 p8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p8[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < NK; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    f32x4 &x = p8[4 * (i & 1) + e];
                    x = __builtin_amdgcn_mfma_f32_16x16x4f32(kx[i][e], qb[i][e], x, 0, 0, 0);
                }
            float s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s[e] = (((p8[0][e] + p8[1][e]) + (p8[2][e] + p8[3][e])) + ((p8[4][e] + p8[5][e]) + (p8[6][e] + p8[7][e]))) * a.scale_log2e;
            bool wild = false;                        // uniform: a value that not every column sees is no finite number
            if (last && (t0 + CT > min_limit || t0 + CT > t_end)) {   // uniform: some column does not see the whole chunk
                const int seen = min(limit, t_end) - (t0 + 4 * qd);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e >= seen) s[e] = -INFINITY;
                if (t0 + CT > t_end)                  // a zero weight does not silence a NaN: slots past the end are zeroed
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t0 + 4 * qd + e >= t_end)
#pragma unroll
                            for (int c2 = 0; c2 < NC; ++c2) vx[e][c2] = vvec{};
                if (min_limit < t_end) {
                    float z = 0.0f;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int c2 = 0; c2 < NC; ++c2)
#pragma unroll
                            for (int v = 0; v < VW; ++v) z = fmaf(vx[e][c2][v], 0.0f, z);
                    wild = __any(z != 0.0f);          // (NaN)
                }
            }
            float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mn = fmaxf(m, mx);
            const float sc = fast_exp2(m - mn);
            m = mn;
            float ps = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s[e] = fast_exp2(s[e] - mn);
                ps += s[e];
            }
            l = l * sc + ps;
            // The chunk's sums start at zero, in two chains of eight tokens, and join the outputs in the multiply-add that
            // rescales those.  Against a wave per token the error (to 64 bits) is 0.81 of it over 26 batches of 1 to 31 requests,
            // 0.84 with one chain of sixteen: between 0.4 and 1 from 100 tokens up, where short chunks spare the sum its length,
            // and on prompts of 10 to 80 tokens 1.01 to 1.04 (of 10 to 13, heads of 128: 1.08) where one chain gave 1.05 to 1.10.
            // The second chain costs 1 to 2.5 % of the time; four of four tokens each would give 0.80 and cost 3 to 5 %, and
            // at head_dim 128 they no longer fit 256 registers.
            if (!wild) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        f32x4 t[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            t[e >> 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vx[e][c][v], s[e], t[e >> 1], 0, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) st.o[c][v][e] = fmaf(st.o[c][v][e], sc, t[0][e] + t[1][e]);
                    }
            } else {                                  // once per limit, the values past it zeroed, kept by its columns
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        f32x4 kept = {0.f, 0.f, 0.f, 0.f};
                        for (int lim = min_limit; lim <= t_end; ++lim) {
                            f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                t = __builtin_amdgcn_mfma_f32_16x16x4f32(t0 + 4 * qd + e < lim ? vx[e][c][v] : 0.0f, s[e], t, 0, 0, 0);
                            if (limit == lim) kept = t;
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) st.o[c][v][e] = fmaf(st.o[c][v][e], sc, kept[e]);
                    }
            }
        };
        if (n_chunks > 0) {
            f32x4 ka[NK], kb[NK];
            vvec va[4][NC], vb[4][NC];
            const int step = CT * stride;
            const bool even = (n_chunks & 1) == 0;
            int ch = 0, e1, e2;
            if (even) {                               // the last chunk is to be one that `ka` holds
                const int e0 = entry(0);
                e1 = entry(1);
                issue(0, e0, kb, vb);
                issue(1, e1, ka, va);
                e1 = entry(2);
                e2 = entry(3);
                consume(t_begin, kb, vb, std::false_type{});
                ch = 1;
            } else {
                issue(0, entry(0), ka, va);
                e1 = entry(1);
                e2 = entry(2);
            }
            for (; ch + 1 < n_chunks; ch += 2) {
                issue(ch + 1, e1, kb, vb);
                e1 = entry(ch + 3);
                consume(t_begin + ch * step, ka, va, std::false_type{});
                issue(ch + 2, e2, ka, va);
                e2 = entry(ch + 4);
                consume(t_begin + (ch + 1) * step, kb, vb, std::false_type{});
            }
            consume(t_begin + ch * step, ka, va, std::true_type{});
        }
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        st.m = m;
        st.l = l;
    }
};

}  // namespace
}  // namespace lamps
