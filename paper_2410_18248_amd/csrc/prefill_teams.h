// Prompt attention by two teams of waves that take turns at the matrix cores: prefill_mfma's contraction for launches with many
// new tokens.  Device code; part of prefill_attn.hip.
#pragma once

// One workgroup = one (request, kv head, tile of 256 columns; 128 at head size 256): eight waves of kCB blocks of 16 (new token,
// head-of-group) columns, one workgroup to a CU, two waves to a SIMD, one of either team.  While one team is in its matrix phase -- the scores of
// stage s and the outputs of stage s - 1, back to back, with the LDS reads of the next operands between them -- the
// other is in its softmax phase -- weights of its stage, the next loads from the pools -- and a barrier ends each phase.  Left to themselves,
// as in prefill_mfma, the two waves of a SIMD fall into step: both want the matrix cores, then both the vector ALUs (which share
// one issue port with them besides), and a wave-stage of 32 x 32 takes 1 100 to 1 300 cycles for 544 of matrix work; here 830.  The stages'
// tiles come by global_load_lds into a ring of 128 KiB, up to six stages ahead, and serve twice the columns.
//
// Bound by the two phases -- matrix pipe busy 0.56 of the launch, LDS 0.66, 0.4 of that conflicts of the tiled layout's 8-byte value reads -- and by
// power: the chip runs this at 2.2 GHz (prefill_mfma, matrix pipe 0.46, at 2.3), and what takes fewer cycles at more energy loses.  With
// 32x32x16 products, 1 600 cycles to a pair of wave-stages in place of 1 665, it ran at 1.95 GHz: 4 prompts of 4 096, 32 / 8 heads of
// 128, 501 us against 482.  Waves whose columns see no more of the positions do no products (ragged prompts -6 %).  Attention
// alone, us, tiles of 128 by prefill_mfma / so: those 550 / 486, one of 8 000 511 / 438, 4 of 1 000 52 / 43, 16 of 500 on 2 000 to 4 000 cached
// 444 / 386; 40 plain heads, 4 of 2 048, 215 / 198; heads of 256, 4 of 512 on 500 to 2 000 (attention of a recompute's chunk) 76 / 68, 8 of 1 000
// to 2 000 237 / 198.
//
// What each phase holds is measured (cycles of a matrix / softmax phase): all operand reads at the start of the softmax phase 780 /
// 1 100, for the wave waits for room in the LDS queue before its first weight; reads among the products, loads there too 770 / 550; loads, with
// their address arithmetic, in the softmax phase 640 / 780, the least together.  Grouped layout: a value operand is two 8-byte reads, half of
// a unit each; 16-byte reads want 8 register swaps (500 cycles) or, with values brought in by 4 bytes such that they lie as operands, three more
// loads a wave (+3 %).
//
// The reference point of the exponentials moves where prefill_mfma's does and to the same value, so that a row has the same bits whichever of the two
// kernels a call's totals choose.  That it has to is found after the fact, by a weight of 2^kSlack and more: the largest by packed maxima of
// three (two instructions to eight weights; by packed maxima of two the phase is 5 % longer).  A move is far from rare where scores are
// peaked, and all eight waves wait for it at the barrier; only the block that asks for it is weighed again, and lanes compare without LDS.  4 prompts
// of 4 096, 32 / 8 heads, us, queries of N(0, 1) / N(0, 16) by prefill_mfma 549 / 579, with the reference looked for in both blocks through LDS
// 483 / 640, so 482 / 551; 4 of 2 048 on 40 plain heads 207 / 216, 200 / 270, 195 / 229.
template <int D, bool TILED, int kCB>
__global__ __launch_bounds__(512, 2) void prefill_teams(const PrefillArgs p, const int tiles, const int full_groups)
{
    constexpr int W = 8, kCols = 16 * kCB;
    constexpr int NK = D / 32, NS = D / 16, U = D * 2, NU = D / 8;
    constexpr int SUBB = 16 * D * 2, VOFF = 2 * SUBB, STAGE = 4 * SUBB;
    constexpr int NB = 131072 / STAGE;
    constexpr int VA = NB - 2, KA = NB == 4 ? NB : NB - 2;
    constexpr int NE = U / 256;                      // sub-tiles a wave loads from: half of the waves a sub-tile, or each a part of both
    static_assert(NB * STAGE == 131072 && (NE == 1 || NE == 2), "head_dim");
    extern __shared__ __align__(16) char lds[];

    const DecodeArgs &a = p.d;
    const int G = a.num_q_heads / a.num_kv_heads, TW = kCols / G, WT = W * TW;
    Place at;
    if (!place<false>(p, a.num_kv_heads, tiles, full_groups, WT, false, at)) return;
    const int r = at.r, g = at.head, tile = at.tile, first = at.first, n_new = at.n_new, C = at.ctx;
    const int base_pos = C - n_new;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = wv >> 2;
    const int j = lane & 15, qd = lane >> 4;
    const int wave_tok = tile * WT + wv * TW;
    const int wave_minpos = __builtin_amdgcn_readfirstlane(wave_tok < n_new ? base_pos + wave_tok : 0x7fffffff);
    const int wg_maxpos = base_pos + min(n_new, (tile + 1) * WT) - 1;
    const int n_stages = wg_maxpos / kStage + 1;
    const int valid_end = min(C, (wg_maxpos | 15) + 1);
    // the wave's own: its columns see no more (one for a wave without columns, too)
    const int wave_stages = __builtin_amdgcn_readfirstlane(wave_tok < n_new ? (base_pos + min(n_new, wave_tok + TW) - 1) / kStage + 1 : 1);

    const table_ptr table = (table_ptr)(uintptr_t)(a.block_table + (size_t)r * a.max_blocks);
    const uint32_t tile_bytes = (uint32_t)a.block_size * D * 2;
    const uint32_t block_stride = (uint32_t)a.num_layers * a.num_kv_heads * tile_bytes;
    const size_t head_off = ((size_t)a.layer * a.num_kv_heads + g) * tile_bytes;
    const uint64_t kp = (uint64_t)a.k_pool + head_off, vp = (uint64_t)a.v_pool + head_off;
    const uint32_t last_entry = (uint32_t)wg_maxpos >> a.log2_block_size;
    const uint32_t last_block = (uint32_t)a.num_blocks - 1;
    struct Entries { uint32_t e[NE]; };
    auto sub_of = [&](int k) { return NE == 1 ? team : k; };
    auto lookup = [&](int st) {
        Entries x;
#pragma unroll
        for (int k = 0; k < NE; ++k)
            x.e[k] = min((uint32_t)table[min((uint32_t)(st * kStage + 16 * sub_of(k)) >> a.log2_block_size, last_entry)], last_block);
        return x;
    };
    typedef __attribute__((address_space(3))) char *lptr;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr)lds + wv * 1024;
    const int x = (NE == 1 ? (wv & 3) : wv) * 64 + lane, row = x / NU, sl = x % NU;
    const uint32_t lane_k = (uint32_t)(TILED ? x : row * NU + (sl ^ row)) * 16;
    const uint32_t lane_v = (uint32_t)(TILED ? x : row * NU + (sl ^ ((2 * row) & 15))) * 16;
    auto load = [&](uint64_t src, uint32_t dst, uint32_t lane_off) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(lane_off), "s"(src) : "memory");
    };
    auto offset = [&](int st, const Entries &e, int k) {
        const int t = min(st, n_stages - 1) * kStage + 16 * sub_of(k);   // (stages past the last: once more the last)
        return (uint64_t)e.e[k] * block_stride + (uint32_t)(((t & (a.block_size - 1)) >> 4) * SUBB);
    };
    auto dma = [&](int sk, const Entries &ek, int sv, const Entries &ev) {
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const uint64_t off = offset(sk, ek, k);
            load(kp + off, lds0 + (sk & (NB - 1)) * STAGE + k * SUBB, lane_k);
            load(vp + (sv == sk ? off : offset(sv, ev, k)), lds0 + (sv & (NB - 1)) * STAGE + k * SUBB + VOFF, lane_v);
        }
    };
    auto dma_k = [&](int st, const Entries &e) {
#pragma unroll
        for (int k = 0; k < NE; ++k) load(kp + offset(st, e, k), lds0 + (st & (NB - 1)) * STAGE + k * SUBB, lane_k);
    };
    Entries eq[3];                                   // of the stages whose values are asked for next, and of those whose keys are
    if constexpr (KA == VA) {
        for (int i = 0; i < 2; ++i) {
            const Entries e = lookup(i);
            dma(i, e, i, e);
        }
    } else {
        eq[0] = lookup(0);
        eq[1] = lookup(1);
        dma_k(0, eq[0]);
        dma_k(1, eq[1]);
        eq[2] = lookup(2);
        dma(2, eq[2], 0, eq[0]);
        eq[0] = eq[1];
        eq[1] = eq[2];
    }

    int pos[kCB];
    size_t orow[kCB];
    bf16x8 qb[kCB][NK];
#pragma unroll
    for (int b = 0; b < kCB; ++b) {
        const int c = b * 16 + j, tl = c / G, hd = c - tl * G, tok = wave_tok + tl;
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
    float m[kCB];
    f32x4 o[kCB][NS];
    f32x4 l[kCB];
    uint4 ones_u = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
    asm("" : "+v"(ones_u.x), "+v"(ones_u.y), "+v"(ones_u.z), "+v"(ones_u.w));
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_u);
#pragma unroll
    for (int b = 0; b < kCB; ++b) {
        m[b] = kLowest;
        l[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) o[b][s] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    const int koff = qd * 256 + j * 16;
    const int voff = VOFF + (qd * 16 + j) * 16;
    int voff1 = voff + 8;                            // (a base of its own: the two halves of a unit are operands of different slabs)
    asm("" : "+v"(voff1));
    int kslot[4], vslot[8];                          // (of units 16 further on: 256 bytes on)
    if constexpr (!TILED) {
#pragma unroll
        for (int i = 0; i < 4; ++i) kslot[i] = (j * NU + ((4 * i + qd) ^ j)) * 16;
#pragma unroll
        for (int s2 = 0; s2 < 8; ++s2) {
            const int rv = 4 * qd + (j >> 2);
            vslot[s2] = VOFF + (rv * NU + ((2 * s2 + ((j & 3) >> 1)) ^ ((2 * rv) & 15))) * 16 + (j & 1) * 8;
        }
    }
    bf16x8 kop[NK][2], vop[NS];
    auto read_k = [&](const char *buf, int i, int h) {
        kop[i][h] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(buf + (TILED ? koff + i * 1024 : kslot[i & 3] + (i >> 2) * 256) + h * SUBB));
    };
    auto read_v = [&](const char *buf, int s) {
        if constexpr (TILED) {
            const char *src = buf + (s & 1 ? voff1 : voff) + (s >> 1) * 1024;
            const uint2 h0 = *reinterpret_cast<const uint2 *>(src), h1 = *reinterpret_cast<const uint2 *>(src + SUBB);
            vop[s] = __builtin_bit_cast(bf16x8, make_uint4(h0.x, h0.y, h1.x, h1.y));
        } else {
            typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
            const s16x4 h0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(buf + vslot[s & 7] + (s >> 3) * 256));
            const s16x4 h1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(buf + vslot[s & 7] + (s >> 3) * 256 + SUBB));
            vop[s] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };
    f32x4 sc0[kCB], sc1[kCB];
    bf16x8 pw[kCB];
    auto qk = [&](int i) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < kCB; ++b) {
            sc0[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[i][0], qb[b][i], i ? sc0[b] : zero, 0, 0, 0);
            sc1[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[i][1], qb[b][i], i ? sc1[b] : zero, 0, 0, 0);
        }
    };
    auto pv = [&](int s) {
#pragma unroll
        for (int b = 0; b < kCB; ++b) o[b][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[s], pw[b], o[b][s], 0, 0, 0);
    };
    auto sums = [&]() {
#pragma unroll
        for (int b = 0; b < kCB; ++b) l[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pw[b], l[b], 0, 0, 0);
    };
    // The weights of block b; whether one of them is 2^kSlack or more (or no finite number).  They are not negative, so their bits compare as they
    // do, and as those of fp16 numbers.
    typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
    auto weigh = [&](int b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pw[b][e] = (__bf16)fast_exp2(fmaf(sc0[b][e], a.scale_log2e, -m[b]));
            pw[b][4 + e] = (__bf16)fast_exp2(fmaf(sc1[b][e], a.scale_log2e, -m[b]));
        }
        uint4 u = __builtin_bit_cast(uint4, pw[b]);
        asm("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w));   // (pairs from here on: carried over the branch one by one, they are converted twice)
        pw[b] = __builtin_bit_cast(bf16x8, u);
        uint32_t most;
        asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(most) : "v"(u.x), "v"(u.y), "v"(u.z));
        asm("v_pk_maximum3_f16 %0, %1, %2, %2" : "=v"(most) : "v"(most), "v"(u.w));
        return most;
    };
    auto over = [](uint32_t most) {
        constexpr unsigned short kBelow = ((127 + (int)kSlack) << 7) - 1;   // the bf16 in front of 2^kSlack
        return __any(__builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, most), u16x2{kBelow, kBelow})) != 0);
    };
    // the larger of a lane's and the one's whose number differs by 16 (32)
    auto max16 = [](float x) {
        const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return fmaxf(__uint_as_float(y[0]), __uint_as_float(y[1]));
    };
    auto max32 = [](float x) {
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return fmaxf(__uint_as_float(y[0]), __uint_as_float(y[1]));
    };
    auto softmax = [&](int t0) {
        if (t0 + kStage - 1 > wave_minpos) {
#pragma unroll
            for (int b = 0; b < kCB; ++b) {
                const int lim = pos[b] - t0 - 4 * qd;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (e > lim) sc0[b][e] = -INFINITY;
                    if (16 + e > lim) sc1[b][e] = -INFINITY;
                }
            }
        }
        uint32_t most[kCB], all = 0;
#pragma unroll
        for (int b = 0; b < kCB; ++b) {
            most[b] = weigh(b);
            if (b == 0) all = most[0];
            else asm("v_pk_maximum3_f16 %0, %1, %2, %2" : "=v"(all) : "v"(all), "v"(most[b]));
        }
        if (over(all)) {
#pragma unroll
            for (int b = 0; b < kCB; ++b) {
                if (kCB > 1 && !over(most[b])) continue;
                float mx = sc0[b][0];                // (as prefill_mfma finds it)
#pragma unroll
                for (int e = 1; e < 8; ++e) mx = __builtin_amdgcn_fmed3f(mx, e < 4 ? sc0[b][e & 3] : sc1[b][e & 3], INFINITY);
                mx = max32(max16(mx));
                // (there a lane looks first, at the product and the difference rounded once, and then at both rounded)
                const bool above = fmaf(mx, a.scale_log2e, -m[b]) > kSlack;
                mx *= a.scale_log2e;
                asm("" : "+v"(mx));
                const float mn = above && mx - m[b] > kSlack ? mx : m[b];
                const float f = fast_exp2(m[b] - mn);
                m[b] = mn;
                l[b] *= f;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[b][s][e] *= f;
                weigh(b);
            }
        }
    };
    auto pin = [&]() { __builtin_amdgcn_sched_barrier(0); };
    auto barrier = [&]() {
        pin();
        asm volatile("s_barrier" ::: "memory");
        pin();
    };
    auto buffer = [&](int st) { return lds + (st & (NB - 1)) * STAGE; };
    // scores of stage st, outputs of stage st - 1; reads the values of st - 1 and the keys of st + 1
    auto matrix = [&](int st) {
        const char *vb = buffer(st - 1), *kb = buffer(st + 1);
        pin();
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            qk(i);
            if constexpr (D <= 128) {
                read_v(vb, 2 * i);
                read_v(vb, 2 * i + 1);
            } else {
                read_v(vb, i);                       // (half of them: registers)
            }
            pin();
        }
        sums();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            pv(s);
            if constexpr (D <= 128) {
                read_k(kb, s >> 1, s & 1);
            } else if (s < NS / 2) {
                read_v(vb, NS / 2 + s);
            } else {
                read_k(kb, s - NS / 2, 0);
                read_k(kb, s - NS / 2, 1);
            }
            pin();
        }
    };
    __builtin_amdgcn_s_waitcnt(vmcnt(0));
    barrier();
    if constexpr (KA == VA) {
#pragma unroll
        for (int i = 2; i < KA; ++i) {
            const Entries e = lookup(i);
            dma(i, e, i, e);
        }
    } else {
        eq[2] = lookup(3);
        dma(3, eq[2], 1, eq[0]);
        eq[0] = eq[1];
        eq[1] = eq[2];
    }
    eq[2] = lookup(KA);
#pragma unroll
    for (int i = 0; i < NS; ++i) read_k(lds, i >> 1, i & 1);
    if (team) {
        // (the first keys are in registers by the end of phase 0: at head size 256 phase 1 asks for others in their place)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier();
    }
#pragma unroll
    for (int i = 0; i < NK; ++i) qk(i);
#pragma unroll
    for (int i = 0; i < NS; ++i) read_k(buffer(1), i >> 1, i & 1);
    int st = 0;
    // Phases: the first team's matrix phase of stage s is 2 s, its softmax phase 2 s + 1, the second's one later.  Keys of stage s are read in
    // the matrix phase of s - 1 (2 s - 2, 2 s - 1) and in registers by the end of the softmax phase behind it (2 s); its values in that
    // of s + 1 (2 s + 2, 2 s + 3).  In the softmax phase of stage s, not before phase 2 s + 1, a wave asks for keys of stage s + KA and
    // values of s + VA; what lay there, of stages s + KA - NB and s + VA - NB, is read by phases 2 (s + KA - NB) and 2 (s + VA - NB) + 3 at the latest.
    auto ask = [&]() {
        if constexpr (KA == VA) {
            dma(st + KA, eq[2], st + KA, eq[2]);
        } else {
            dma(st + KA, eq[2], st + VA, eq[0]);
            eq[0] = eq[1];
            eq[1] = eq[2];
        }
        eq[2] = lookup(st + KA + 1);
    };
    auto softmax_phase = [&]() {
        ask();
        softmax(st * kStage);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the next keys are in registers: their place in LDS may be written to
    };
    // A matrix phase ends with the wave's own part of the keys of st + 2 and the values of st in LDS, where the next phase may read them.
    constexpr int kBehind = (VA - (KA == VA ? 3 : 1)) * 2 * NE;
    __builtin_amdgcn_s_waitcnt(vmcnt(kBehind));
    barrier();
    softmax_phase();
    barrier();
    for (st = 1; st < wave_stages; ++st) {
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0), which it is: said again where the compiler sees it, or it waits so among the products
        __builtin_amdgcn_s_setprio(1);
        matrix(st);
        __builtin_amdgcn_s_waitcnt(vmcnt(kBehind));
        __builtin_amdgcn_s_setprio(0);
        barrier();
        softmax_phase();
        barrier();
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) read_v(buffer(wave_stages - 1), s);
    if (wave_stages * kStage > valid_end) {             // positions at or past the end carry no values
        const int v0 = valid_end - (wave_stages - 1) * kStage - 4 * qd, v1 = v0 - 16;
        const auto mask = [](int n) { return n >= 2 ? 0xFFFFFFFFu : n == 1 ? 0x0000FFFFu : 0u; };
        const uint32_t m0 = mask(v0), m1 = mask(v0 - 2), m2 = mask(v1), m3 = mask(v1 - 2);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            uint4 y = __builtin_bit_cast(uint4, vop[s]);
            y.x &= m0; y.y &= m1; y.z &= m2; y.w &= m3;
            vop[s] = __builtin_bit_cast(bf16x8, y);
        }
    }
    sums();
#pragma unroll
    for (int s = 0; s < NS; ++s) pv(s);
    for (; st < n_stages; ++st) {                    // its loads are for the others
        __builtin_amdgcn_s_waitcnt(vmcnt(kBehind));
        barrier();
        ask();
        barrier();
    }
    __builtin_amdgcn_s_waitcnt(vmcnt(0));            // no load of the wave's is left on its way to LDS
    if (!team) barrier();
#pragma unroll
    for (int b = 0; b < kCB; ++b) {
        const float lt = l[b][0];
        store_column<NS>(static_cast<uint16_t *>(a.out) + orow[b], qd, pos[b] >= 0, lt > 0.0f ? 1.0f / lt : 0.0f, o[b]);
    }
}
