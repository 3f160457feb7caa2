// Whole backward of one (batch, head) in one workgroup and one pass over memory, for sequences of at most
// 32 * NW tokens with 64 channels (spatial attention over a frame's 14 x 14 tokens, captions).
//
// At these lengths the backward is bound by memory: 8 tensors of N x 64 for 10 N^2 64 operations.  The two
// kernels of avion_bwd.h read Q, K, V, O, dO and Q, K, V, dO and form S and dP twice; here Q, K and dO come
// into LDS once, V and O into registers, S and dP are formed once, and dQ, dK and dV leave together.
//
// Wavefront w owns keys 32w..32w+31: K, V as B operands, dK^T and dV^T as accumulators, exactly the unit of
// avion_dkdv_body.  The workgroup walks the NB query blocks j of 32 together.  Each wavefront leaves its
// 32 x 32 block of dS (rounded to the element format, as the second contraction takes it) in LDS, one row
// per key; after one barrier the NW wavefronts form dQ^T of block j, [64 channels x 32 queries], in
// 16 x 16 tiles over all keys (16x16x32 products): their K^T fragments stay in registers, dS^T is read
// through transposing loads.  Two dS buffers, so that one barrier per block is enough: dQ of block j is formed behind it,
// in the same stretch of code as the scores of block j + 1, so that neither chain of products waits alone.  NB is a
// template parameter: no branch breaks that stretch, and no key block beyond the last is read.  No atomics, no
// partial sums in memory.  avion_dq_body's TILE16 form takes the same operands in the same order, so the
// backward's two phases give this kernel's bits.
//
// 8 wavefronts (129..256 tokens): 134 KB of LDS, one workgroup per compute unit, so nothing else covers its
// loads.  It walks the heads: K's tile is free once the operands are in registers, 64 rows of Q and dO once
// their two blocks are done, and the next head's rows are fetched into them right then, without registers
// (LDS-direct loads); O, V and LSE follow in registers.
// 4 wavefronts (33..128 tokens): one head each, the workgroups of a compute unit overlap each other, so what counts is how
// many fit: LDS of NB blocks, dS in K's place (K is in registers by then), and up to 96 tokens 168 registers, which costs
// dQ beside the scores and the early request of the transposed operands and buys a third workgroup.
// Measured, whole backward, us: dQ right behind its barrier, with the LDS of 4 or 8 blocks and two workgroups of 4
// wavefronts per compute unit -> this form: 3072 heads x 196 187 -> 171 (616 MB: 3.6 TB/s), x 160 139 -> 127, x 130
// 125 -> 113, x 256 234 -> 221, 8000 x 200 causal 434 -> 424; 16384 x 77 causal 295 -> 268 (4.8 TB/s), without mask 303 -> 273,
// x 64 244 -> 216, x 40 205 -> 157, 4000 x 128 117 -> 114; few heads: 8 x 200 15.0 -> 14.1, 384 x 200 32.8 -> 30.5, 768 x 77
// causal 18.4 -> 15.5, 513 x 64 14.9 -> 11.1, 513 x 33 12.7 -> 8.5, 8 x 77 8.3 -> 8.1.  At 16384 x 77 causal, three
// workgroups with dQ beside the scores (spills) 352, two 284.
// Tiles in rows of 144 bytes and descriptors made per request -> quad_at's layout (a block's offset is an addition, a fragment's
// address a register and the instruction's offset) and descriptors once per head: 3072 x 196 180 -> 166 (3.7 TB/s), x 160
// 130 -> 121, x 130 114 -> 104, x 224 196 -> 184, x 256 225 -> 218, 8000 x 200 causal 416 -> 394, 16384 x 77 causal 267 -> 261,
// x 64 221 -> 216, x 40 153 -> 146; 8 x 200 14.0 -> 12.6, 384 x 200 29.0 -> 27.7, 768 x 128 causal 26.0 -> 25.0, the smallest equal.
// Where every workgroup has one head and nearly every compute unit a workgroup, a launch is one burst of requests, which this layout makes
// in half lines: 200 to 256 heads 0.92 to 1.005 of the time without mask, but 0.94 to 1.023 with one (256 x 180 14.45 -> 14.74).
// Against two kernels of avion_bwd.h of one group each it was 0.60 to 0.99 of their time at 1 to 768 heads x 129..256 before
// that; two kernels of two groups each (64-row blocks, two groups) were faster by 0 to 4 % at 196..224
// tokens and 8 to 14 % at 240..256 below 96 heads.
// dQ in 32 x 32 tiles after every fourth block (fewer barriers, longer chains): 226 at 3072 x 196.
#pragma once
#include "avion_common.h"

template <int NW, int NB>
struct HeadCfg {
    static constexpr int D = 64, NT = NW * 64, MAX_N = 32 * NW;
    static constexpr int DS_STRIDE = 72;                 // 32 queries of 2 bytes, padded so that 32 rows hit distinct banks
    // one workgroup per compute unit: it walks several heads
    static constexpr bool WALK = NW == 8;
    static constexpr int ROWS = WALK ? MAX_N : 32 * NB;
    static constexpr int TILE_BYTES = ROWS * 128;        // Q, dO, K: all rows of the head (quad_at)
    static constexpr int DS_BYTES = ROWS * DS_STRIDE;    // one key per row
    // dS lies where K was (and beyond it: two buffers of 72 bytes a row), unless the next head's K is on its way there
    static constexpr int OFF_G = TILE_BYTES, OFF_K = 2 * TILE_BYTES, OFF_DS = WALK ? 3 * TILE_BYTES : OFF_K, OFF_SC = OFF_DS + 2 * DS_BYTES;
    static_assert(2 * DS_BYTES >= TILE_BYTES, "the scalars lie behind K");
    static constexpr int LDS_BYTES = OFF_SC + 2 * MAX_N * 4;  // LSE*log2e and -delta per query
    static constexpr int WAVES_PER_SIMD = WALK || NB > 3 ? 2 : 3;
    // transposed operands requested ahead of the vector work; with 168 registers (three wavefronts per SIMD) behind it.  Behind it
    // at four blocks: 8 x 128 9.10 us instead of 8.95, causal 9.77 (9.67), 513 x 128 21.9 (21.6), 513 x 97 causal 21.64 (21.39).
    static constexpr bool EARLY_TR = WAVES_PER_SIMD == 2;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
    static_assert(!WALK || ROWS % 64 == 0, "walking workgroups fetch 64 rows at a time");
    static_assert(NB * RowStore<D, Bf16>::BYTES <= 2 * DS_BYTES, "the epilogue stages its rows in the dS buffers");
};

// barrier that orders LDS accesses only: loads and stores to memory stay in flight
DEVINL void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int NW, int NB, typename E, bool CAUSAL>
__global__ void __launch_bounds__(NW * 64, (HeadCfg<NW, NB>::WAVES_PER_SIMD))
avion_bwd_head_kernel(const raw16* __restrict__ q, const raw16* __restrict__ k, const raw16* __restrict__ v,
                      const raw16* __restrict__ o, const raw16* __restrict__ dO, const float* __restrict__ lse,
                      raw16* __restrict__ dq, raw16* __restrict__ dk, raw16* __restrict__ dv, int H, int N, int rs_qkv, int rs_o,
                      int nheads, float cs, float scale)
{
    using Cfg = HeadCfg<NW, NB>;
    constexpr int D = 64, KS = 4, CT = 2, QT = 8 / NW;  // QT: 16-query tiles of dQ per wavefront
    // Masked instances of 6 to 8 blocks need up to 44 bytes of scratch with the early request: 8000 heads x 200 435 us instead of
    // 394, 1024 x 256 70.1 instead of 61.4.  The other walking instances do not: behind it, 3072 x 196 174 instead of 166.
    constexpr bool EARLY_TR = Cfg::EARLY_TR && !(CAUSAL && Cfg::WALK && NB >= 6);
    // Eight blocks without mask: dQ of the block before is written in two halves, one to each half of the vector work.  In one piece its eight
    // products are compiled to a chain of their own, each behind a wait for its operands (208 heads x 228 18.8 us instead of 18.05, 16 x 240 14.97
    // instead of 14.18, 3072 x 240 214 instead of 207).  With fewer blocks the compiler spreads them by itself (in halves 180 tokens 1 to 3 %
    // slower), with a mask each is behind a branch (equal or slower).
    constexpr bool SPLIT_DQ = Cfg::WALK && NB == 8 && !CAUSAL;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid % 64, l32 = lane % 32, g = lane / 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const long rs = rs_qkv;
    const int k0 = wave * 32;  // first key, and for the per-query scalars first query, of this wavefront
    const int nslots = (N + 63) / 64;
    const bool wave_active = k0 < N;
    char* ds = smem + Cfg::OFF_DS;
    float* sc = reinterpret_cast<float*>(smem + Cfg::OFF_SC);
    const unsigned lds0 = lds_address(smem);
    const int row_in = min(k0 + l32, N - 1);
    const QuadLane ln(lane, lds0);
    const int c0 = 16 * (wave % 4), q16 = NW == 8 ? 16 * (wave / 4) : 0;  // this wavefront's dQ tile(s)

    auto head_off = [&](int bh) { return (long)(bh / H) * N * rs + (long)(bh % H) * D; };
    auto head_off_o = [&](int bh) { return (long)(bh / H) * N * rs_o + (long)(bh % H) * D; };
    // Wavefront w fetches 1 KB blocks w, w + NW, ... of a tensor; rows past the end arrive as zeros.  The descriptors are made once per
    // head and a block's offset is an addition: with 9-chunk rows (a division per block) and descriptors per call the requests
    // took 13 % of a wavefront's time at 196 tokens.
    struct Fetch {
        u32x4 q, g, k;
    };
    const unsigned voff = quad_voff(wave, lane, (unsigned)(rs * 2)), voff_o = quad_voff(wave, lane, (unsigned)(rs_o * 2));
    auto fetch_of = [&](int bh) {
        const long off = head_off(bh), off_o = head_off_o(bh);
        return Fetch{RawBuffer(q + off, slice_bytes(rs, N, D)).words, RawBuffer(dO + off_o, slice_bytes(rs_o, N, D)).words,
                     RawBuffer(k + off, slice_bytes(rs, N, D)).words};
    };
    const unsigned row_step = 8 * NW * (unsigned)(rs * 2), row_step_o = 8 * NW * (unsigned)(rs_o * 2);  // from block w to w + NW
    constexpr int TURNS = Cfg::ROWS / (8 * NW);
    const int turns = Cfg::WALK ? nslots : TURNS;
    const unsigned lds_w = lds0 + wave * 1024;
    auto fetch_k = [&](const Fetch& f) {
        for (int i = 0; i < turns; ++i) load_to_lds16(RawBuffer(f.k), lds_w + Cfg::OFF_K + i * NW * 1024, voff + i * row_step);
    };
    // the i-th blocks of Q and of dO (walking workgroups: 64 rows)
    auto fetch_rows = [&](const Fetch& f, int i) {
        load_to_lds16_x2<Cfg::OFF_G>(RawBuffer(f.q), RawBuffer(f.g), lds_w + i * NW * 1024, voff + i * row_step, voff_o + i * row_step_o);
    };
    frag8 vf[KS], of[KS];
    float lse_in;
    auto load_v = [&](int bh) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            vf[ks] = *reinterpret_cast<const frag8*>(v + head_off(bh) + (long)row_in * rs + ks * 16 + g * 8);
    };
    auto load_o = [&](int bh) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            of[ks] = *reinterpret_cast<const frag8*>(o + head_off_o(bh) + (long)row_in * rs_o + ks * 16 + g * 8);
        lse_in = lse[(long)bh * N + row_in];
    };

    // Walking workgroups take every gridDim-th head; the others one head each, neighbours on one XCD.
    int bh = Cfg::WALK ? (int)blockIdx.x : xcd_local_id(blockIdx.x, nheads);
    if (bh < 0 || bh >= nheads) return;
    {
        const Fetch f = fetch_of(bh);
        fetch_k(f);
        for (int i = 0; i < turns; ++i) fetch_rows(f, i);
    }
    load_v(bh);
    load_o(bh);

    while (true) {
        const int next = bh + gridDim.x;
        const bool more = Cfg::WALK && next < nheads;
        const long off = head_off(bh);
        const Fetch ahead = fetch_of(more ? next : bh);
        hold(vf);
        hold(of);
        asm volatile("" : "+v"(lse_in));
        asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // this head has landed

        // per-query scalars of this wavefront's query block: LSE*log2e (+inf past the end: weight 0) and -delta
        frag8 kf[KS], ktf[NB];
        if (wave_active) {
            float part = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const frag8 gf = ln.natural_row(Cfg::OFF_G + k0 * 128, ks);
#pragma unroll
                for (int e = 0; e < 8; ++e) part = fmaf(E::widen(of[ks], e), E::widen(gf, e), part);
                kf[ks] = ln.natural_row(Cfg::OFF_K + k0 * 128, ks);
            }
            const float dl = both_halves_sum(part);
            const int row = k0 + l32;
            if (g == 0) {
                sc[row] = row < N ? lse_in * kLog2e : INFINITY;
                sc[Cfg::MAX_N + row] = row < N ? -dl : 0.f;
            }
        }
        // K^T of this wavefront's dQ tiles: 16 channels, all keys
#pragma unroll
        for (int s = 0; s < NB; ++s) ktf[s] = quad_tr16(lds0 + Cfg::OFF_K, lane, c0, s);
        f32x16 dka[CT], dva[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            dka[ct] = f32x16_zero();
            dva[ct] = f32x16_zero();
        }
        lds_barrier();  // the scalars of every query are in LDS, the K tile is no longer read
        if (more) {
            fetch_k(ahead);
            load_o(next);
        }

        // dQ^T of block jj, this wavefront's 16 channels: K^T dS^T over the keys, or over 32-key steps s0 .. s1 - 1 of them
        f32x4 dqa[QT];
        auto form_dq_part = [&](int jj, int s0, int s1) {
            const char* dsj = ds + (jj & 1) * Cfg::DS_BYTES;
            const int nk = CAUSAL ? min(NB, jj + 1) : NB;
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                if (s0 == 0) dqa[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = s0; s < s1; ++s)
                    if (!CAUSAL || s < nk)
                        dqa[t] = E::mfma16(ktf[s], tr16_frag(dsj, Cfg::DS_STRIDE, lane, QT == 1 ? q16 : 16 * t, s), dqa[t]);
            }
        };
        auto form_dq = [&](int jj) { form_dq_part(jj, 0, NB); };
        auto store_dq = [&](int jj) {
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                const int row = 32 * jj + (QT == 1 ? q16 : 16 * t) + (lane & 15);
                if (row < N) store_tile16<E>(dqa[t], scale, dq + off + (long)row * rs + c0, lane);
            }
        };
        // scores and gradients of block j, beside dQ of the block before
        auto unit = [&](auto with_dq, auto diagonal, int j) {
            if (decltype(with_dq)::value && !Cfg::WALK) {
                form_dq(j - 1);
                store_dq(j - 1);
            }
            char* dsj = ds + (j & 1) * Cfg::DS_BYTES;
            const int query_base = 32 * j;
            const float* rowv = sc + query_base + 4 * g;
            f32x16 s, dp;
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                const f32x4 d4 = *reinterpret_cast<const f32x4*>(rowv + Cfg::MAX_N + 8 * a4);
#pragma unroll
                for (int e = 0; e < 4; ++e) dp[4 * a4 + e] = d4[e];
            }
            constexpr bool MASK = decltype(diagonal)::value;
            if constexpr (MASK) s = query_mask_block(query_base, g, k0 + l32);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const frag8 aq = ln.natural_row(query_base * 128, ks);
                const frag8 ag = ln.natural_row(Cfg::OFF_G + query_base * 128, ks);
                s = E::mfma(aq, kf[ks], ks == 0 && !MASK ? f32x16_zero() : s);
                dp = E::mfma(ag, vf[ks], dp);
            }
            if (decltype(with_dq)::value && Cfg::WALK && !SPLIT_DQ) form_dq(j - 1);
            char* mine = dsj + (k0 + l32) * Cfg::DS_STRIDE + 8 * g;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                f32x4 l4[2];
#pragma unroll
                for (int a4 = 0; a4 < 2; ++a4) l4[a4] = *reinterpret_cast<const f32x4*>(rowv + 8 * (2 * half + a4));
                if (decltype(with_dq)::value && SPLIT_DQ) form_dq_part(j - 1, half * (NB / 2), half ? NB : NB / 2);
                frag8 tg[CT], tq[CT];
                auto load_tr = [&] {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        tg[ct] = ln.transposed_row(Cfg::OFF_G + query_base * 128, ct, half);
                        tq[ct] = ln.transposed_row(query_base * 128, ct, half);
                    }
                };
                if (EARLY_TR) load_tr();
                u32x4 pf, df;
#pragma unroll
                for (int e = 8 * half; e < 8 * half + 8; ++e) {
                    const float pe = fast_exp2(fmaf(s[e], cs, -l4[e / 4 % 2][e % 4]));
                    s[e] = pe;
                    dp[e] = pe * dp[e];
                    if (e % 2 == 1) {
                        pf[(e / 2) % 4] = E::pack(s[e - 1], s[e]);
                        df[(e / 2) % 4] = E::pack(dp[e - 1], dp[e]);
                    }
                }
                if (!EARLY_TR) {
                    __builtin_amdgcn_sched_barrier(0);
                    load_tr();
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    dva[ct] = E::mfma(tg[ct], as_frag8(pf), dva[ct]);
                    dka[ct] = E::mfma(tq[ct], as_frag8(df), dka[ct]);
                }
                // keys past the end: their weights are taken against a score of 0 and may be anything
                if (k0 + 32 > N && k0 + l32 >= N) df = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    *reinterpret_cast<u32x2*>(mine + 16 * (2 * half + a)) = u32x2{df[2 * a], df[2 * a + 1]};
            }
        };
        // after dS of block j is complete its rows of Q and dO, and dS of the block before, are no longer read
        auto end_block = [&](int j) {
            lds_barrier();
            if (more && ((j & 1) || j + 1 == NB)) fetch_rows(ahead, j >> 1);
        };
        // causal: a block whose queries all lie before this wavefront's keys is not read by dQ either
        const int from = !wave_active ? NB : CAUSAL ? wave : 0;
        if (from == 0) unit(std::false_type{}, std::bool_constant<CAUSAL>{}, 0);
        end_block(0);
        int j = 1;
#pragma unroll 1
        for (; j < from; ++j) {
            form_dq(j - 1);
            store_dq(j - 1);
            end_block(j);
        }
        if (CAUSAL && from > 0 && from < NB) {
            unit(std::true_type{}, std::true_type{}, j);
            if (Cfg::WALK) store_dq(j - 1);
            end_block(j);
            ++j;
        }
#pragma unroll 1
        for (; j < NB; ++j) {
            unit(std::true_type{}, std::false_type{}, j);
            if (Cfg::WALK) store_dq(j - 1);
            end_block(j);
        }
        form_dq(NB - 1);
        store_dq(NB - 1);
        if (more) load_v(next);
        lds_barrier();  // the dS buffers are no longer read and stage the rows of dK and dV
        if (wave_active) {
            char* region = ds + wave * RowStore<D, E>::BYTES;
            const int lane_now = lane_from_exec();
            RowStore<D, E>::run(region, dka, scale, dk + off + (long)k0 * rs, rs, N - k0, lane_now);
            RowStore<D, E>::run(region, dva, 1.0f, dv + off + (long)k0 * rs, rs, N - k0, lane_now);
        }
        if (!more) break;
        bh = next;
    }
}
