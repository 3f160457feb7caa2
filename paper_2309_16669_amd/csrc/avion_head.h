// Whole backward of one (batch, head) in one workgroup and one pass over memory, for sequences of at most
// 32 * NW tokens with 64 channels (spatial attention over a frame's 14 x 14 tokens, captions).
//
// At these lengths the backward is bound by memory: 8 tensors of N x 64 for 10 N^2 64 operations.  The two
// kernels of avion_bwd.h read Q, K, V, O, dO and Q, K, V, dO and form S and dP twice; here Q, K and dO come
// into LDS once, V and O into registers, S and dP are formed once, and dQ, dK and dV leave together.
//
// Wavefront w owns keys 32w..32w+31: K, V as B operands, dK^T and dV^T as accumulators, exactly the unit of
// avion_dkdv_body.  The workgroup walks the query blocks j of 32 together.  Each wavefront leaves its
// 32 x 32 block of dS (rounded to the element format, as the second contraction takes it) in LDS, one row
// per key; after one barrier the NW wavefronts form dQ^T of block j, [64 channels x 32 queries], in
// 16 x 16 tiles over all keys (16x16x32 products): their K^T fragments stay in registers, dS^T is read
// through transposing loads.  Two dS buffers, so that one barrier per block is enough.  No atomics, no
// partial sums in memory.  avion_dq_body's TILE16 form takes the same operands in the same order, so the
// backward's two phases give this kernel's bits.
//
// 8 wavefronts (129..256 tokens): 146 KB of LDS, one workgroup per compute unit, so nothing else covers its
// loads.  It walks the heads: K's tile is free once the operands are in registers, 64 rows of Q and dO once
// their two blocks are done, and the next head's rows are fetched into them right then, without registers
// (LDS-direct loads); O, V and LSE follow in registers.  4 wavefronts (33..128 tokens): two workgroups per
// compute unit overlap each other, one head each.
// Measured, whole backward, us, two kernels -> this one: 3072 heads x 196 252 -> 191 (616 MB: 3.2 TB/s; one
// head per workgroup 259), x 160 203 -> 144, x 256 298 -> 248, 8000 x 200 causal 583 -> 460; one launch of
// two passes -> this one: 16384 x 77 causal 367 -> 304 (4.3 TB/s), 4000 x 128 143 -> 119, 8 x 77 10.5 -> 8.6.
// Few heads (nothing is walked up to 256; 257..511 leave half the chip idle in the second round), two kernels
// of one group each -> this one: 8 x 200 16.9 -> 15.3, 256 x 200 27.9 -> 19.5, 257 x 200 31.4 -> 30.1,
// 384 x 200 36.7 -> 32.7, 8 x 256 17.7 -> 17.0, 257 x 256 36.1 -> 35.5; 0.60 to 0.99 of the two at 1 to 768
// heads x 129..256, causal and not.  Two kernels of two groups each (by_split's form for at most 256 64-row
// blocks) are slower than this one up to 192 tokens and from 96 heads on, and faster below that: by 0 to 4 %
// at 196..224 tokens, 8 to 14 % at 240..256.
// dQ in 32 x 32 tiles after every fourth block (fewer barriers, longer chains): 226 at 3072 x 196.
#pragma once
#include "avion_common.h"

template <int NW>
struct HeadCfg {
    static constexpr int D = 64, NT = NW * 64, MAX_N = 32 * NW;
    static constexpr int STRIDE = tile_stride<D>();
    static constexpr int TILE_BYTES = MAX_N * STRIDE;    // Q, dO, K: all rows of the head
    static constexpr int DS_STRIDE = 72;                 // 32 queries of 2 bytes, padded so that 32 rows hit distinct banks
    static constexpr int DS_BYTES = MAX_N * DS_STRIDE;   // one key per row
    static constexpr int OFF_G = TILE_BYTES, OFF_K = 2 * TILE_BYTES, OFF_DS = 3 * TILE_BYTES, OFF_SC = OFF_DS + 2 * DS_BYTES;
    static constexpr int LDS_BYTES = OFF_SC + 2 * MAX_N * 4;  // LSE*log2e and -delta per query
    // one workgroup per compute unit: it walks several heads
    static constexpr bool WALK = 2 * LDS_BYTES > 160 * 1024;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
    static_assert(TILE_BYTES % 1024 == 0, "the tile mover fills whole 1 KB blocks");
    static_assert(NW * RowStore<D, Bf16>::BYTES <= 2 * DS_BYTES, "the epilogue stages its rows in the dS buffers");
};

// barrier that orders LDS accesses only: loads and stores to memory stay in flight
DEVINL void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int NW, typename E, bool CAUSAL>
__global__ void __launch_bounds__(NW * 64, 2)
avion_bwd_head_kernel(const raw16* __restrict__ q, const raw16* __restrict__ k, const raw16* __restrict__ v,
                      const raw16* __restrict__ o, const raw16* __restrict__ dO, const float* __restrict__ lse,
                      raw16* __restrict__ dq, raw16* __restrict__ dk, raw16* __restrict__ dv, int H, int N, int rs_qkv, int rs_o,
                      int nheads, float cs, float scale)
{
    using Cfg = HeadCfg<NW>;
    constexpr int D = 64, KS = 4, CT = 2, STRIDE = Cfg::STRIDE, QT = 8 / NW;  // QT: 16-query tiles of dQ per wavefront
    constexpr int SUB_BLOCKS = 64 * STRIDE / 1024;                            // 1 KB blocks of 64 rows of one tensor
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid % 64, l32 = lane % 32, g = lane / 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const long rs = rs_qkv;
    const int k0 = wave * 32;  // first key, and for the per-query scalars first query, of this wavefront
    const int nb = (N + 31) / 32, nslots = (N + 63) / 64;
    const bool wave_active = k0 < N;
    const char *qt = smem, *gt = smem + Cfg::OFF_G, *kt = smem + Cfg::OFF_K;
    char* ds = smem + Cfg::OFF_DS;
    float* sc = reinterpret_cast<float*>(smem + Cfg::OFF_SC);
    const unsigned lds0 = lds_address(smem);
    const int row_in = min(k0 + l32, N - 1);
    const int tr_off = tr_lane_offset(lane, STRIDE);
    const int c0 = 16 * (wave % 4), q16 = NW == 8 ? 16 * (wave / 4) : 0;  // this wavefront's dQ tile(s)

    auto head_off = [&](int bh) { return (long)(bh / H) * N * rs + (long)(bh % H) * D; };
    auto head_off_o = [&](int bh) { return (long)(bh / H) * N * rs_o + (long)(bh % H) * D; };
    // 1 KB blocks dealt round robin to the wavefronts; rows past the end arrive as zeros
    auto fetch_k = [&](int bh) {
        const RawBuffer buf(k + head_off(bh), slice_bytes(rs, N, D));
        for (int idx = wave; idx < nslots * SUB_BLOCKS; idx += NW)
            load_to_lds16(buf, __builtin_amdgcn_readfirstlane(lds0 + Cfg::OFF_K + idx * 1024),
                          padded_block_voff<D>(idx, lane, (unsigned)(rs * 2)));
    };
    // 64 rows of Q and of dO
    auto fetch_slot = [&](int bh, int slot) {
        const RawBuffer qb(q + head_off(bh), slice_bytes(rs, N, D)), gb(dO + head_off_o(bh), slice_bytes(rs_o, N, D));
        for (int i = wave; i < 2 * SUB_BLOCKS; i += NW) {
            const bool of_q = i < SUB_BLOCKS;
            const int idx = slot * SUB_BLOCKS + (of_q ? i : i - SUB_BLOCKS);
            load_to_lds16(pick(of_q, qb, gb), __builtin_amdgcn_readfirstlane(lds0 + (of_q ? 0 : Cfg::OFF_G) + idx * 1024),
                          padded_block_voff<D>(idx, lane, (unsigned)((of_q ? rs : (long)rs_o) * 2)));
        }
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
    fetch_k(bh);
    for (int slot = 0; slot < nslots; ++slot) fetch_slot(bh, slot);
    load_v(bh);
    load_o(bh);

    while (true) {
        const int next = bh + gridDim.x;
        const bool more = Cfg::WALK && next < nheads;
        const long off = head_off(bh);
        hold(vf);
        hold(of);
        asm volatile("" : "+v"(lse_in));
        asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // this head has landed

        // per-query scalars of this wavefront's query block: LSE*log2e (+inf past the end: weight 0) and -delta
        frag8 kf[KS], ktf[NW];
        if (wave_active) {
            float part = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const frag8 gf = nat_frag(gt, STRIDE, k0 + l32, ks, g);
#pragma unroll
                for (int e = 0; e < 8; ++e) part = fmaf(E::widen(of[ks], e), E::widen(gf, e), part);
                kf[ks] = nat_frag(kt, STRIDE, k0 + l32, ks, g);
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
        for (int s = 0; s < NW; ++s)
            if (s < nb) ktf[s] = tr16_frag(kt, STRIDE, lane, c0, s);
        f32x16 dka[CT], dva[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            dka[ct] = f32x16_zero();
            dva[ct] = f32x16_zero();
        }
        lds_barrier();  // the scalars of every query are in LDS, the K tile is no longer read
        if (more) {
            fetch_k(next);
            load_o(next);
        }

        for (int j = 0; j < nb; ++j) {
            char* dsj = ds + (j & 1) * Cfg::DS_BYTES;
            const int query_base = 32 * j;
            // causal: a block whose queries all lie before this wavefront's keys is not read below either
            if (wave_active && !(CAUSAL && j < wave)) {
                const float* rowv = sc + query_base + 4 * g;
                f32x16 s, dp;
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) {
                    const f32x4 d4 = *reinterpret_cast<const f32x4*>(rowv + Cfg::MAX_N + 8 * a4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dp[4 * a4 + e] = d4[e];
                }
                if constexpr (CAUSAL) {
                    if (j == wave) s = query_mask_block(query_base, g, k0 + l32);
                    else s = f32x16_zero();
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const frag8 aq = nat_frag(qt, STRIDE, query_base + l32, ks, g);
                    const frag8 ag = nat_frag(gt, STRIDE, query_base + l32, ks, g);
                    s = E::mfma(aq, kf[ks], ks == 0 && !CAUSAL ? f32x16_zero() : s);
                    dp = E::mfma(ag, vf[ks], dp);
                }
                f32x4 l4[4];
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) l4[a4] = *reinterpret_cast<const f32x4*>(rowv + 8 * a4);
                char* mine = dsj + (k0 + l32) * Cfg::DS_STRIDE + 8 * g;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    frag8 tg[CT], tq[CT];
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        tg[ct] = tr_frag(gt, STRIDE, tr_off, ct, 2 * j + half);
                        tq[ct] = tr_frag(qt, STRIDE, tr_off, ct, 2 * j + half);
                    }
                    u32x4 pf, df;
#pragma unroll
                    for (int e = 8 * half; e < 8 * half + 8; ++e) {
                        const float pe = fast_exp2(fmaf(s[e], cs, -l4[e / 4][e % 4]));
                        s[e] = pe;
                        dp[e] = pe * dp[e];
                        if (e % 2 == 1) {
                            pf[(e / 2) % 4] = E::pack(s[e - 1], s[e]);
                            df[(e / 2) % 4] = E::pack(dp[e - 1], dp[e]);
                        }
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
            }
            lds_barrier();  // dS of block j is complete; its rows of Q and dO are no longer read
            if (more && ((j & 1) || j + 1 == nb)) fetch_slot(next, j >> 1);

            // dQ^T of block j, this wavefront's 16 channels: K^T dS^T over the keys
            const int nk = CAUSAL ? min(nb, j + 1) : nb;
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                const int qc = QT == 1 ? q16 : 16 * t;
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < NW; ++s)
                    if (s < nk) acc = E::mfma16(ktf[s], tr16_frag(dsj, Cfg::DS_STRIDE, lane, qc, s), acc);
                const int row = query_base + qc + (lane & 15);
                if (row < N) store_tile16<E>(acc, scale, dq + off + (long)row * rs + c0, lane);
            }
        }
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
