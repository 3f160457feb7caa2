// Forward kernel: O = softmax(scale * Q K^T) V and LSE, one pass over the keys, nothing N x N stored
// (Sec. 3, "Flash Attention": implicit softmax weights, block-wise work out of on-chip memory;
// Sec. 1: block results combined into the exact output).
//
// Work split: one workgroup = NW wavefronts = 32*NW consecutive queries of one (batch, head).
// Each wavefront owns 32 queries and keeps
//   Q as MFMA B-operand fragments (lane = query, 8 channels per 16-deep step),
//   O^T accumulators (lane = query, registers = channels), the reference maximum and row sums.
// Keys and values come in LDS tiles of 64 tokens, two (K | V) buffers, rows in quad_at's order at 64 channels (padded
// ones at 80),
// filled straight from global memory by LDS-direct loads (no staging registers, no LDS writes):
// K rows are the A operand of S^T = K Q^T, and V is read through transposing LDS loads as the A
// operand of O^T = V^T P^T.  Computing the transposed products keeps every score of a query inside
// one lane pair, so the accumulator of the first contraction is, after rounding to the element
// format E (bf16 or fp16), directly the B operand of the second one (no LDS round trip).
//
// Schedule.  A wavefront issues in order, and an MFMA queued behind another one blocks what
// follows it, so a single wavefront cannot keep the matrix cores and the vector ALUs busy at once.
// The kernel therefore keeps the per-wavefront code simple and small in registers -- S^T, softmax,
// P V of one 32-key unit after the other -- and relies on several resident wavefronts per SIMD
// (four for d = 64) to fill each other's waits.  One workgroup barrier per 64-key tile: passing it
// certifies that the next tile has landed and that the previous one is no longer read, so that its
// buffer can be refilled.
//
// Softmax reference.  Weights are exp2(cs*s - m) with m fixed per query to the maximum over the
// first 32 keys.  Softmax is invariant to m, floating point keeps its relative precision at any
// magnitude, and the final division by the row sum cancels m exactly; the only failure mode is
// overflow when a later score exceeds m by ~100 binades (bf16; ~15 binades for fp16, whose weights
// must stay below 65504).  That is detected from the final row sum against E::kRowSumLimit
// (workgroup-wide), and the whole workgroup then recomputes its rows with the classic running
// maximum (avion_fwd_safe_pass).  Random or trained activations never get there.
//
// Small launches.  With KG > 1 a workgroup holds KG groups of NW wavefronts for the same 32*NW queries;
// each group walks its own share of the key tiles through its own two buffers, with its own reference,
// and group 0 adds the others' accumulators and sums, rescaled to the larger reference, in a fixed
// order at the end.  What bounds a launch that leaves compute units with one workgroup is the serial
// chain of one wavefront per SIMD, which this shortens (the rule and both sides' times stand at
// fwd_cut in avion_attn.hip).
//
// What bounds it on a full chip: vector issue and, behind it, LDS.  Padded rows of 144 bytes -> quad_at's layout (no bank conflicts,
// an eighth less deposited, a tile's loads in one statement), us, same bits: 384 heads x 1568 285.7 -> 280.9, causal 172.1 -> 168.7, 96 x
// 3000 253.8 -> 249.3, 3072 x 196 78.1 -> 76.0, 16384 x 77 183.4 -> 175.6 (causal 176.4), x 40 causal 101.5 -> 95.8; 0.93 to 1.007 of the time over 31
// shapes.  Launches in a graph: 8 x 77 causal 4.92 -> 4.63, 8 x 600 8.91 -> 8.26, 16 x 400 7.96 -> 7.39.  Of the LDS cycles on 384 x 1568, 2.9 %
// instead of 34 % are conflicts, and LDS is busy 25 % of the launch instead of 37.  (dK/dV in it, at three wavefronts per SIMD,
// 452.7 -> 465.2: the two addresses more take registers that keep operands in flight.)
//
// Template parameters: head dim D, wavefronts per group NW, groups KG, element format E (Bf16 or F16),
// CAUSAL (query i sees keys 0..i; the reference m is then the maximum over the visible ones of the
// first 32 keys -- key 0 is visible to every query).
#pragma once
#include "avion_common.h"

template <int D, int NW, int KG>
struct FwdCfg {
    static constexpr int BN = 64;
    static constexpr int NT = NW * KG * 64;
    static constexpr int BM = 32 * NW;
    using Ring = std::conditional_t<D == 64, QuadRing<NW>, TileRing<D, NW, 2, false>>;
    using Stage = TileStage<D, BN, NT>;  // the fallback pass stages its tiles through registers
    // the fallback's two buffers of padded tiles (its last row's reads too), or the groups' rings
    static constexpr int SAFE_BYTES = 4 * Stage::BYTES + (D % 32 != 0 ? 64 : 0);
    static constexpr int LDS_BYTES = KG * Ring::LDS_BYTES > SAFE_BYTES ? KG * Ring::LDS_BYTES : SAFE_BYTES;
    // wavefronts per SIMD the register budget is sized for: what LDS lets a compute unit hold, at most 4;
    // with several groups one workgroup per compute unit, with two groups up to two: six wavefronts each may put four on one SIMD
    // (40 heads x 785 18.4 -> 22.4 us at 130 registers instead of 128; blocks of 64 rows, which never need it, take 128 to 130 either way
    // and the same time: 8 x 77 causal 4.66, 4.68 without)
    static constexpr int WG_PER_CU = 160 * 1024 / LDS_BYTES;
    static constexpr int WAVES_PER_SIMD = KG == 2 && D == 64 ? 4 : KG > 1 ? (NW * KG + 3) / 4 : WG_PER_CU * NW / 4 > 4 ? 4 : WG_PER_CU * NW / 4;
};

// Classic online softmax with a running maximum, one 64-key tile at a time, staged through
// registers into two buffers of padded tiles.  Used only as the fallback described above; same register
// layouts as the main loop.
// key_limit: this lane's query sees keys below it (N, or query + 1 for causal attention).
template <int D, int NW, int KG, typename E>
DEVINL void avion_fwd_safe_pass(char* smem, const SliceView& kh, const SliceView& vh, const frag8 (&qf)[D / 16],
                                f32x16 (&oacc)[(D + 31) / 32], float& m_used, float& lsum, float& rsum, int N,
                                int key_limit, float cs, bool wave_active, int tid, int lane)
{
    using Cfg = FwdCfg<D, NW, KG>;
    using Stage = typename Cfg::Stage;
    constexpr int BN = 64, STRIDE = Stage::STRIDE, KS = D / 16, CT = (D + 31) / 32;
    const int l32 = lane % 32, g = lane / 32, tr_off = tr_lane_offset(lane, STRIDE);
    auto kbuf = [&](int i) { return smem + i * 2 * Stage::BYTES; };
    auto vbuf = [&](int i) { return smem + (2 * i + 1) * Stage::BYTES; };
    m_used = -INFINITY;
    lsum = 0.f;
    rsum = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) oacc[ct] = f32x16_zero();
    Stage kst, vst;
    __syncthreads();
    kst.load(kh, 0, tid);
    vst.load(vh, 0, tid);
    kst.store(kbuf(0), tid);
    vst.store(vbuf(0), tid);
    __syncthreads();
    const int ntiles = (N + BN - 1) / BN;
    for (int t = 0; t < ntiles; ++t) {
        const char* kc = kbuf(t & 1);
        const char* vc = vbuf(t & 1);
        const bool more = t + 1 < ntiles;
        if (more) {
            kst.load(kh, (t + 1) * BN, tid);
            vst.load(vh, (t + 1) * BN, tid);
        }
        if (wave_active) {
#pragma unroll
            for (int kt = 0; kt < BN / 32; ++kt) {
                f32x16 s;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    s = E::mfma(nat_frag(kc, STRIDE, 32 * kt + l32, ks, g), qf[ks], ks == 0 ? f32x16_zero() : s);
                const int key0 = t * BN + 32 * kt + 4 * g;
                if (key0 + 28 >= key_limit) {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (key0 + 8 * (i / 4) + (i % 4) >= key_limit) s[i] = -INFINITY;
                }
                const float m2 = both_halves_max(max16(s)) * cs;
                const float mn = fmaxf(m_used, m2);  // finite: key 0 is seen by every query
                const float alpha = fast_exp2(m_used - mn);
                m_used = mn;
                lsum *= alpha;
                rsum *= alpha;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[ct][i] *= alpha;
                float rowsum = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float p = fast_exp2(fmaf(s[i], cs, -mn));
                    s[i] = p;
                    rowsum += p;
                }
                lsum += rowsum;
                const frag8 pf0 = acc_to_frag<E>(s, 0), pf1 = acc_to_frag<E>(s, 1);
                rsum = frag_sum<E>(pf1, frag_sum<E>(pf0, rsum));
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        oacc[ct] = E::mfma(tr_frag(vc, STRIDE, tr_off, ct, 2 * kt + half), half == 0 ? pf0 : pf1, oacc[ct]);
            }
        }
        if (more) {
            kst.store(kbuf((t + 1) & 1), tid);
            vst.store(vbuf((t + 1) & 1), tid);
        }
        __syncthreads();
    }
}

// (The causal instances too fit 128 registers without a spill at d = 64; at 136 and three wavefronts per SIMD 16384 heads x 77
// took 153 us instead of 135, x 40 99 instead of 85, 384 x 1568 192 instead of 179.)
template <int D, int NW, int KG, typename E, bool CAUSAL>
__global__ void __launch_bounds__((FwdCfg<D, NW, KG>::NT), (FwdCfg<D, NW, KG>::WAVES_PER_SIMD))
avion_fwd_kernel(const raw16* __restrict__ q, const raw16* __restrict__ k, const raw16* __restrict__ v,
                 raw16* __restrict__ o, float* __restrict__ lse, int H, int N, int rs_qkv, int rs_o, int nqb, int nblocks,
                 float cs)
{
    using Cfg = FwdCfg<D, NW, KG>;
    using Ring = typename Cfg::Ring;
    constexpr int BN = Cfg::BN, BM = Cfg::BM;
    constexpr int KS = D / 16;         // 16-deep steps over the channels
    constexpr int CT = (D + 31) / 32;  // 32-channel tiles of O^T
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int logical = xcd_local_id(blockIdx.x, nblocks);
    if (logical < 0) return;
    const int bh = logical / nqb, qb = logical % nqb;
    const int b = bh / H, h = bh % H;
    const int tid = threadIdx.x, lane = tid % 64, l32 = lane % 32, g = lane / 32;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid / 64);
    // Wavefront of its group, and the group.  Which one has the last rows turns with the head, so that the one without rows (or,
    // causal, with the longest walk) is not on the same SIMD in every workgroup: 384 heads x 1568 causal 167.6 -> 164.1 us, 3072 x
    // 196 79.3 -> 77.8, 384 x 200 12.57 -> 12.35, whole blocks without mask equal.
    const int wave = (wave_id + bh) % NW, grp = KG == 1 ? 0 : wave_id / NW;
    // token rows of Q, K, V are rs_qkv elements apart, those of O rs_o; a batch entry is N such rows
    const long rs = rs_qkv;
    const long head_off = (long)b * N * rs + (long)h * D;
    const long head_off_o = (long)b * N * rs_o + (long)h * D;
    const SliceView kh(k + head_off, rs, N, D);
    const SliceView vh(v + head_off, rs, N, D);
    const int q0 = qb * BM + wave * 32;  // first query of this wavefront
    const bool wave_active = q0 < N;
    // Keys this lane's query sees: all N, or 0..query for causal attention.  For the whole wavefront:
    // units that start at or beyond wave_key_end are skipped, units that reach beyond mask_from start
    // their scores from the mask; the workgroup streams the tiles up to its last query only.
    const int key_limit = CAUSAL ? min(N, q0 + l32 + 1) : N;
    const int wave_key_end = CAUSAL ? min(N, q0 + 32) : N;
    const int mask_from = CAUSAL ? min(N, q0 + 1) : N;
    const int ntiles = ((CAUSAL ? min(N, qb * BM + BM) : N) + BN - 1) / BN;

    // tiles of this key group; every group passes the same barriers
    const int per = (ntiles + KG - 1) / KG, t0 = grp * per, t1 = min(ntiles, t0 + per);

    const Ring ring(k + head_off, rs, v + head_off, rs, N, nullptr, 0, ntiles, smem + grp * Ring::LDS_BYTES, wave, lane);
    if (KG == 1 || t0 < t1) ring.fetch(t0);
    RingLane<Ring> ln(ring, lane, t0);

    // Q fragments stay in registers for the whole kernel
    frag8 qf[KS];
    {
        const int row = min(q0 + l32, N - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = *reinterpret_cast<const frag8*>(q + head_off + (long)row * rs + ks * 16 + g * 8);
    }
    f32x16 oacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) oacc[ct] = f32x16_zero();
    float m_used = 0.f, lsum = 0.f;
    f32x4 rs4 = {0.f, 0.f, 0.f, 0.f};  // four equal values

    hold(qf);
    Ring::landed_barrier();  // tile 0 is in LDS (and the Q fragments have arrived)

    // S^T of one unit (32 keys starting at row 32*hk of the K tile); RAGGED units reach past the
    // last key and start from the key mask instead of zero
    auto scores = [&](auto ragged, int hk, int key_base) -> f32x16 {
        constexpr bool RAGGED = decltype(ragged)::value;
        f32x16 s;
        if constexpr (RAGGED) s = key_mask_block(key_base, g, key_limit);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            s = E::mfma(ln.natural(0, hk, ks), qf[ks], ks == 0 && !RAGGED ? f32x16_zero() : s);
        return s;
    };
    // reference maximum: over the first 32 keys (of this group's); their scores serve the first unit too, one of three
    // at 77 tokens (forming them twice: 8 heads x 77 causal 5.44 -> 5.13 us, 16384 x 40 84.0 -> 80.7, x 77 134.4 -> 132.7,
    // 3072 x 196 84.3 -> 82.8, d = 80 113.8 -> 112.0)
    f32x16 first = f32x16_zero();
    if (wave_active && (KG == 1 || t0 < t1)) {
        first = scores(std::true_type{}, 0, t0 * BN);
        m_used = both_halves_max(max16(first)) * cs;
        // a query that sees none of them (causal, a later group): any finite reference will do, its weights
        // must come out as 0
        if (KG > 1 && CAUSAL) m_used = t0 * BN < key_limit ? m_used : 0.f;
    }
    // weights of one unit from its scores, and their product with V
    auto weigh = [&](f32x16 s, int hk) {
        // the V^T operands are requested before the vector work so that they are there after it
        frag8 vf[2][CT];
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) vf[half][ct] = ln.transposed(Ring::OFF_B, ct, 2 * hk + half);
        u32x4 pf[2];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float p = fast_exp2(fmaf(s[i], cs, -m_used));
            s[i] = p;
            lsum += p;
            if (i % 2 == 1) pf[i / 8][(i / 2) % 4] = E::pack(s[i - 1], p);
        }
        // the second row sum runs over the weights as rounded to the element format, i.e. the numbers the
        // second contraction multiplies V with; O is divided by it.  Summed by products with ones: 8 cycles of
        // the matrix cores for four weights, where two packed additions keep the vector issue port, which is
        // the scarcer of the two here, for 16.  384 heads x 1568 293 -> 281 us, causal 192 -> 182.
#pragma unroll
        for (int i = 0; i < 4; ++i) rs4 = E::add_four(u32x2{pf[i / 2][2 * (i % 2)], pf[i / 2][2 * (i % 2) + 1]}, rs4);
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) oacc[ct] = E::mfma(vf[half][ct], as_frag8(pf[half]), oacc[ct]);
    };
    auto tile = [&](auto first_tile, int t) {
        if (KG == 1 || t + 1 < t1) ring.fetch(t + 1);  // into the buffer of tile t-1, which nobody reads any more
        ln.enter(ring, t);
        if (wave_active && (KG == 1 || t < t1)) {
#pragma unroll
            for (int hk = 0; hk < 2; ++hk) {
                const int key_base = t * BN + 32 * hk;
                if (key_base >= wave_key_end) continue;  // past the last key, or (causal) seen by no query of this wavefront
                if (decltype(first_tile)::value && hk == 0) {
                    weigh(first, hk);
                    continue;
                }
                f32x16 s;
                if (key_base + 32 > mask_from) s = scores(std::true_type{}, hk, key_base);
                else s = scores(std::false_type{}, hk, key_base);
                weigh(s, hk);
            }
        }
        ln.leave(t);
        Ring::landed_barrier();  // tile t+1 has landed; tile t is no longer read
    };
    tile(std::true_type{}, t0);
    for (int t = t0 + 1; t < t0 + per; ++t) tile(std::false_type{}, t);

    float rsum = rs4[0];
    // overflow of the fixed reference: redo this workgroup's rows with the running maximum
    bool bad = false;
    if (wave_active) bad = !(both_halves_sum(lsum) <= E::kRowSumLimit);
    const bool redo = __syncthreads_or(bad ? 1 : 0);
    if (redo)
        avion_fwd_safe_pass<D, NW, KG, E>(smem, kh, vh, qf, oacc, m_used, lsum, rsum, N, key_limit, cs,
                                          wave_active && grp == 0, tid, lane_from_exec());
    if constexpr (KG > 1) {
        // The groups' results meet in LDS (behind the row-store areas of the epilogue) as [value][lane]
        // floats and are added in group order, each scaled to the larger of the two references.  After a
        // redone pass group 0 holds everything.
        constexpr int VALS = CT * 16 + 3, WAVE_BYTES = VALS * 256;
        static_assert(NW * RowStore<D, E>::BYTES + (KG - 1) * NW * WAVE_BYTES <= Cfg::LDS_BYTES, "exchange area");
        char* area = smem + NW * RowStore<D, E>::BYTES;
        if (grp > 0 && wave_active && !redo) {
            float* mine = reinterpret_cast<float*>(area + ((grp - 1) * NW + wave) * WAVE_BYTES) + lane_from_exec();
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int i = 0; i < 16; ++i) mine[(ct * 16 + i) * 64] = oacc[ct][i];
            mine[(VALS - 3) * 64] = lsum;
            mine[(VALS - 2) * 64] = rsum;
            // a query that sees no key of this group: reference -inf, so that nothing of it counts
            mine[(VALS - 1) * 64] = t0 < t1 && t0 * BN < key_limit ? m_used : -INFINITY;
        }
        __syncthreads();
        if (grp > 0) return;
        if (wave_active && !redo) {
#pragma unroll
            for (int og = 0; og < KG - 1; ++og) {
                const float* other = reinterpret_cast<const float*>(area + (og * NW + wave) * WAVE_BYTES) + lane_from_exec();
                const float m2 = other[(VALS - 1) * 64];
                const float mn = fmaxf(m_used, m2), a1 = fast_exp2(m_used - mn), a2 = fast_exp2(m2 - mn);
                lsum = lsum * a1 + other[(VALS - 3) * 64] * a2;
                rsum = rsum * a1 + other[(VALS - 2) * 64] * a2;
                m_used = mn;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[ct][i] = oacc[ct][i] * a1 + other[(ct * 16 + i) * 64] * a2;
            }
        }
    }

    // every wavefront is past its last tile read (barrier above): the tile buffers are free and
    // serve as the per-wavefront staging area of the output rows
    if (!wave_active) return;
    const float l = both_halves_sum(lsum);
    const float inv = 1.0f / both_halves_sum(rsum);
    // each lane scales by its own query's divisor before the rows are transposed
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][i] *= inv;
    const int lane_now = lane_from_exec();
    RowStore<D, E>::run(smem + wave * RowStore<D, E>::BYTES, oacc, 1.0f, o + head_off_o + (long)q0 * rs_o, rs_o, N - q0, lane_now);
    if (lane_now < 32 && q0 + lane_now < N) lse[(long)bh * N + q0 + lane_now] = (m_used + __builtin_amdgcn_logf(l)) * kLn2;
}
