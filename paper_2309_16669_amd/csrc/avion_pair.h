// dQ with two blocks of 32 queries per wavefront, for 64 channels, no mask, and launches that fill the chip (by_pair in
// avion_attn.hip).  Same operation, order of sums and, but for shared last blocks, bits as avion_dq_kernel's 32 x 32 form.
//
// That kernel runs a 32 x 32 block as a serial chain -- 8 products, the vector work, 4 products -- and leaves it to three
// wavefronts per SIMD to overlap; they do so poorly (its cycles are the sum of its matrix and its vector cycles).
// Here the overlap is in the code: while block A's scores of a 32-key step go through the vector work, the products
// of block B's (S, dP, and dQ of its previous step) stand beside it, then the other way round.  256 registers, two
// wavefronts per SIMD.  Both blocks read one K^T fragment, and 256 queries share a tile: half the transposed LDS
// reads and half the tile traffic.
// Workgroup = 4 wavefronts = 8 blocks; the last one of a head has the remaining blocks, of which one or two are shared
// by wavefronts that take every second or fourth 32-key unit and are added through LDS in a fixed order.
//
// Tiles are 64 rows of 128 bytes without padding (quad_at: four rows by four chunks at a time, the chunks permuted by a XOR
// with bits of the row number).  16 consecutive rows at one chunk, and 4 consecutive rows at 4 chunks (a transposing read's
// half wavefront), hit distinct banks: conflicts are 4 % of the LDS cycles instead of a third, a tile 16 KB instead of 18.
// The XOR touches two bits of the chunk, of which a lane's reads vary one, so four addresses per lane serve every read with
// the rest in the instruction's offset; they move on with the tile.  (With the chunks of a row permuted over all eight
// places each read needed an addition of its own, 12 % of the vector instructions.)  Four buffers: the
// products run one step ahead into the next tile, and a fetch has a whole tile's time beyond that to land.  Row operands
// are requested six products ahead.
// Measured, us, avion_dq_kernel -> this with an addition per read and operands three products ahead -> this: 384 heads x 1568
// 409 -> 385; 368.4 -> 358.2, 96 x 3000 317.5 -> 308.6, 96 x 1200 71.9 -> 64.7; 60.0 -> 58.7.  Not what binds: the order of the
// three products of a step (358 to 360 in three orders).  On all-zero operands 289 -> 276: on real ones the card's power
// limit takes a third of the clock.
// The same form of the forward gives nothing over four wavefronts per SIMD (281 -> 279).  dK/dV, one block per wavefront with the
// operands requested eight products ahead, is no faster at two wavefronts per SIMD than avion_dkdv_kernel at three (96 x 3000 390.7 ->
// 389.6, 384 x 1568 447.7 -> 466.5), and at one, with two blocks and half the LDS reads, slower (384 x 1568 456 -> 502): one
// wavefront issues an instruction every 4.6 cycles at most.
#pragma once
#include "avion_bwd.h"

// K and V tiles; every wavefront issues four loads a tile
struct PairRing {
    static constexpr int TILE = 64 * 128, BUF = 2 * TILE, NBUF = 4, LDS_BYTES = NBUF * BUF;
    unsigned smem_addr, va, half;
    u32x4 da, db;
    DEVINL PairRing(const raw16* a, long rs_a, const raw16* b, long rs_b, int N, const char* smem, int wave, int lane)
    {
        const RawBuffer ab(a, slice_bytes(rs_a, N, 64)), bb(b, slice_bytes(rs_b, N, 64));
        da = ab.words;
        db = bb.words;
        smem_addr = lds_address(smem) + wave * 1024;
        // quad_voff(wave, ...), spelt out: the compiler then needs no scratch for what it keeps of it (254 registers and 68 bytes otherwise)
        const int row = 8 * wave + lane / 32 * 4 + lane / 4 % 4, ch = lane / 16 % 2 * 4 + ((lane ^ (row >> 2)) & 3);
        va = row * (unsigned)(rs_a * 2) + ch * 16;
        half = 32 * (unsigned)(rs_a * 2);
    }
    DEVINL void fetch(int ti) const
    {
        const unsigned o0 = va + (unsigned)ti * 2 * half, o1 = o0 + half;
        load_to_lds16_x4<4096>(RawBuffer(da), RawBuffer(da), RawBuffer(db), RawBuffer(db), smem_addr + (ti & (NBUF - 1)) * BUF, o0, o1, o0, o1);
    }
    // all but the newest fetch of this wavefront have landed
    DEVINL static void landed_barrier() { asm volatile("s_waitcnt vmcnt(4)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
    DEVINL static void all_landed_barrier() { asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
};
constexpr int kPairBlocks = 8;  // blocks of 32 queries per workgroup
// which blocks a wavefront has (`mine` from blk0 on), and, where a block is shared, which of its `parts`.  The wavefront
// with a block less than the others moves with the workgroup (rot), so that no SIMD has it always.
struct PairSplit {
    int parts, part, mine, blk0;
    DEVINL PairSplit(int N, int qb, int wave, int rot)
    {
        const int nb = (N + 31) / 32, first = qb * kPairBlocks, cnt = min(kPairBlocks, nb - first), rw = (wave + rot) & 3;
        parts = cnt == 1 ? 4 : cnt == 2 ? 2 : 1;
        part = cnt == 1 ? wave : cnt == 2 ? wave / 2 : 0;
        mine = cnt <= 2 ? 1 : cnt / 4 + (rw < cnt % 4 ? 1 : 0);
        blk0 = cnt == 1 ? first : cnt == 2 ? first + wave % 2 : first + rw * (cnt / 4) + min(rw, cnt % 4);
    }
};

template <typename E>
struct PairD {
    frag8 qf[4], gf[4];
    f32x16 acc[2], s, dp;
    u32x4 df[2];
    float nlc, dl;
};
template <typename E>
__global__ void __launch_bounds__(256, 2)
avion_dq_pair_kernel(const raw16* __restrict__ q, const raw16* __restrict__ k, const raw16* __restrict__ v,
                    const raw16* __restrict__ o, const raw16* __restrict__ dO, const float* __restrict__ lse,
                    raw16* __restrict__ dq, float* __restrict__ rowsc, int H, int N, int rs_qkv, int rs_o, int nqb,
                    int nblocks, float cs, float scale)
{
    constexpr int D = 64, KS = 4, BN = 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int logical = xcd_local_id(blockIdx.x, nblocks);
    if (logical < 0) return;
    const int bh = logical / nqb, qb = logical % nqb;
    const int b = bh / H, h = bh % H;
    const int tid = threadIdx.x, lane = tid % 64, l32 = lane % 32, g = lane / 32;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const long rs = rs_qkv;
    const long head_off = (long)b * N * rs + (long)h * D;
    const long head_off_o = (long)b * N * rs_o + (long)h * D;
    const PairSplit sp(N, qb, wave, logical);
    const int ntiles = (N + BN - 1) / BN, nb = (N + 31) / 32;
    const PairRing ring(k + head_off, rs, v + head_off, rs, N, smem, wave, lane);
    QuadLane ln(lane, lds_address(smem));
    ring.fetch(0);
    ring.fetch(1);
    ring.fetch(2);
    using Blk = PairD<E>;
    Blk A, B;
    auto init = [&](Blk& x, int blk, bool write) {
        const int q0 = blk * 32;
        const int row = min(q0 + l32, N - 1);
        const long off = head_off + (long)row * rs + g * 8;
        const long off_o = head_off_o + (long)row * rs_o + g * 8;
        float psum = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            x.qf[ks] = *reinterpret_cast<const frag8*>(q + off + ks * 16);
            x.gf[ks] = *reinterpret_cast<const frag8*>(dO + off_o + ks * 16);
            const frag8 of = *reinterpret_cast<const frag8*>(o + off_o + ks * 16);
#pragma unroll
            for (int e = 0; e < 8; ++e) psum = fmaf(E::widen(of, e), E::widen(x.gf[ks], e), psum);
        }
        x.dl = both_halves_sum(psum);
        const float lc = lse[(long)bh * N + row] * kLog2e;
        x.nlc = -lc;
        const int qrow = q0 + l32, npad = (N + 63) & ~63;
        if (write && g == 0) {
            float* ws = rowsc + (long)bh * 2 * npad;
            ws[qrow] = qrow < N ? lc : INFINITY;
            ws[npad + qrow] = qrow < N ? -x.dl : 0.f;
            // an odd last block: the other half of its 64 rows is padding
            if (blk + 1 == nb && nb % 2 == 1) {
                ws[qrow + 32] = INFINITY;
                ws[npad + qrow + 32] = 0.f;
            }
        }
        x.acc[0] = x.acc[1] = f32x16_zero();
        x.df[0] = x.df[1] = u32x4{0, 0, 0, 0};
    };
    init(A, sp.blk0, sp.mine > 0 && sp.part == 0);
    init(B, sp.blk0 + (sp.mine > 1), sp.mine > 1);
    hold(A.qf); hold(B.qf); hold(A.gf); hold(B.gf);
    PairRing::all_landed_barrier();
    // from tile ti's buffer to the next one
    auto onward = [](int ti) { return (ti & 3) == 3 ? -3 * PairRing::BUF : PairRing::BUF; };
    auto grad = [&](Blk& x, int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i) {
            const float pe = fast_exp2(fmaf(x.s[i], cs, x.nlc));
            x.s[i] = pe * (x.dp[i] - x.dl);
            if (i % 2 == 1) x.df[i / 8][(i / 2) % 4] = E::pack(x.s[i - 1], x.s[i]);
        }
    };
    auto unit = [&](Blk& x, int key_base, int hk) {
        if (key_base >= N) return;
        x.s = key_base + 32 > N ? key_mask_block(key_base, lane_from_exec() / 32, N) : f32x16_zero();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            x.s = E::mfma(ln.natural(0, hk, ks), x.qf[ks], x.s);
            x.dp = E::mfma(ln.natural(PairRing::TILE, hk, ks), x.gf[ks], ks == 0 ? f32x16_zero() : x.dp);
        }
        grad(x, 0, 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) x.acc[i % 2] = E::mfma(ln.transposed(0, i % 2, 2 * hk + i / 2), as_frag8(x.df[i / 2]), x.acc[i % 2]);
    };
    const int nfast = N / BN;
    if (sp.mine == 2) {
        frag8 kf[4], fk[2], fv[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) kf[i] = frag8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            A.s = E::mfma(ln.natural(0, 0, ks), A.qf[ks], ks == 0 ? f32x16_zero() : A.s);
            A.dp = E::mfma(ln.natural(PairRing::TILE, 0, ks), A.gf[ks], ks == 0 ? f32x16_zero() : A.dp);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            fk[ks] = ln.natural(0, 0, ks);
            fv[ks] = ln.natural(PairRing::TILE, 0, ks);
        }
        // One phase: x's vector work beside y's products.  hk: the half tile y's scores are of; hkn: the one after it, to
        // whose buffer the addresses move by `by`.  Natural operands are requested two steps ahead.
        auto phase = [&](auto first, Blk& x, Blk& y, auto hk, auto hkn, int by) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                __builtin_amdgcn_sched_barrier(0);
                if (ks == 2 && by != 0) ln.move_nat(by);
                y.acc[ks % 2] = E::mfma(kf[ks], as_frag8(y.df[ks / 2]), y.acc[ks % 2]);
                if (decltype(first)::value) kf[ks] = ln.transposed(0, ks % 2, 2 * hk + ks / 2);
                y.s = E::mfma(fk[ks & 1], y.qf[ks], ks == 0 ? f32x16_zero() : y.s);
                y.dp = E::mfma(fv[ks & 1], y.gf[ks], ks == 0 ? f32x16_zero() : y.dp);
                fk[ks & 1] = ln.natural(0, ks < 2 ? hk : hkn, (ks + 2) % 4);
                fv[ks & 1] = ln.natural(PairRing::TILE, ks < 2 ? hk : hkn, (ks + 2) % 4);
                grad(x, 4 * ks, 4 * ks + 4);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        constexpr std::integral_constant<int, 0> lo{};
        constexpr std::integral_constant<int, 1> hi{};
        auto step = [&](auto hk, auto hkn, int by) {
            phase(std::true_type{}, A, B, hk, hkn, by);
            phase(std::false_type{}, B, A, hkn, hkn, 0);
        };
        for (int t = 0; t < nfast; ++t) {
            ring.fetch(t + 3);
            step(lo, hi, 0);
            step(hi, lo, onward(t));
            ln.move_tr(onward(t));
            PairRing::landed_barrier();
        }
        if (N % BN >= 32) step(lo, hi, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) B.acc[i % 2] = E::mfma(kf[i], as_frag8(B.df[i / 2]), B.acc[i % 2]);
        const int last = N / 32 * 32;
        if (N % BN >= 32) {
            unit(A, last, 1);
            unit(B, last, 1);
        } else {
            unit(A, last, 0);
            unit(B, last, 0);
        }
    } else {
        for (int t = 0; t < ntiles; ++t) {
            if (t < nfast) ring.fetch(t + 3);
#pragma unroll
            for (int hk = 0; hk < 2; ++hk)
                if (sp.mine == 1 && ((2 * t + hk) & (sp.parts - 1)) == sp.part) unit(A, t * BN + 32 * hk, hk);
            ln.move_nat(onward(t));
            ln.move_tr(onward(t));
            if (t < nfast) PairRing::landed_barrier();
        }
    }
    PairRing::all_landed_barrier();
    if (sp.parts > 1) {
        float* area = reinterpret_cast<float*>(smem + 4 * RowStore<D, E>::BYTES) + wave * 32 * 64 + lane_from_exec();
        if (sp.part > 0) {
#pragma unroll
            for (int i = 0; i < 32; ++i) area[i * 64] = A.acc[i / 16][i % 16];
        }
        __syncthreads();
        if (sp.part > 0) return;
        for (int p = 1; p < sp.parts; ++p) {
            const float* other = area + p * (4 / sp.parts) * 32 * 64;
#pragma unroll
            for (int i = 0; i < 32; ++i) A.acc[i / 16][i % 16] += other[i * 64];
        }
    }
    if (sp.mine == 0) return;
    char* region = smem + wave * RowStore<D, E>::BYTES;
    RowStore<D, E>::run(region, A.acc, scale, dq + head_off + (long)sp.blk0 * 32 * rs, rs, N - sp.blk0 * 32, lane_from_exec());
    if (sp.mine > 1)
        RowStore<D, E>::run(region, B.acc, scale, dq + head_off + (long)(sp.blk0 + 1) * 32 * rs, rs, N - (sp.blk0 + 1) * 32, lane_from_exec());
}

