// dQ with two blocks of 32 queries per wavefront, for 64 channels, no mask, and launches that fill the chip (by_pair in
// avion_attn.hip).  Same operation, order of sums and, but for shared last blocks, bits as avion_dq_kernel's 32 x 32 form.
//
// That kernel runs a 32 x 32 block as a serial chain -- 8 products, the vector work, 4 products -- and leaves it to three
// wavefronts per SIMD to overlap; they do so poorly (its cycles are the sum of its matrix and its vector cycles).
// Here the overlap is in the code: while block A's scores of a 32-key step go through the vector work, the products
// of block B's (S, dP, and dQ of its previous step) stand beside it, then the other way round.  255 registers, two
// wavefronts per SIMD.  Both blocks read one K^T fragment, and 256 queries share a tile: half the transposed LDS
// reads and half the tile traffic.
// Workgroup = 4 wavefronts = 8 blocks; the last one of a head has the remaining blocks, of which one or two are shared
// by wavefronts that take every second or fourth 32-key unit and are added through LDS in a fixed order.
//
// Tiles are 64 rows of 128 bytes without padding, 16-byte chunks permuted within a row by a XOR with bits of the row
// number: 16 consecutive rows at one chunk, and 4 consecutive rows at 4 chunks (a transposing read's half wavefront), hit
// distinct banks; conflicts fall from a third of the LDS cycles to 4 %, a tile from 18 KB to 16.  Four buffers: the
// products run one step ahead into the next tile, and a fetch has a whole tile's time beyond that to land.
// Measured, us, avion_dq_kernel -> this: 384 heads x 1568 409 -> 385 (389 -> 367 on another card), x 3000 1367 -> 1227,
// 64 x 3528 333 -> 316.  What bounds it now: matrix cores 55 % and vector issue 70 % of the cycles busy at 1.75 GHz.
// The same form of the forward gives nothing over four wavefronts per SIMD (281 -> 279), of dK/dV (one block, pipelined
// over half steps) 431 -> 478: it reads twice the LDS operands per product.
#pragma once
#include "avion_bwd.h"

// chunk permutation of a row
DEVINL int swz(int row) { const int p = row >> 1; return (p & 1) << 2 | (p & 2) | (p >> 2 & 1); }
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
        const int row = 8 * wave + lane / 8;
        va = row * (unsigned)(rs_a * 2) + ((lane % 8) ^ swz(row)) * 16;
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
// this lane's addresses in a tile
struct PairLane {
    unsigned nat0, tr0;
    DEVINL PairLane(int lane)
    {
        const int l32 = lane % 32, g = lane / 32, G = lane >> 4, j = lane & 15, r = 4 * (G >> 1) + (j >> 2);
        nat0 = l32 * 128 + (g ^ swz(l32)) * 16;
        tr0 = r * 128 + ((2 * (G & 1) + ((j & 3) >> 1)) ^ swz(r)) * 16 + (j & 1) * 8;
    }
    // the XORs below stay at their uses instead of living in registers of their own
    DEVINL frag8 natural(unsigned tile, int hk, int ks) const
    {
        typedef const __attribute__((address_space(3))) frag8* ptr;
        return *(ptr)((nat0 ^ (unsigned)(ks * 32)) + tile + hk * 4096);
    }
    DEVINL frag8 transposed(unsigned tile, int ct, int step) const
    {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((tr0 ^ (unsigned)(ct * 64)) + tile + step * 2048));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((tr0 ^ (unsigned)(ct * 64 + 16)) + tile + step * 2048 + 1024));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        return as_frag8(u32x4{l2[0], l2[1], h2[0], h2[1]});
    }
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
    const PairLane ln(lane);
    const unsigned lds0 = lds_address(smem);
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
    auto buf = [&](int ti) { return lds0 + (unsigned)(ti & 3) * PairRing::BUF; };
    auto grad = [&](Blk& x, int i0, int i1) {
#pragma unroll
        for (int i = i0; i < i1; ++i) {
            const float pe = fast_exp2(fmaf(x.s[i], cs, x.nlc));
            x.s[i] = pe * (x.dp[i] - x.dl);
            if (i % 2 == 1) x.df[i / 8][(i / 2) % 4] = E::pack(x.s[i - 1], x.s[i]);
        }
    };
    auto unit = [&](Blk& x, int t, int hk) {
        const int key_base = t * BN + 32 * hk;
        if (key_base >= N) return;
        const unsigned kt = buf(t);
        x.s = key_base + 32 > N ? key_mask_block(key_base, lane_from_exec() / 32, N) : f32x16_zero();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            x.s = E::mfma(ln.natural(kt, hk, ks), x.qf[ks], x.s);
            x.dp = E::mfma(ln.natural(kt + PairRing::TILE, hk, ks), x.gf[ks], ks == 0 ? f32x16_zero() : x.dp);
        }
        grad(x, 0, 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) x.acc[i % 2] = E::mfma(ln.transposed(kt, i % 2, 2 * hk + i / 2), as_frag8(x.df[i / 2]), x.acc[i % 2]);
    };
    const int nfast = N / BN;
    if (sp.mine == 2) {
        frag8 kf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kf[i] = frag8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            A.s = E::mfma(ln.natural(buf(0), 0, ks), A.qf[ks], ks == 0 ? f32x16_zero() : A.s);
            A.dp = E::mfma(ln.natural(buf(0) + PairRing::TILE, 0, ks), A.gf[ks], ks == 0 ? f32x16_zero() : A.dp);
        }
        frag8 fk = ln.natural(buf(0), 0, 0), fv = ln.natural(buf(0) + PairRing::TILE, 0, 0);
        // one phase: x's vector work beside y's products
        auto phase = [&](auto reload, Blk& x, Blk& y, unsigned kt, int hk, unsigned ktn, int hkn) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                __builtin_amdgcn_sched_barrier(0);
                const frag8 ck = fk, cv = fv;
                fk = ks + 1 < KS ? ln.natural(kt, hk, (ks + 1) % KS) : ln.natural(ktn, hkn, 0);
                fv = ks + 1 < KS ? ln.natural(kt + PairRing::TILE, hk, (ks + 1) % KS) : ln.natural(ktn + PairRing::TILE, hkn, 0);
                y.s = E::mfma(ck, y.qf[ks], ks == 0 ? f32x16_zero() : y.s);
                y.dp = E::mfma(cv, y.gf[ks], ks == 0 ? f32x16_zero() : y.dp);
                y.acc[ks % 2] = E::mfma(kf[ks], as_frag8(y.df[ks / 2]), y.acc[ks % 2]);
                if (decltype(reload)::value) kf[ks] = ln.transposed(kt, ks % 2, 2 * hk + ks / 2);
                grad(x, 4 * ks, 4 * ks + 4);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto step = [&](unsigned kt, int hk, unsigned ktn, int hkn) {
            phase(std::true_type{}, A, B, kt, hk, ktn, hkn);
            phase(std::false_type{}, B, A, ktn, hkn, ktn, hkn);
        };
        for (int t = 0; t < nfast; ++t) {
            ring.fetch(t + 3);
            step(buf(t), 0, buf(t), 1);
            step(buf(t), 1, buf(t + 1), 0);
            PairRing::landed_barrier();
        }
        if (N % BN >= 32) step(buf(nfast), 0, buf(nfast), 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) B.acc[i % 2] = E::mfma(kf[i], as_frag8(B.df[i / 2]), B.acc[i % 2]);
        const int t = N / 64, hk = N / 32 % 2;
        unit(A, t, hk);
        unit(B, t, hk);
    } else {
        for (int t = 0; t < ntiles; ++t) {
            if (t < nfast) ring.fetch(t + 3);
#pragma unroll
            for (int hk = 0; hk < 2; ++hk)
                if (sp.mine == 1 && ((2 * t + hk) & (sp.parts - 1)) == sp.part) unit(A, t, hk);
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

