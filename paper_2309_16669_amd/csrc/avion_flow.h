// dK and dV where the launch leaves compute units with one workgroup (by_flow in avion_attn.hip), 64 channels, no mask: two groups
// of wavefronts.  Same operation, order of sums and bits as avion_dkdv_kernel<64, NW, 2>.
//
// What bounds that kernel there is the latency of one wavefront's unit: two wavefronts per SIMD cannot fill each other's
// waits for LDS and for the last product of a chain.  Here the wavefront's own products stand beside its vector work: while the
// scores of 32 queries become weights, dV and dK of the 32 before them and S and dP of the 32 after them are formed, and every
// operand is requested eight products ahead into the registers that the product eight before it has left.  242 registers, two
// wavefronts per SIMD.  In a loop without tile fetches a unit of the chain takes 832 cycles at two wavefronts per SIMD (1052 at
// one), of this form 676 (859).
// Tiles as in avion_pair.h, four buffers: a barrier in the middle of a tile, when nothing of the tile before is needed any more (the
// columns of its last unit were taken in the first half tile), certifies that the next one has landed and lets the one three ahead
// be fetched.
// Measured, us, avion_dkdv_kernel -> this: 16 heads x 785 13.6 -> 12.0, 8 x 1568 19.8 (four groups) -> 17.4, 6 x 3000 43.4 -> 38.3, 12 x 1568
// 26.0 -> 23.4; on the other side of the lines 36 x 789 17.4 -> 16.8, 61 x 289 9.9 -> 10.1.  Waiting for three tiles instead of one before
// the first unit cost 0.2 to 0.8 us more, the loads of a tile one by one instead of in fours and fives up to 2, walking units past the end (an odd
// tile's worth of zeros, or half of one) 0.1 to 0.9.
// On a full chip, one group, it is no faster than three wavefronts per SIMD of that kernel (avion_pair.h).
#pragma once
#include "avion_pair.h"

// Q, dO and the per-query scalars for one group of NW wavefronts
template <int NW>
struct FlowRing : QuadTiles<NW> {
    using QuadTiles<NW>::PER;
    using QuadTiles<NW>::TILE;
    static constexpr int OFF_SC = 2 * TILE, BUF = OFF_SC + 1024, NBUF = 4, LDS_BYTES = NBUF * BUF;
    static constexpr int LOADS = 2 * PER + 1;
    unsigned vs;
    u32x4 ds;
    DEVINL FlowRing(const raw16* a, long rs_a, const raw16* b, long rs_b, int N, const float* scalars, int npad, const char* smem, int wave_, int lane)
        : QuadTiles<NW>(a, rs_a, b, rs_b, N, smem, wave_, lane)
    {
        ds = RawBuffer(scalars + (wave_ & 1) * npad, npad * 4u).words;
        vs = lane * 4;
    }
    // the loads of one wavefront; rows and scalars past the end arrive as zeros
    DEVINL void fetch(int ti, unsigned buf) const
    {
        const unsigned base = this->smem_addr + buf;
        this->fetch_tiles(ti, base);
        // LSE by even wavefronts, -delta by odd ones, 256 bytes each
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     : : "s"(base + OFF_SC - this->wave * 768), "v"(vs + (unsigned)ti * 256), "s"(ds) : "memory", "m0");
    }
    // all but the newest fetch of this wavefront have landed
    DEVINL static void landed_barrier() { asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"i"(LOADS) : "memory"); }
    DEVINL static void all_landed_barrier() { asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
};

template <int NW, typename E>
__global__ void __launch_bounds__(NW * 128, 2)
avion_dkdv_flow_kernel(const raw16* __restrict__ q, const raw16* __restrict__ k, const raw16* __restrict__ v,
                      const raw16* __restrict__ dO, const float* __restrict__ rowsc, raw16* __restrict__ dk,
                      raw16* __restrict__ dv, int H, int N, int rs_qkv, int rs_o, int nkb, int nblocks, float cs,
                      float scale)
{
    using Ring = FlowRing<NW>;
    constexpr int D = 64, KS = 4, KG = 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int logical = xcd_local_id(blockIdx.x, nblocks);
    if (logical < 0) return;
    const int bh = logical / nkb, kb = logical % nkb;
    const int b = bh / H, h = bh % H;
    const int tid = threadIdx.x, lane = tid % 64, l32 = lane % 32, g = lane / 32;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid / 64), wave = wave_id % NW, grp = wave_id / NW;
    const long rs = rs_qkv;
    const long head_off = (long)b * N * rs + (long)h * D;
    const long head_off_o = (long)b * N * rs_o + (long)h * D;
    const int npad = (N + 63) & ~63, ntiles = npad / 64;
    const int k0 = kb * 32 * NW + wave * 32;  // first key of this wavefront
    // Units of 32 queries of this group, from tile t0 on (at least one: the launch has five tiles or more).  Units that lie wholly past
    // the end, in the last tile or in a tile that only the first group has, are left out, as avion_dkdv_body does: their rows are zeros, but
    // zeros times a key's infinite component are not.
    const int per = (ntiles + KG - 1) / KG, t0 = grp * per, units = min(2 * per, (N + 31) / 32 - 2 * t0);
    char* mine = smem + grp * Ring::LDS_BYTES;
    const Ring ring(q + head_off, rs, dO + head_off_o, rs_o, N, rowsc + (long)bh * 2 * npad, npad, mine, wave, lane);
    QuadLane ln(lane, lds_address(mine));
    ring.fetch(t0, 0);
    // K and V fragments (B operands: lane = key); keys past the end are computed and not stored
    frag8 kf[KS], vf[KS];
    {
        const long off = head_off + (long)min(k0 + l32, N - 1) * rs + g * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kf[ks] = *reinterpret_cast<const frag8*>(k + off + ks * 16);
            vf[ks] = *reinterpret_cast<const frag8*>(v + off + ks * 16);
        }
    }
    f32x16 dka[2], dva[2];
    dka[0] = dka[1] = dva[0] = dva[1] = f32x16_zero();
    hold(kf);
    hold(vf);
    Ring::all_landed_barrier();  // the first tile is in LDS (and the fragments have arrived)
    ring.fetch(t0 + 1, Ring::BUF);
    ring.fetch(t0 + 2, 2 * Ring::BUF);

    typedef const __attribute__((address_space(3))) f32x4* lds_f4;
    unsigned sa = lds_address(mine) + Ring::OFF_SC + g * 16;  // LSE * log2e of this lane group's first queries; -delta 256 bytes on
    auto put4 = [](f32x16& x, int a, f32x4 y) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * a + e] = y[e];
    };
    struct Scores {
        f32x16 s, dp;
    } A, B;  // of even and of odd units
    frag8 f[8];  // operands on their way: rows of the next unit, then columns of this one
    u32x4 pf[2], df[2];
    f32x4 l4[4];
    pf[0] = pf[1] = df[0] = df[1] = u32x4{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        put4(A.dp, i, *(lds_f4)(sa + 256 + i * 32));
        l4[i] = *(lds_f4)(sa + i * 32);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        A.s = E::mfma(ln.natural(0, 0, ks), kf[ks], ks == 0 ? f32x16_zero() : A.s);
        A.dp = E::mfma(ln.natural(Ring::TILE, 0, ks), vf[ks], A.dp);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = frag8{0, 0, 0, 0, 0, 0, 0, 0};
    // exp2 and dS of x beside dV and dK of the unit before; the rows of the unit after (half tile 1 - hk) are requested
    auto first_half = [&](Scores& x, Scores& y, auto hk_) {
        constexpr int hkn = 1 - decltype(hk_)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            const int half = i / 2, ct = i % 2;
            dva[ct] = E::mfma(f[2 * i], as_frag8(pf[half]), dva[ct]);
            f[2 * i] = ln.natural(0, hkn, i);
            dka[ct] = E::mfma(f[2 * i + 1], as_frag8(df[half]), dka[ct]);
            f[2 * i + 1] = ln.natural(Ring::TILE, hkn, i);
            put4(y.dp, i, *(lds_f4)(sa + 256 + hkn * 128 + i * 32));
#pragma unroll
            for (int e = 4 * i; e < 4 * i + 4; ++e) {
                x.s[e] = fast_exp2(fmaf(x.s[e], cs, -l4[i][e % 4]));
                x.dp[e] = x.s[e] * x.dp[e];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // roundings of x beside S and dP of the unit after; the columns of x's unit (half tile hk) are requested
    auto second_half = [&](Scores& x, Scores& y, auto hk_) {
        constexpr int hk = decltype(hk_)::value, hkn = 1 - hk;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            y.s = E::mfma(f[2 * i], kf[i], i == 0 ? f32x16_zero() : y.s);
            f[2 * i] = ln.transposed(Ring::TILE, i % 2, 2 * hk + i / 2);
            y.dp = E::mfma(f[2 * i + 1], vf[i], y.dp);
            f[2 * i + 1] = ln.transposed(0, i % 2, 2 * hk + i / 2);
            l4[i] = *(lds_f4)(sa + hkn * 128 + i * 32);
#pragma unroll
            for (int e = 4 * i; e < 4 * i + 4; e += 2) {
                pf[e / 8][(e / 2) % 4] = E::pack(x.s[e], x.s[e + 1]);
                df[e / 8][(e / 2) % 4] = E::pack(x.dp[e], x.dp[e + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> lo{};
    constexpr std::integral_constant<int, 1> hi{};
    for (int i = 0; i < units / 2; ++i) {
        const int by = (i & 3) == 3 ? -3 * Ring::BUF : Ring::BUF;  // to the next tile's buffer
        first_half(A, B, lo);
        second_half(A, B, lo);
        Ring::landed_barrier();  // tile i + 1 has landed; tile i - 1 is no longer read
        ring.fetch(t0 + i + 3, (i + 3 & 3) * Ring::BUF);
        ln.move_nat(by);
        sa += by;
        asm volatile("" : "+v"(sa));
        first_half(B, A, hi);
        second_half(B, A, hi);
        ln.move_tr(by);
    }
    for (int i = units / 2; i < per; ++i) Ring::landed_barrier();  // every wavefront passes the same barriers
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        dva[i % 2] = E::mfma(f[2 * i], as_frag8(pf[i / 2]), dva[i % 2]);
        dka[i % 2] = E::mfma(f[2 * i + 1], as_frag8(df[i / 2]), dka[i % 2]);
    }
    if (units & 1) {  // half a tile: its scores are in A
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const float p0 = fast_exp2(fmaf(A.s[e], cs, -l4[e / 4][e % 4])), p1 = fast_exp2(fmaf(A.s[e + 1], cs, -l4[e / 4][e % 4 + 1]));
            pf[e / 8][(e / 2) % 4] = E::pack(p0, p1);
            df[e / 8][(e / 2) % 4] = E::pack(p0 * A.dp[e], p1 * A.dp[e + 1]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dva[i % 2] = E::mfma(ln.transposed(Ring::TILE, i % 2, i / 2), as_frag8(pf[i / 2]), dva[i % 2]);
            dka[i % 2] = E::mfma(ln.transposed(0, i % 2, i / 2), as_frag8(df[i / 2]), dka[i % 2]);
        }
    }
    Ring::all_landed_barrier();  // no load is on its way, no tile is read any more
    const bool wave_active = k0 < N;
    const int lane_now = lane_from_exec();
    char* area = smem + NW * RowStore<D, E>::BYTES;
    static_assert(NW * RowStore<D, E>::BYTES + NW * 8192 <= KG * Ring::LDS_BYTES, "exchange area");
    add_groups<NW, KG>(area, dka, grp, wave, lane_now, wave_active);
    __syncthreads();
    add_groups<NW, KG>(area, dva, grp, wave, lane_now, wave_active);
    if (grp > 0 || !wave_active) return;
    char* region = smem + wave * RowStore<D, E>::BYTES;
    RowStore<D, E>::run(region, dka, scale, dk + head_off + (long)k0 * rs, rs, N - k0, lane_now);
    RowStore<D, E>::run(region, dva, 1.0f, dv + head_off + (long)k0 * rs, rs, N - k0, lane_now);
}
