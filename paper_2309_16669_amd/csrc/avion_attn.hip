// C ABI of the gfx950 attention library: argument checks, kernel-instance selection, launches.
// See include/avion_attn.h for the contract of every entry point.
#include "avion_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <atomic>
#include <cstring>
#include <mutex>

#include "avion_bwd.h"
#include "avion_flow.h"
#include "avion_fwd.h"
#include "avion_head.h"
#include "avion_ln.h"
#include "avion_pair.h"
#include "avion_small.h"
#include "avion_gelu.h"

// Built-in scratch of avion_attn_bwd_noalloc: the per-query scalars that the backward's two passes
// hand to each other live here instead of in a caller's workspace.  One copy per GPU, held until
// the process ends.  In host code this name is only a handle for hipGetSymbolAddress; kernels get
// the device address that call returns.
constexpr size_t kScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

thread_local char g_hip_error[256] = "";

int hip_fail(hipError_t e, const char* what)
{
    std::snprintf(g_hip_error, sizeof g_hip_error, "%s: %s", what, hipGetErrorString(e));
    return AVION_EHIP;
}

// Device address of `scratch` on each GPU, looked up once per device with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return AVION_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return AVION_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Token strides (elements between consecutive tokens of one head) of the two tensor groups.
struct Strides {
    int qkv;  // Q, K, V and their gradients: H*d, or 3*H*d when they are packed in one tensor
    int o;    // O and dO: H*d
};

// Which kernel family an entry point runs: element format and masking.
struct Variant {
    bool f16;
    bool causal;
};

constexpr long long kComputeUnits = 256;

constexpr float kMinScale = 8.673617379884035e-19f;  // 2^-60

int check_shape(int B, int H, int N, int d, float scale, int packed = 1)
{
    if (B < 1 || H < 1 || N < 1) return AVION_EINVAL;
    // Keys past the end of a ragged tile (and keys a causal query must not see) are removed by a
    // score of -1e30 that is then multiplied by scale*log2(e); the product has to stay far below any
    // real score for the weight to come out as exactly 0, hence the floor of 2^-60 on scale.
    if (!(scale >= kMinScale) || !std::isfinite(scale)) return AVION_EINVAL;
    if (d != 64 && d != 80) return AVION_EUNSUPPORTED;
    if (N > (1 << 24) || (long long)B * H > (1 << 24)) return AVION_EUNSUPPORTED;
    // one (batch, head) slice is addressed with 32-bit byte offsets (buffer loads), and tile loads
    // may start up to four 64-row tiles past the end of the sequence
    if (((long long)N + 256) * packed * H * d * 2 >= (1LL << 31)) return AVION_EUNSUPPORTED;
    return AVION_OK;
}

// Workgroups are launched in multiples of 8 (one per XCD); the padding ones exit at once.
bool grid_for(long long nblocks, unsigned* grid)
{
    const long long padded = ((nblocks + 7) / 8) * 8;
    if (padded > 0x7fffffffLL) return false;
    *grid = (unsigned)padded;
    return true;
}

// Raises the kernel's dynamic LDS limit once; `done` is the caller's per-instance flag.  A failure
// is not remembered, so the next call tries again.
template <typename K>
hipError_t allow_lds(K kernel, int bytes, std::atomic<bool>& done)
{
    if (done.load(std::memory_order_acquire)) return hipSuccess;
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.store(true, std::memory_order_release);
    return e;
}

// Result of the launch just made on this thread.  Errors left behind by earlier, unrelated work of
// the caller are cleared before the launch (begin_launch) so that they are not mistaken for it.
void begin_launch() { (void)hipGetLastError(); }
int end_launch(const char* what)
{
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? AVION_OK : hip_fail(e, what);
}

template <int D, int NW, int KG, typename E, bool CAUSAL>
int launch_fwd(const raw16* q, const raw16* k, const raw16* v, raw16* o, float* lse, int B, int H, int N, Strides rs,
               float scale, hipStream_t st)
{
    using Cfg = FwdCfg<D, NW, KG>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_fwd_kernel<D, NW, KG, E, CAUSAL>, Cfg::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(fwd)");
    const int nqb = (N + Cfg::BM - 1) / Cfg::BM;
    const long long nblocks = (long long)nqb * B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_fwd_kernel<D, NW, KG, E, CAUSAL>), dim3(grid), dim3(Cfg::NT), Cfg::LDS_BYTES, st, q, k, v, o, lse, H, N, rs.qkv,
                       rs.o, nqb, (int)nblocks, scale * kLog2e);
    return end_launch("launch avion_fwd_kernel");
}

template <int D, int NW, int KG, typename E, bool CAUSAL, bool TILE16>
int launch_dq(const raw16* q, const raw16* k, const raw16* v, const raw16* o, const raw16* dO, const float* lse, raw16* dq,
              float* rowsc, int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    using Cfg = DqCfg<D, NW, KG>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_dq_kernel<D, NW, KG, E, CAUSAL, TILE16>, Cfg::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(dq)");
    const int nqb = (N + Cfg::BM - 1) / Cfg::BM;
    const long long nblocks = (long long)nqb * B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_dq_kernel<D, NW, KG, E, CAUSAL, TILE16>), dim3(grid), dim3(Cfg::NT), Cfg::LDS_BYTES, st, q, k, v, o, dO, lse, dq,
                       rowsc, H, N, rs.qkv, rs.o, nqb, (int)nblocks, scale * kLog2e, scale);
    return end_launch("launch avion_dq_kernel");
}

template <typename E>
int launch_dq_pair(const raw16* q, const raw16* k, const raw16* v, const raw16* o, const raw16* dO, const float* lse, raw16* dq,
                   float* rowsc, int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_dq_pair_kernel<E>, PairRing::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(dq_pair)");
    const int nqb = ((N + 31) / 32 + kPairBlocks - 1) / kPairBlocks;
    const long long nblocks = (long long)nqb * B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_dq_pair_kernel<E>), dim3(grid), dim3(256), PairRing::LDS_BYTES, st, q, k, v, o, dO, lse, dq,
                       rowsc, H, N, rs.qkv, rs.o, nqb, (int)nblocks, scale * kLog2e, scale);
    return end_launch("launch avion_dq_pair_kernel");
}

template <int D, int NW, int KG, typename E, bool CAUSAL>
int launch_dkdv(const raw16* q, const raw16* k, const raw16* v, const raw16* dO, const float* rowsc, raw16* dk, raw16* dv,
                int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    using Cfg = DkvCfg<D, NW, KG>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_dkdv_kernel<D, NW, KG, E, CAUSAL>, Cfg::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(dkdv)");
    const int nkb = (N + Cfg::BNK - 1) / Cfg::BNK;
    const long long nblocks = (long long)nkb * B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_dkdv_kernel<D, NW, KG, E, CAUSAL>), dim3(grid), dim3(Cfg::NT), Cfg::LDS_BYTES, st, q, k, v, dO, rowsc, dk,
                       dv, H, N, rs.qkv, rs.o, nkb, (int)nblocks, scale * kLog2e, scale);
    return end_launch("launch avion_dkdv_kernel");
}

template <int NW, typename E>
int launch_dkdv_flow(const raw16* q, const raw16* k, const raw16* v, const raw16* dO, const float* rowsc, raw16* dk, raw16* dv,
                     int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    constexpr int LDS_BYTES = 2 * FlowRing<NW>::LDS_BYTES;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_dkdv_flow_kernel<NW, E>, LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(dkdv_flow)");
    const int nkb = (N + 32 * NW - 1) / (32 * NW);
    const long long nblocks = (long long)nkb * B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_dkdv_flow_kernel<NW, E>), dim3(grid), dim3(NW * 128), LDS_BYTES, st, q, k, v, dO, rowsc, dk, dv, H, N, rs.qkv,
                       rs.o, nkb, (int)nblocks, scale * kLog2e, scale);
    return end_launch("launch avion_dkdv_flow_kernel");
}

template <int D, int NW, typename E, bool CAUSAL>
int launch_bwd_small(const raw16* q, const raw16* k, const raw16* v, const raw16* o, const raw16* dO, const float* lse,
                     raw16* dq, raw16* dk, raw16* dv, float* rowsc, int B, int H, int N, Strides rs, float scale,
                     hipStream_t st)
{
    using Cfg = BwdSmallCfg<D, NW>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_bwd_small_kernel<D, NW, E, CAUSAL>, Cfg::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(bwd_small)");
    const long long nblocks = (long long)B * H;
    unsigned grid;
    if (!grid_for(nblocks, &grid)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_bwd_small_kernel<D, NW, E, CAUSAL>), dim3(grid), dim3(Cfg::NT), Cfg::LDS_BYTES, st, q, k, v, o,
                       dO, lse, dq, dk, dv, rowsc, H, N, rs.qkv, rs.o, (int)nblocks, scale * kLog2e, scale);
    return end_launch("launch avion_bwd_small_kernel");
}

// Whole backward, one workgroup per head at a time (avion_head.h).
template <int NW, int NB, typename E, bool CAUSAL>
int launch_bwd_head(const raw16* q, const raw16* k, const raw16* v, const raw16* o, const raw16* dO, const float* lse,
                    raw16* dq, raw16* dk, raw16* dv, int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    using Cfg = HeadCfg<NW, NB>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_bwd_head_kernel<NW, NB, E, CAUSAL>, Cfg::LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(bwd_head)");
    const int heads = B * H;
    unsigned grid;
    if (!grid_for(heads, &grid)) return AVION_EUNSUPPORTED;
    if (Cfg::WALK) grid = (unsigned)std::min<long long>(heads, kComputeUnits);  // workgroups walk the heads
    begin_launch();
    hipLaunchKernelGGL((avion_bwd_head_kernel<NW, NB, E, CAUSAL>), dim3(grid), dim3(Cfg::NT), Cfg::LDS_BYTES, st, q, k, v, o,
                       dO, lse, dq, dk, dv, H, N, rs.qkv, rs.o, heads, scale * kLog2e, scale);
    return end_launch("launch avion_bwd_head_kernel");
}

// Sequences of at most 32 tokens: one wavefront per window of floor(32 / N) problems (avion_small.h).
constexpr int kWindowMaxN = 32;
struct WindowGrid {
    int G, nitems;
    unsigned grid;
};
template <int D>
bool window_grid(int B, int H, int N, WindowGrid* w)
{
    w->G = 32 / N;
    const long long nwin = ((long long)B + w->G - 1) / w->G, nitems = nwin * H;
    if (nitems > 0x7fffffffLL) return false;
    w->nitems = (int)nitems;
    const long long wgs = (nitems + WinCfg<D>::NW - 1) / WinCfg<D>::NW;
    w->grid = (unsigned)(wgs < 256 * 16 ? wgs : 256 * 16);  // wavefronts walk the windows with a stride
    return true;
}

template <int D, typename E, bool CAUSAL>
int launch_win_fwd(const raw16* q, const raw16* k, const raw16* v, raw16* o, float* lse, int B, int H, int N, Strides rs,
                   float scale, hipStream_t st)
{
    using Cfg = WinCfg<D>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_win_fwd_kernel<D, E, CAUSAL>, Cfg::FWD_LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(win_fwd)");
    WindowGrid w;
    if (!window_grid<D>(B, H, N, &w)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_win_fwd_kernel<D, E, CAUSAL>), dim3(w.grid), dim3(Cfg::NT), Cfg::FWD_LDS_BYTES, st, q, k, v, o,
                       lse, B, H, N, rs.qkv, rs.o, w.G, w.nitems, scale * kLog2e);
    return end_launch("launch avion_win_fwd_kernel");
}

template <int D, typename E, bool CAUSAL>
int launch_win_bwd(const raw16* q, const raw16* k, const raw16* v, const raw16* o, const raw16* dO, const float* lse,
                   raw16* dq, raw16* dk, raw16* dv, int B, int H, int N, Strides rs, float scale, hipStream_t st)
{
    using Cfg = WinCfg<D>;
    static std::atomic<bool> lds_allowed{false};
    const hipError_t attr = allow_lds(avion_win_bwd_kernel<D, E, CAUSAL>, Cfg::BWD_LDS_BYTES, lds_allowed);
    if (attr != hipSuccess) return hip_fail(attr, "hipFuncSetAttribute(win_bwd)");
    WindowGrid w;
    if (!window_grid<D>(B, H, N, &w)) return AVION_EUNSUPPORTED;
    begin_launch();
    hipLaunchKernelGGL((avion_win_bwd_kernel<D, E, CAUSAL>), dim3(w.grid), dim3(Cfg::NT), Cfg::BWD_LDS_BYTES, st, q, k, v, o,
                       dO, lse, dq, dk, dv, B, H, N, rs.qkv, rs.o, w.G, w.nitems, scale * kLog2e, scale);
    return end_launch("launch avion_win_bwd_kernel");
}

// Kernel instances by head size, format and masking (wavefronts per workgroup: fwd_cut, bwd_cut and head_impl below).
// by_variant calls f(head dim, element format, causal) with the three as compile-time tags, by_format
// f(element format, causal).
template <typename T>
struct TypeTag {
    using type = T;
};
template <typename F>
int by_format(Variant var, F f)
{
    auto by_mask = [&](auto fmt) {
        if (var.causal) return f(fmt, std::true_type{});
        return f(fmt, std::false_type{});
    };
    if (var.f16) return by_mask(TypeTag<F16>{});
    return by_mask(TypeTag<Bf16>{});
}
template <typename F>
int by_variant(Variant var, int d, F f)
{
    return by_format(var, [&](auto fmt, auto causal) {
        if (d == 64) return f(std::integral_constant<int, 64>{}, fmt, causal);
        return f(std::integral_constant<int, 80>{}, fmt, causal);
    });
}

// How one launch of the big kernels is cut.  A workgroup owns 32 * nw rows of the stationary side; with kg > 1 it has kg
// groups of nw wavefronts, each of which walks its own share of the streamed tiles.  One group of 128 rows is the full
// chip's cut: three to four workgroups per compute unit fill each other's waits.  Smaller launches leave compute units
// with one workgroup, a wavefront per SIMD, and a 32 x 32 unit then takes 560 ns of it instead of 333 (460 with two); shorter
// blocks fill more of the chip, groups shorten each wavefront's walk, and both cost an exchange or more tile traffic.
// The lines stand where both sides' times crossed over 2044 shapes of 6..400 heads x 257..3600 tokens (964 causal, 921 at 80 channels).
// Measured, us, one group of 128 rows -> this rule (forward; whole backward): 12 heads x 1568 30.4 -> 17.5; 65 -> 49,
// 32 x 785 16.9 -> 12.9; 39 -> 33, 8 x 1568 17.3 (two groups) -> 16.0; 41.6 -> 38.9, 6 x 3000 29.6 -> 26.0; 84 -> 75.
struct Cut {
    int nw, kg;
};
struct Fill {  // workgroups of 64, 96 and 128 rows of a launch, and its 64-row tiles
    long long w64, w96, w128;
    int tiles;
    Fill(long long heads, int N) : w64(heads * ((N + 63) / 64)), w96(heads * ((N + 95) / 96)), w128(heads * ((N + 127) / 128)), tiles((N + 63) / 64) {}
};
Cut fwd_cut(const Fill& f, int d, bool causal)
{
    const int t = f.tiles;
    // four groups: at 64 channels (LDS holds two at 80), where each still has a walk (64 rows: at 8 tiles they lose 3 % to two, at 13
    // they are equal; 96 rows: 13 tiles equal, 9 tiles 11.1 -> 11.5 us)
    if (t >= 2 && f.w64 <= kComputeUnits) return {2, d == 64 && t >= 11 ? 4 : 2};
    if (d == 80) return t >= 6 && f.w128 <= kComputeUnits ? Cut{4, 2} : Cut{4, 1};
    // 96 rows, two groups -> 128 rows, two groups: 48 x 400 8.9 -> 9.3 us; four groups: 12 x 1568 17.5 -> 19.3
    if (t >= 6 && f.w96 <= kComputeUnits) return {3, t >= 16 ? 4 : 2};
    if (t >= 6 && f.w128 <= kComputeUnits) return {4, t >= 16 ? 4 : 2};
    // Up to two workgroups of 96 rows per compute unit: two groups each, three wavefronts per SIMD instead of one or two.  24 x 1568 32.4 ->
    // 29.4 us, 16 x 2400 46.5 -> 40.9, 12 x 3136 59.5 -> 52.1, 40 x 785 18.9 -> 18.1; 0.93 of the time in the mean of 189 shapes, 1.03 at most; at 300 to
    // 350 tokens up to 1.08.  (Beyond it and up to two of 128 rows, 128 rows in two groups measured 0.97 in the mean; that line is not drawn
    // yet, and one group stays there.)
    if (!causal && t >= 7 && f.w96 <= 2 * kComputeUnits) return {3, 2};
    // causal blocks are of unequal length, which shorter ones even out: 0.80 of the time up to 560 workgroups of 64 rows (30 shapes,
    // none slower), 1.05 and more from 600 on; two groups of 128 rows up to 512 0.93 (153 shapes, 1.04 at most)
    if (causal && t >= 10 && f.w64 <= 560) return {2, 2};
    if (causal && t >= 8 && f.w128 <= 2 * kComputeUnits) return {4, 2};
    return {4, 1};
}
// The backward's two kernels.  Registers allow two groups of 96 and 128 rows, four of 64 at 64 channels.  Where the whole backward
// is one launch, up to 256 tokens at 64 channels and 128 at 80, its two phases keep one group, whose bits it gives.
Cut bwd_cut(const Fill& f, int d, bool causal)
{
    const int t = f.tiles;
    if (t >= (d == 64 ? 5 : 3) && f.w64 <= kComputeUnits) return {2, d == 64 && t >= 15 ? 4 : 2};  // (four: 11 tiles equal, 13 2.5 % slower)
    // 96 rows -> 128: dQ 40 x 400 10.6 -> 11.5 us, 24 x 785 15.2 -> 16.0, 12 x 1568 23.7 -> 24.6; dK/dV 11.3 -> 11.9, 16.4 -> 16.8, 26.0 -> 26.2; whole
    // backward at 80 channels 0.98 of the time, causal 0.96
    if (t >= 5 && f.w96 <= kComputeUnits) return {3, 2};
    // (beyond it two groups lose: 24 x 1568 85 -> 99 us, 64 x 785 53 -> 60)
    if (t >= 6 && f.w128 <= kComputeUnits) return {4, 2};
    // causal: 0.83 of the time up to 600 workgroups of 64 rows (46 shapes, none slower by 3 %), up to 1.12 at 640
    if (causal && d == 64 && t >= 8 && f.w64 <= 600) return {2, 2};
    return {4, 1};
}
// calls f(nw, kg) with the cut's two numbers as compile-time tags; f builds what these lists hold
template <typename F>
int by_cut(Cut c, F f)
{
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 3> three{};
    constexpr std::integral_constant<int, 4> four{};
    switch (8 * c.nw + c.kg) {
        case 8 * 2 + 2: return f(two, two);
        case 8 * 2 + 4: return f(two, four);
        case 8 * 3 + 2: return f(three, two);
        case 8 * 3 + 4: return f(three, four);
        case 8 * 4 + 2: return f(four, two);
        case 8 * 4 + 4: return f(four, four);
        default: return f(four, one);
    }
}

int fwd_impl(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d, int packed,
             Variant var, float scale, void* stream)
{
    if (!q || !k || !v || !o || !lse) return AVION_EINVAL;
    const int rc = check_shape(B, H, N, d, scale, packed);
    if (rc != AVION_OK) return rc;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(lse)) return AVION_EUNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Strides rs{packed * H * d, H * d};
    const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v);
    raw16* oo = static_cast<raw16*>(o);
    if (N <= kWindowMaxN)
        return by_variant(var, d, [&](auto dim, auto fmt, auto causal) {
            return launch_win_fwd<decltype(dim)::value, typename decltype(fmt)::type, decltype(causal)::value>(
                qq, kk, vv, oo, lse, B, H, N, rs, scale, st);
        });
    return by_cut(fwd_cut(Fill((long long)B * H, N), d, var.causal), [&](auto nw, auto kg) {
        return by_variant(var, d, [&](auto dim, auto fmt, auto causal) {
            constexpr int D = decltype(dim)::value, NW = decltype(nw)::value, KG = decltype(kg)::value;
            if constexpr (D == 64 || (NW != 3 && KG <= 2))
                return launch_fwd<D, NW, KG, typename decltype(fmt)::type, decltype(causal)::value>(qq, kk, vv, oo, lse, B, H, N, rs, scale, st);
            else return AVION_EUNSUPPORTED;  // not a cut that fwd_cut gives
        });
    });
}

bool workspace_ok(const void* workspace, size_t workspace_bytes, int B, int H, int N, int d)
{
    return workspace && (reinterpret_cast<uintptr_t>(workspace) & 255u) == 0 &&
           workspace_bytes >= avion_attn_bwd_workspace_bytes(B, H, N, d);
}

// Whole heads per workgroup (avion_head.h): what its LDS holds at 64 channels (at 80 three tiles of 256 rows
// take 160 KB), above the window kernels' lengths, whatever the number of heads.  Both sides' times stand there.
constexpr int kHeadMaxN = 256;
bool by_head(int N, int d) { return d == 64 && N > kWindowMaxN && N <= kHeadMaxN; }

int head_impl(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
              void* dk, void* dv, int B, int H, int N, int packed, Variant var, float scale, void* stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Strides rs{packed * H * 64, H * 64};
    const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v),
                *oo = static_cast<const raw16*>(o), *gg = static_cast<const raw16*>(dO);
    raw16 *dqq = static_cast<raw16*>(dq), *dkk = static_cast<raw16*>(dk), *dvv = static_cast<raw16*>(dv);
    return by_format(var, [&](auto fmt, auto causal) {
        using E = typename decltype(fmt)::type;
        constexpr bool C = decltype(causal)::value;
        auto run = [&](auto nw, auto nb) {
            return launch_bwd_head<decltype(nw)::value, decltype(nb)::value, E, C>(qq, kk, vv, oo, gg, lse, dqq, dkk, dvv, B, H, N, rs, scale, st);
        };
        constexpr std::integral_constant<int, 4> w4{};
        constexpr std::integral_constant<int, 8> w8{};
        switch ((N + 31) / 32) {
            case 2: return run(w4, std::integral_constant<int, 2>{});
            case 3: return run(w4, std::integral_constant<int, 3>{});
            case 4: return run(w4, std::integral_constant<int, 4>{});
            case 5: return run(w8, std::integral_constant<int, 5>{});
            case 6: return run(w8, std::integral_constant<int, 6>{});
            case 7: return run(w8, std::integral_constant<int, 7>{});
            default: return run(w8, std::integral_constant<int, 8>{});
        }
    });
}

// whether bwd_cut gives this cut
template <int D, int NW, int KG>
constexpr bool kBwdCut = KG <= 2 || (D == 64 && NW == 2);

// dQ in two blocks of queries per wavefront (avion_pair.h), for launches beyond one workgroup of 128 rows per compute unit.  Its
// workgroups take 256 rows, and a compute unit does one in the time of 1.75 of avion_dq_kernel's 128-row ones, whether it has
// one at a time or two; both launches end with the unit that has most.  So it is taken where its share of workgroups per unit, rounded
// up, is at most 7/12 of the other kernel's.  Time over avion_dq_kernel's by the two shares (131 shapes, repeated launches in a graph): 1 of 2
// 0.89 (0.96 at most), 2 of 4 0.85 (0.93), 3 of 6 0.88 (0.98), 4 of 7 0.94, 5 of 9 0.93, 6 of 11 0.92, 7 of 12 0.96 (0.98), more 0.87 to 0.96; on
// the other side (single launches) 2 of 2 1.43, 2 of 3 1.10, 3 of 4 1.17, 3 of 5 1.03, 5 of 8 1.00, 6 of 10 0.98, 7 of 11 1.03.  A head's short last
// workgroup counts as one.  Us: 32 x 3136 152.8 -> 121.5, 64 x 1568 81.4 -> 67.8, 24 x 1568 40.5 -> 36.3, 80 x 1200 66.2 -> 56.1, 384 x 1568
// 400 -> 363, 192 x 784 65.0 -> 60.0 (67.6 -> 67.1 between the other kernels of an encoder layer, whose caches are cold and rows packed).
// Below 500 tokens (700 from five shares on) its longer prologue takes what it gives: at 400 0.97 to 1.04 of the time, at 500 to 700 and six
// shares 1.00.
bool by_pair(long long heads, int N, int d, Variant var)
{
    const long long wgs = heads * ((N + 127) / 128), pair_wgs = heads * (((N + 31) / 32 + kPairBlocks - 1) / kPairBlocks);
    if (d != 64 || var.causal || wgs <= kComputeUnits) return false;
    const long long share = (wgs + kComputeUnits - 1) / kComputeUnits, pair_share = (pair_wgs + kComputeUnits - 1) / kComputeUnits;
    return N >= (share <= 4 ? 500 : 700) && 12 * pair_share <= 7 * share;
}

int dq_impl(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq, int B,
            int H, int N, int d, int packed, Variant var, float scale, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!q || !k || !v || !o || !lse || !dO || !dq) return AVION_EINVAL;
    const int rc = check_shape(B, H, N, d, scale, packed);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {q, k, v, o, lse, dO, dq};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    if (!workspace_ok(workspace, workspace_bytes, B, H, N, d)) return AVION_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Strides rs{packed * H * d, H * d};
    float* rowsc = static_cast<float*>(workspace);  // receives LSE*log2e and -delta for the second pass
    const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v),
               *oo = static_cast<const raw16*>(o), *gg = static_cast<const raw16*>(dO);
    raw16* dqq = static_cast<raw16*>(dq);
    // the lengths of the head kernel: avion_attn_bwd_dq alone comes here with them, and only its form is built
    if (by_head(N, d) && (var.f16 || var.causal)) return AVION_EUNSUPPORTED;
    if (by_head(N, d)) return launch_dq<64, 4, 1, Bf16, false, true>(qq, kk, vv, oo, gg, lse, dqq, rowsc, B, H, N, rs, scale, st);
    if (by_pair((long long)B * H, N, d, var)) {
        if (var.f16) return launch_dq_pair<F16>(qq, kk, vv, oo, gg, lse, dqq, rowsc, B, H, N, rs, scale, st);
        return launch_dq_pair<Bf16>(qq, kk, vv, oo, gg, lse, dqq, rowsc, B, H, N, rs, scale, st);
    }
    return by_cut(bwd_cut(Fill((long long)B * H, N), d, var.causal), [&](auto nw, auto kg) {
        return by_variant(var, d, [&](auto dim, auto fmt, auto causal) {
            constexpr int D = decltype(dim)::value, NW = decltype(nw)::value, KG = decltype(kg)::value;
            if constexpr (kBwdCut<D, NW, KG>)
                return launch_dq<D, NW, KG, typename decltype(fmt)::type, decltype(causal)::value, D == 80>(
                    qq, kk, vv, oo, gg, lse, dqq, rowsc, B, H, N, rs, scale, st);
            else return AVION_EUNSUPPORTED;
        });
    });
}

// dK and dV by the pipelined kernel (avion_flow.h): always two groups.  Its time over avion_dkdv_kernel's in the same cut (94 shapes, launches
// in a graph): 64 rows 0.96 at 5 tiles, 0.91 at 9, 0.89 at 14 (two groups there), 0.89 to 0.92 from 15 to 45 (four); 96 rows 1.03 at 5 and 6, 1.00 at
// 7, 0.98 to 1.01 at 8, 0.97 at 9, 0.95 at 12, 0.92 at 45; 128 rows 0.99 at 6 to 8, 0.97 at 12 to 16, 0.95 at 45.  The lines at 8 and 15 tiles were
// drawn when it still walked units past the end (128 rows then 1.03 at 6 to 8 tiles, 0.99 at 12 to 14).
bool by_flow(Cut c, const Fill& f, int d, Variant var)
{
    return d == 64 && !var.causal && c.kg > 1 && f.tiles >= (c.nw == 2 ? 0 : c.nw == 3 ? 8 : 15);
}

int dkdv_impl(const void* q, const void* k, const void* v, const float* lse, const void* dO, void* dk, void* dv, int B,
              int H, int N, int d, int packed, Variant var, float scale, const void* workspace, size_t workspace_bytes,
              void* stream)
{
    if (!q || !k || !v || !lse || !dO || !dk || !dv) return AVION_EINVAL;
    const int rc = check_shape(B, H, N, d, scale, packed);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {q, k, v, lse, dO, dk, dv};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    if (!workspace_ok(workspace, workspace_bytes, B, H, N, d)) return AVION_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Strides rs{packed * H * d, H * d};
    const float* rowsc = static_cast<const float*>(workspace);  // LSE*log2e and -delta, left by the dQ pass
    const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v),
               *gg = static_cast<const raw16*>(dO);
    raw16 *dkk = static_cast<raw16*>(dk), *dvv = static_cast<raw16*>(dv);
    const Fill fill((long long)B * H, N);
    const Cut cut = bwd_cut(fill, d, var.causal);
    if (by_flow(cut, fill, d, var)) {
        auto flow = [&](auto nw) {
            constexpr int NW = decltype(nw)::value;
            if (var.f16) return launch_dkdv_flow<NW, F16>(qq, kk, vv, gg, rowsc, dkk, dvv, B, H, N, rs, scale, st);
            return launch_dkdv_flow<NW, Bf16>(qq, kk, vv, gg, rowsc, dkk, dvv, B, H, N, rs, scale, st);
        };
        if (cut.nw == 2) return flow(std::integral_constant<int, 2>{});
        if (cut.nw == 3) return flow(std::integral_constant<int, 3>{});
        return flow(std::integral_constant<int, 4>{});
    }
    return by_cut(cut, [&](auto nw, auto kg) {
        return by_variant(var, d, [&](auto dim, auto fmt, auto causal) {
            constexpr int D = decltype(dim)::value, NW = decltype(nw)::value, KG = decltype(kg)::value;
            if constexpr (kBwdCut<D, NW, KG> && (D != 64 || NW != 2 || decltype(causal)::value))
                return launch_dkdv<D, NW, KG, typename decltype(fmt)::type, decltype(causal)::value>(qq, kk, vv, gg, rowsc, dkk, dvv, B, H,
                                                                                                     N, rs, scale, st);
            else return AVION_EUNSUPPORTED;
        });
    });
}

// Whole backward in one launch of both passes (d = 80, N <= 128); arguments already checked by the caller.
int bwd_small_impl(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
                   void* dk, void* dv, int B, int H, int N, int packed, Variant var, float scale, void* workspace,
                   void* stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Strides rs{packed * H * 80, H * 80};
    float* rowsc = static_cast<float*>(workspace);
    const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v),
                *oo = static_cast<const raw16*>(o), *gg = static_cast<const raw16*>(dO);
    raw16 *dqq = static_cast<raw16*>(dq), *dkk = static_cast<raw16*>(dk), *dvv = static_cast<raw16*>(dv);
    return by_format(var, [&](auto fmt, auto causal) {
        return launch_bwd_small<80, 4, typename decltype(fmt)::type, decltype(causal)::value>(
            qq, kk, vv, oo, gg, lse, dqq, dkk, dvv, rowsc, B, H, N, rs, scale, st);
    });
}

int bwd_impl(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
             void* dk, void* dv, int B, int H, int N, int d, int packed, Variant var, float scale, void* workspace,
             size_t workspace_bytes, void* stream)
{
    // every argument is checked before the first launch, so an error leaves all outputs untouched
    if (!q || !k || !v || !o || !lse || !dO || !dq || !dk || !dv) return AVION_EINVAL;
    const int rc = check_shape(B, H, N, d, scale, packed);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {q, k, v, o, lse, dO, dq, dk, dv};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    if (!workspace_ok(workspace, workspace_bytes, B, H, N, d)) return AVION_EWORKSPACE;
    if (N <= kWindowMaxN) {
        // one wavefront per window of problems; needs no workspace (it is still checked, as for every shape)
        hipStream_t st = static_cast<hipStream_t>(stream);
        const Strides rs{packed * H * d, H * d};
        const raw16 *qq = static_cast<const raw16*>(q), *kk = static_cast<const raw16*>(k), *vv = static_cast<const raw16*>(v),
                    *oo = static_cast<const raw16*>(o), *gg = static_cast<const raw16*>(dO);
        raw16 *dqq = static_cast<raw16*>(dq), *dkk = static_cast<raw16*>(dk), *dvv = static_cast<raw16*>(dv);
        return by_variant(var, d, [&](auto dim, auto fmt, auto causal) {
            return launch_win_bwd<decltype(dim)::value, typename decltype(fmt)::type, decltype(causal)::value>(
                qq, kk, vv, oo, gg, lse, dqq, dkk, dvv, B, H, N, rs, scale, st);
        });
    }
    if (by_head(N, d))
        return head_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, packed, var, scale, stream);
    if (N <= BwdSmallCfg<80, 4>::MAX_N)
        return bwd_small_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, packed, var, scale, workspace, stream);
    const int rq = dq_impl(q, k, v, o, lse, dO, dq, B, H, N, d, packed, var, scale, workspace, workspace_bytes, stream);
    if (rq != AVION_OK) return rq;
    return dkdv_impl(q, k, v, lse, dO, dk, dv, B, H, N, d, packed, var, scale, workspace, workspace_bytes, stream);
}

// ------------------------------------------------------------------------------ layer normalisation
int ln_check(long long M, int D, unsigned flags)
{
    if (M < 1 || D < 1) return AVION_EINVAL;
    if (flags & ~AVION_FLAG_F16) return AVION_EINVAL;
    if (D % 8 != 0 || D > 64 * 8 * kLnMaxChunks) return AVION_EUNSUPPORTED;
    if (M > (1LL << 40)) return AVION_EUNSUPPORTED;
    return AVION_OK;
}
unsigned ln_grid(long long M)
{
    const long long wgs = (M + kLnWaves - 1) / kLnWaves;
    return (unsigned)(wgs < kLnMaxGrid ? wgs : kLnMaxGrid);
}
// calls f(chunks per lane, element format) with both as compile-time tags
template <typename F>
int ln_dispatch(int D, bool f16, F f)
{
    const int per_lane = (D / 8 + 63) / 64;
    auto by_fmt = [&](auto nch) {
        if (f16) return f(nch, TypeTag<F16>{});
        return f(nch, TypeTag<Bf16>{});
    };
    if (per_lane <= 1) return by_fmt(std::integral_constant<int, 1>{});
    if (per_lane <= 2) return by_fmt(std::integral_constant<int, 2>{});
    return by_fmt(std::integral_constant<int, 4>{});
}

// ------------------------------------------------------------------------------------ bias + GELU
constexpr int kGeluMaxF = 1 << 16;
int gelu_check(long long M, int F, unsigned flags)
{
    if (M < 1 || F < 1) return AVION_EINVAL;
    if (flags & ~AVION_FLAG_F16) return AVION_EINVAL;
    if (F % 8 != 0 || F > kGeluMaxF) return AVION_EUNSUPPORTED;
    if (M > (1LL << 40)) return AVION_EUNSUPPORTED;
    return AVION_OK;
}
// column blocks of 1024 columns, and row groups so that the launch has at most kGeluMaxGrid workgroups
struct GeluGrid {
    int ncb, nrg;
};
// tensors beyond half of the 256 MB last-level cache are streamed past it
bool gelu_streams(long long M, int F) { return M * F * 2 > (128LL << 20); }
GeluGrid gelu_grid(long long M, int F)
{
    GeluGrid g;
    g.ncb = (F / 8 + kGeluThreads - 1) / kGeluThreads;
    const long long most = kGeluMaxGrid / g.ncb;
    g.nrg = (int)(M < most ? M : most);
    return g;
}

template <bool WITH_Y>
int gelu_bwd_impl(const void* x, const float* bias, const void* dy, void* dx, void* y, float* dbias, long long M, int F,
                  unsigned flags, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !bias || !dy || !dx || !dbias) return AVION_EINVAL;
    const int rc = gelu_check(M, F, flags);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {x, bias, dy, dx, y, dbias};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 ||
        workspace_bytes < avion_bias_gelu_bwd_workspace_bytes(M, F))
        return AVION_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part = static_cast<float*>(workspace);
    const GeluGrid g = gelu_grid(M, F);
    const bool f16 = (flags & AVION_FLAG_F16) != 0, stream_past_cache = gelu_streams(M, F);
    auto launch = [&](auto fmt, auto streaming) {
        using E = typename decltype(fmt)::type;
        constexpr bool STREAM = decltype(streaming)::value;
        const dim3 grid((unsigned)(g.ncb * g.nrg)), block(kGeluThreads);
        const raw16 *xx = static_cast<const raw16*>(x), *dyy = static_cast<const raw16*>(dy);
        raw16* dxx = static_cast<raw16*>(dx);
        if constexpr (WITH_Y)
            hipLaunchKernelGGL((avion_bias_gelu_bwd_y_kernel<E, STREAM>), grid, block, 0, st, xx, bias, dyy, dxx,
                               static_cast<raw16*>(y), part, (long)M, F, g.ncb);
        else
            hipLaunchKernelGGL((avion_bias_gelu_bwd_kernel<E, STREAM>), grid, block, 0, st, xx, bias, dyy, dxx, part, (long)M, F,
                               g.ncb);
    };
    begin_launch();
    if (f16 && stream_past_cache) launch(TypeTag<F16>{}, std::true_type{});
    else if (f16) launch(TypeTag<F16>{}, std::false_type{});
    else if (stream_past_cache) launch(TypeTag<Bf16>{}, std::true_type{});
    else launch(TypeTag<Bf16>{}, std::false_type{});
    const int r1 = end_launch("launch avion_bias_gelu_bwd_kernel");
    if (r1 != AVION_OK) return r1;
    // column sums of the row groups' partials: the reduction kernel splits its 2 * (F / 2) columns into two outputs
    begin_launch();
    hipLaunchKernelGGL((avion_ln_param_reduce_kernel<void>), dim3((F + kLnReduceCols - 1) / kLnReduceCols),
                       dim3(kLnReduceCols * kLnReduceGroups), 0, st, part, dbias, dbias + F / 2, g.nrg, F / 2);
    return end_launch("launch avion_ln_param_reduce_kernel");
}
// column sums: 256 columns a workgroup; row groups so that a thread has about kSumFly rows, at most 1024 workgroups.
// Up to kSumOneLaunch rows one row group, whose few more loads in a row cost less than the second launch.
GeluGrid sum_grid(long long M, int F)
{
    GeluGrid g;
    g.ncb = (F + kSumCols - 1) / kSumCols;
    g.nrg = 1;
    if (M <= kSumOneLaunch) return g;
    const long long want = (M + kSumRows * kSumFly - 1) / (kSumRows * kSumFly), most = std::max(1, 1024 / g.ncb);
    g.nrg = (int)std::min(want, most);
    return g;
}

constexpr unsigned kAllFlags = AVION_FLAG_F16 | AVION_FLAG_CAUSAL | AVION_FLAG_QKVPACKED;

// q, k, v planes of a packed [B, N, 3, H, d] tensor
struct Planes {
    const char *q, *k, *v;
    Planes(const void* qkv, int H, int d)
    {
        const char* p = static_cast<const char*>(qkv);
        const size_t plane = (size_t)H * d * 2;
        q = p;
        k = p ? p + plane : nullptr;
        v = p ? p + 2 * plane : nullptr;
    }
};

}  // namespace

extern "C" {

int avion_version(void) { return 20200; }  // 2.2.0

const char* avion_strerror(int code)
{
    switch (code) {
        case AVION_OK: return "ok";
        case AVION_EINVAL: return "invalid argument (null pointer, B/H/N < 1, or scale not finite or below 2^-60)";
        case AVION_EUNSUPPORTED: return "unsupported shape or alignment (d must be 64 or 80; pointers 16-byte aligned)";
        case AVION_EWORKSPACE: return "workspace missing, misaligned or too small";
        case AVION_EHIP: return "HIP runtime error (see avion_last_hip_error)";
        case AVION_ESCRATCH: return "problem needs more than the 32 MiB built-in scratch of avion_attn_bwd_noalloc";
        default: return "unknown avion error code";
    }
}

const char* avion_last_hip_error(void) { return g_hip_error; }

int avion_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d,
                   float scale, void* stream)
{
    return fwd_impl(q, k, v, o, lse, B, H, N, d, 1, Variant{false, false}, scale, stream);
}

int avion_attn_fwd_qkvpacked(const void* qkv, void* o, float* lse, int B, int H, int N, int d, float scale, void* stream)
{
    if (H < 1 || d < 1) return AVION_EINVAL;
    const Planes p(qkv, H, d);
    return fwd_impl(p.q, p.k, p.v, o, lse, B, H, N, d, 3, Variant{false, false}, scale, stream);
}

size_t avion_attn_bwd_workspace_bytes(int B, int H, int N, int d)
{
    if (check_shape(B, H, N, d, 1.0f) != AVION_OK) return 0;
    // per (batch, head): LSE*log2e and -delta, each padded to a multiple of 64 rows
    const size_t npad = ((size_t)N + 63) & ~(size_t)63;
    const size_t bytes = (size_t)B * H * 2 * npad * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int avion_attn_bwd_dq(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                      void* dq, int B, int H, int N, int d, float scale, void* workspace, size_t workspace_bytes,
                      void* stream)
{
    return dq_impl(q, k, v, o, lse, dO, dq, B, H, N, d, 1, Variant{false, false}, scale, workspace, workspace_bytes, stream);
}

int avion_attn_bwd_dkdv(const void* q, const void* k, const void* v, const float* lse, const void* dO, void* dk,
                        void* dv, int B, int H, int N, int d, float scale, const void* workspace,
                        size_t workspace_bytes, void* stream)
{
    return dkdv_impl(q, k, v, lse, dO, dk, dv, B, H, N, d, 1, Variant{false, false}, scale, workspace, workspace_bytes,
                     stream);
}

int avion_attn_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                   void* dq, void* dk, void* dv, int B, int H, int N, int d, float scale, void* workspace,
                   size_t workspace_bytes, void* stream)
{
    return bwd_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, d, 1, Variant{false, false}, scale, workspace, workspace_bytes,
                    stream);
}

int avion_attn_bwd_noalloc(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                           void* dq, void* dk, void* dv, int B, int H, int N, int d, float scale, void* stream)
{
    // argument errors first, so that they are reported as for avion_attn_bwd
    if (!q || !k || !v || !o || !lse || !dO || !dq || !dk || !dv) return AVION_EINVAL;
    const int rc = check_shape(B, H, N, d, scale);
    if (rc != AVION_OK) return rc;
    const size_t need = avion_attn_bwd_workspace_bytes(B, H, N, d);
    if (need > kScratchBytes) return AVION_ESCRATCH;
    void* ws = nullptr;
    const int rs = scratch_of_current_device(&ws);
    if (rs != AVION_OK) return rs;
    // every entry of the scratch that the second pass reads is written by the first one (padding
    // rows included), so nothing has to be cleared between calls
    return bwd_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, d, 1, Variant{false, false}, scale, ws, need, stream);
}

int avion_attn_fwd_causal(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d,
                          float scale, void* stream)
{
    return fwd_impl(q, k, v, o, lse, B, H, N, d, 1, Variant{false, true}, scale, stream);
}

int avion_attn_bwd_causal(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                          void* dq, void* dk, void* dv, int B, int H, int N, int d, float scale, void* workspace,
                          size_t workspace_bytes, void* stream)
{
    return bwd_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, d, 1, Variant{false, true}, scale, workspace, workspace_bytes,
                    stream);
}

int avion_attn_fwd_f16(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d,
                       float scale, void* stream)
{
    return fwd_impl(q, k, v, o, lse, B, H, N, d, 1, Variant{true, false}, scale, stream);
}

int avion_attn_bwd_f16(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                       void* dq, void* dk, void* dv, int B, int H, int N, int d, float scale, void* workspace,
                       size_t workspace_bytes, void* stream)
{
    return bwd_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, d, 1, Variant{true, false}, scale, workspace, workspace_bytes,
                    stream);
}

int avion_attn_bwd_qkvpacked(const void* qkv, const void* o, const float* lse, const void* dO, void* dqkv, int B, int H,
                             int N, int d, float scale, void* workspace, size_t workspace_bytes, void* stream)
{
    return avion_attn_bwd_ex(qkv, nullptr, nullptr, o, lse, dO, dqkv, nullptr, nullptr, B, H, N, d, scale,
                             AVION_FLAG_QKVPACKED, workspace, workspace_bytes, stream);
}

int avion_attn_fwd_ex(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d,
                      float scale, unsigned flags, void* stream)
{
    if (flags & ~kAllFlags) return AVION_EINVAL;
    const Variant var{(flags & AVION_FLAG_F16) != 0, (flags & AVION_FLAG_CAUSAL) != 0};
    if (flags & AVION_FLAG_QKVPACKED) {
        if (k || v || H < 1 || d < 1) return AVION_EINVAL;
        const Planes p(q, H, d);
        return fwd_impl(p.q, p.k, p.v, o, lse, B, H, N, d, 3, var, scale, stream);
    }
    return fwd_impl(q, k, v, o, lse, B, H, N, d, 1, var, scale, stream);
}

int avion_attn_bwd_ex(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO,
                      void* dq, void* dk, void* dv, int B, int H, int N, int d, float scale, unsigned flags,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    if (flags & ~kAllFlags) return AVION_EINVAL;
    const Variant var{(flags & AVION_FLAG_F16) != 0, (flags & AVION_FLAG_CAUSAL) != 0};
    if (flags & AVION_FLAG_QKVPACKED) {
        if (k || v || dk || dv || !q || !dq || H < 1 || d < 1) return AVION_EINVAL;
        const Planes in(q, H, d), out(dq, H, d);
        return bwd_impl(in.q, in.k, in.v, o, lse, dO, const_cast<char*>(out.q), const_cast<char*>(out.k),
                        const_cast<char*>(out.v), B, H, N, d, 3, var, scale, workspace, workspace_bytes, stream);
    }
    return bwd_impl(q, k, v, o, lse, dO, dq, dk, dv, B, H, N, d, 1, var, scale, workspace, workspace_bytes, stream);
}

int avion_layernorm_fwd(const void* x, const float* gamma, const float* beta, void* y, float* mean, float* rstd,
                        long long M, int D, float eps, unsigned flags, void* stream)
{
    if (!x || !gamma || !beta || !y || !mean || !rstd) return AVION_EINVAL;
    if (!(eps >= 0.f) || !std::isfinite(eps)) return AVION_EINVAL;
    const int rc = ln_check(M, D, flags);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {x, gamma, beta, y, mean, rstd};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return ln_dispatch(D, (flags & AVION_FLAG_F16) != 0, [&](auto nch, auto fmt) {
        begin_launch();
        hipLaunchKernelGGL((avion_ln_fwd_kernel<decltype(nch)::value, typename decltype(fmt)::type>), dim3(ln_grid(M)),
                           dim3(kLnWaves * 64), 0, st, static_cast<const raw16*>(x), gamma, beta, static_cast<raw16*>(y), mean,
                           rstd, (long)M, D, eps);
        return end_launch("launch avion_ln_fwd_kernel");
    });
}

size_t avion_layernorm_bwd_workspace_bytes(long long M, int D)
{
    if (ln_check(M, D, 0) != AVION_OK) return 0;
    const size_t bytes = (size_t)ln_grid(M) * 2 * D * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int avion_layernorm_bwd(const void* x, const float* gamma, const float* mean, const float* rstd, const void* dy, void* dx,
                        float* dgamma, float* dbeta, long long M, int D, unsigned flags, void* workspace,
                        size_t workspace_bytes, void* stream)
{
    if (!x || !gamma || !mean || !rstd || !dy || !dx || !dgamma || !dbeta) return AVION_EINVAL;
    const int rc = ln_check(M, D, flags);
    if (rc != AVION_OK) return rc;
    const void* ptrs[] = {x, gamma, mean, rstd, dy, dx, dgamma, dbeta};
    for (const void* p : ptrs)
        if (!aligned16(p)) return AVION_EUNSUPPORTED;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 ||
        workspace_bytes < avion_layernorm_bwd_workspace_bytes(M, D))
        return AVION_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part = static_cast<float*>(workspace);
    const unsigned grid = ln_grid(M);
    const int r1 = ln_dispatch(D, (flags & AVION_FLAG_F16) != 0, [&](auto nch, auto fmt) {
        begin_launch();
        hipLaunchKernelGGL((avion_ln_bwd_kernel<decltype(nch)::value, typename decltype(fmt)::type>), dim3(grid),
                           dim3(kLnWaves * 64), (kLnWaves - 1) * 2 * D * sizeof(float), st, static_cast<const raw16*>(x), gamma,
                           mean, rstd, static_cast<const raw16*>(dy), static_cast<raw16*>(dx), part, (long)M, D);
        return end_launch("launch avion_ln_bwd_kernel");
    });
    if (r1 != AVION_OK) return r1;
    begin_launch();
    hipLaunchKernelGGL((avion_ln_param_reduce_kernel<void>), dim3((2 * D + kLnReduceCols - 1) / kLnReduceCols),
                       dim3(kLnReduceCols * kLnReduceGroups), 0, st, part, dgamma, dbeta, (int)grid, D);
    return end_launch("launch avion_ln_param_reduce_kernel");
}

size_t avion_bias_gelu_bwd_workspace_bytes(long long M, int F)
{
    if (gelu_check(M, F, 0) != AVION_OK) return 0;
    const size_t bytes = (size_t)gelu_grid(M, F).nrg * F * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int avion_bias_gelu_fwd(const void* x, const float* bias, void* y, long long M, int F, unsigned flags, void* stream)
{
    if (!x || !bias || !y) return AVION_EINVAL;
    const int rc = gelu_check(M, F, flags);
    if (rc != AVION_OK) return rc;
    if (!aligned16(x) || !aligned16(y) || !aligned16(bias)) return AVION_EUNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const GeluGrid g = gelu_grid(M, F);
    const bool f16 = (flags & AVION_FLAG_F16) != 0, stream_past_cache = gelu_streams(M, F);
    auto launch = [&](auto fmt, auto streaming) {
        hipLaunchKernelGGL((avion_bias_gelu_fwd_kernel<typename decltype(fmt)::type, decltype(streaming)::value>),
                           dim3((unsigned)(g.ncb * g.nrg)), dim3(kGeluThreads), 0, st, static_cast<const raw16*>(x), bias,
                           static_cast<raw16*>(y), (long)M, F, g.ncb);
    };
    begin_launch();
    if (f16 && stream_past_cache) launch(TypeTag<F16>{}, std::true_type{});
    else if (f16) launch(TypeTag<F16>{}, std::false_type{});
    else if (stream_past_cache) launch(TypeTag<Bf16>{}, std::true_type{});
    else launch(TypeTag<Bf16>{}, std::false_type{});
    return end_launch("launch avion_bias_gelu_fwd_kernel");
}

int avion_bias_gelu_bwd(const void* x, const float* bias, const void* dy, void* dx, float* dbias, long long M, int F,
                        unsigned flags, void* workspace, size_t workspace_bytes, void* stream)
{
    return gelu_bwd_impl<false>(x, bias, dy, dx, nullptr, dbias, M, F, flags, workspace, workspace_bytes, stream);
}

int avion_bias_gelu_bwd_y(const void* x, const float* bias, const void* dy, void* dx, void* y, float* dbias, long long M,
                          int F, unsigned flags, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!y) return AVION_EINVAL;
    return gelu_bwd_impl<true>(x, bias, dy, dx, y, dbias, M, F, flags, workspace, workspace_bytes, stream);
}

size_t avion_column_sum_workspace_bytes(long long M, int F)
{
    if (gelu_check(M, F, 0) != AVION_OK) return 0;
    const size_t bytes = (size_t)sum_grid(M, F).nrg * F * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int avion_column_sum(const void* x, void* sum, long long M, int F, unsigned flags, void* workspace, size_t workspace_bytes,
                     void* stream)
{
    if (!x || !sum) return AVION_EINVAL;
    const int rc = gelu_check(M, F, flags);
    if (rc != AVION_OK) return rc;
    if (!aligned16(x) || !aligned16(sum)) return AVION_EUNSUPPORTED;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 ||
        workspace_bytes < avion_column_sum_workspace_bytes(M, F))
        return AVION_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part = static_cast<float*>(workspace);
    const GeluGrid g = sum_grid(M, F);
    auto run = [&](auto fmt) {
        using E = typename decltype(fmt)::type;
        const dim3 grid((unsigned)(g.ncb * g.nrg)), block(kSumCols / 8 * kSumRows);
        const raw16* in = static_cast<const raw16*>(x);
        raw16* out = static_cast<raw16*>(sum);
        begin_launch();
        if (g.nrg == 1)
            hipLaunchKernelGGL((avion_column_sum_kernel<E, true>), grid, block, 0, st, in, out, part, (long)M, F, g.ncb);
        else
            hipLaunchKernelGGL((avion_column_sum_kernel<E, false>), grid, block, 0, st, in, out, part, (long)M, F, g.ncb);
        const int r1 = end_launch("launch avion_column_sum_kernel");
        if (r1 != AVION_OK || g.nrg == 1) return r1;
        begin_launch();
        hipLaunchKernelGGL((avion_ln_param_reduce_kernel<E>), dim3((F + kLnReduceCols - 1) / kLnReduceCols),
                           dim3(kLnReduceCols * kLnReduceGroups), 0, st, part, out, out + F / 2, g.nrg, F / 2);
        return end_launch("launch avion_ln_param_reduce_kernel");
    };
    return (flags & AVION_FLAG_F16) != 0 ? run(TypeTag<F16>{}) : run(TypeTag<Bf16>{});
}

}  // extern "C"
