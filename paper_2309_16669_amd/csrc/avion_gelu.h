// Bias + GELU, forward and backward: the elementwise step between the two matrix products of the
// encoder's MLP (Sec. 3, "Video Transformer": every layer holds a 2-layer MLP), the third entry of the
// paper's memory profile (Sec. 4.1).  The paper names no activation; this is the exact (erf) form of
// the plain ViT.  Per element, with h = x + bias_c:
//     y  = h Phi(h),                    Phi(h) = (1 + erf(h / sqrt 2)) / 2
//     dx = dy (Phi(h) + h phi(h)),      phi(h) = exp(-h^2 / 2) / sqrt(2 pi)
//     dbias_c = sum_rows dx_c           (summed from the unrounded fp32 dx)
// The backward rebuilds Phi and phi from x: the activation's output need not be kept for it.
//
// Bound by memory bandwidth (forward one read and one write of 2 bytes per element, backward two reads
// and one write).  A workgroup of 128 threads owns 1024 consecutive columns (thread = one 16-byte
// chunk, so its 8 bias values and its 8 partial sums of dbias live in registers for the whole kernel)
// and walks the rows of its row group with a stride, four rows in flight.  The partial sums of the row
// groups are added by avion_ln_param_reduce_kernel in a fixed order: no atomics, bit-reproducible.
//
// Tensors much larger than the chip's last-level cache (256 MB) are read and written with
// nontemporal accesses (STREAM): nothing of them will be found there again, and keeping them out of it
// is worth 4 % (forward) and 7 % (backward) on [50176, 3072]; smaller tensors take ordinary accesses,
// so that a consumer right after finds them cached.
//
// erf: 1 - erf(z) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-z^2), t = 1 / (1 + p z), z >= 0
// (Abramowitz and Stegun 7.1.26, absolute error < 1.5e-7, far below the rounding of the outputs);
// its exponential exp(-z^2) = exp(-h^2 / 2) is the one phi(h) needs, so each element costs one
// exponential and one reciprocal.
#pragma once
#include "avion_common.h"
#include "avion_ln.h"

constexpr int kGeluThreads = 128;     // threads per workgroup = 16-byte column chunks per workgroup
constexpr int kGeluRows = 4;          // rows in flight per thread
constexpr int kGeluMaxGrid = 4096;    // workgroups of a launch (column blocks x row groups)

template <bool STREAM>
DEVINL u32x4 gelu_load(const raw16* p)
{
    const u32x4* q = reinterpret_cast<const u32x4*>(p);
    return STREAM ? __builtin_nontemporal_load(q) : *q;
}
template <bool STREAM>
DEVINL void gelu_store(raw16* p, u32x4 v)
{
    u32x4* q = reinterpret_cast<u32x4*>(p);
    if (STREAM) __builtin_nontemporal_store(v, q);
    else *q = v;
}

// Phi(h) and h * phi(h)
DEVINL void gelu_terms(float h, float& cdf, float& hpdf)
{
    const float e = fast_exp2(h * h * (-0.5f * kLog2e));  // exp(-h^2 / 2)
    const float z = fabsf(h) * 0.70710678f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    const float tail = 0.5f * poly * t * e;  // (1 - erf(|h| / sqrt 2)) / 2
    cdf = h >= 0.f ? 1.0f - tail : tail;
    hpdf = h * e * 0.3989422804f;
}

// ncb = column blocks; gridDim.x = ncb * (row groups)
template <typename E, bool STREAM>
__global__ void __launch_bounds__(kGeluThreads)
avion_bias_gelu_fwd_kernel(const raw16* __restrict__ x, const float* __restrict__ bias, raw16* __restrict__ y, long M, int F,
                           int ncb)
{
    const int cb = blockIdx.x % ncb;
    const long rg = blockIdx.x / ncb, nrg = gridDim.x / ncb;
    const int col = (cb * kGeluThreads + threadIdx.x) * 8;
    if (col >= F) return;
    float b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = bias[col + e];
    for (long r = rg; r < M; r += nrg * kGeluRows) {
        u32x4 in[kGeluRows];
#pragma unroll
        for (int k = 0; k < kGeluRows; ++k) {
            const long row = r + k * nrg;
            if (row < M) in[k] = gelu_load<STREAM>(x + row * F + col);
        }
#pragma unroll
        for (int k = 0; k < kGeluRows; ++k) {
            const long row = r + k * nrg;
            if (row < M) {
                float o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float h = E::widen(as_frag8(in[k]), e) + b[e];
                    float cdf, hpdf;
                    gelu_terms(h, cdf, hpdf);
                    o[e] = h * cdf;
                }
                u32x4 w;
#pragma unroll
                for (int p = 0; p < 4; ++p) w[p] = E::pack(o[2 * p], o[2 * p + 1]);
                gelu_store<STREAM>(y + row * F + col, w);
            }
        }
    }
}

// dx, and this row group's partial sums of dbias into part[row group][F].  With WITH_Y also the activation's output,
// which the second product's weight gradient needs: 8 bytes an element in one pass instead of 10 in two (a forward
// and this): [12544, 3072] 31 + 55 -> 62 us with dx in dy's place, [50176, 3072] 124 + 190 -> 251.
template <typename E, bool STREAM, bool WITH_Y>
DEVINL void gelu_bwd_body(const raw16* x, const float* bias, const raw16* dy, raw16* dx, raw16* y, float* part, long M, int F,
                          int ncb)
{
    const int cb = blockIdx.x % ncb;
    const long rg = blockIdx.x / ncb, nrg = gridDim.x / ncb;
    const int col = (cb * kGeluThreads + threadIdx.x) * 8;
    if (col >= F) return;
    float b[8], acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        b[e] = bias[col + e];
        acc[e] = 0.f;
    }
    for (long r = rg; r < M; r += nrg * kGeluRows) {
        u32x4 in[kGeluRows], gin[kGeluRows];
#pragma unroll
        for (int k = 0; k < kGeluRows; ++k) {
            const long row = r + k * nrg;
            if (row < M) {
                in[k] = gelu_load<STREAM>(x + row * F + col);
                gin[k] = gelu_load<STREAM>(dy + row * F + col);
            }
        }
#pragma unroll
        for (int k = 0; k < kGeluRows; ++k) {
            const long row = r + k * nrg;
            if (row < M) {
                float o[8], act[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float h = E::widen(as_frag8(in[k]), e) + b[e];
                    float cdf, hpdf;
                    gelu_terms(h, cdf, hpdf);
                    o[e] = E::widen(as_frag8(gin[k]), e) * (cdf + hpdf);
                    acc[e] += o[e];
                    act[e] = h * cdf;
                }
                u32x4 w;
#pragma unroll
                for (int p = 0; p < 4; ++p) w[p] = E::pack(o[2 * p], o[2 * p + 1]);
                gelu_store<STREAM>(dx + row * F + col, w);
                if constexpr (WITH_Y) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) w[p] = E::pack(act[2 * p], act[2 * p + 1]);
                    gelu_store<STREAM>(y + row * F + col, w);
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[rg * F + col + e] = acc[e];
}

template <typename E, bool STREAM>
__global__ void __launch_bounds__(kGeluThreads)
avion_bias_gelu_bwd_kernel(const raw16* __restrict__ x, const float* __restrict__ bias, const raw16* __restrict__ dy,
                           raw16* __restrict__ dx, float* __restrict__ part, long M, int F, int ncb)
{
    gelu_bwd_body<E, STREAM, false>(x, bias, dy, dx, nullptr, part, M, F, ncb);
}
// dx may be dy: an element is read and written by one thread
template <typename E, bool STREAM>
__global__ void __launch_bounds__(kGeluThreads)
avion_bias_gelu_bwd_y_kernel(const raw16* __restrict__ x, const float* __restrict__ bias, const raw16* dy, raw16* dx,
                             raw16* __restrict__ y, float* __restrict__ part, long M, int F, int ncb)
{
    gelu_bwd_body<E, STREAM, true>(x, bias, dy, dx, y, part, M, F, ncb);
}

// Column sums of a [M, F] tensor of 16-bit elements, in fp32, rounded once: the gradient of a bias that is added to
// every row (the second product's).  A workgroup takes 256 columns (32 threads of 16 bytes) and every nrg-th group of
// 8 rows; its 8 row lanes meet in LDS.  With one row group the sums leave as they are, otherwise as fp32 partials that
// avion_ln_param_reduce_kernel adds in a fixed order.
// Bound by memory where M is large, by its launches where it is small.  Calls one after the other, torch's sum -> this:
// 12544 x 768 19.8 -> 7.3 us, 50176 x 768 34.4 -> 16.1, 12544 x 3072 29.1 -> 15.6, 1024 x 768 9.8 -> 6.4, 77 x 512 5.3 -> 3.3.
// One launch instead of two up to 256 rows, at 768 columns (in brackets without the host, in a graph): 128 rows 3.6 us against 6.3
// (3.5; 4.5), 256 4.7 against 6.3 (4.8; 4.6), 384 6.2 against 6.3 (6.3; 4.6), 1024 13.7 against 6.4; the same from 64 to 8192 columns.
constexpr int kSumCols = 256, kSumRows = 8, kSumFly = 4, kSumOneLaunch = 256;
template <typename E, bool ONLY>
__global__ void __launch_bounds__(kSumCols / 8 * kSumRows)
avion_column_sum_kernel(const raw16* __restrict__ x, raw16* __restrict__ sum, float* __restrict__ part, long M, int F, int ncb)
{
    __shared__ __attribute__((aligned(16))) float sh[kSumRows - 1][kSumCols];
    const int cb = blockIdx.x % ncb, c = threadIdx.x % (kSumCols / 8), lane_row = threadIdx.x / (kSumCols / 8);
    const long rg = blockIdx.x / ncb, stride = gridDim.x / ncb * kSumRows;
    const int col = cb * kSumCols + c * 8;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (col < F) {
        for (long r = rg * kSumRows + lane_row; r < M; r += stride * kSumFly) {
            u32x4 in[kSumFly];
#pragma unroll
            for (int k = 0; k < kSumFly; ++k) {
                const long row = r + k * stride;
                in[k] = row < M ? *reinterpret_cast<const u32x4*>(x + row * F + col) : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int k = 0; k < kSumFly; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += E::widen(as_frag8(in[k]), e);
        }
    }
    if (lane_row > 0) store8(&sh[lane_row - 1][c * 8], acc);
    __syncthreads();
    if (lane_row > 0 || col >= F) return;
#pragma unroll
    for (int i = 0; i < kSumRows - 1; ++i) {
        float a[8];
        load8(&sh[i][c * 8], a);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += a[e];
    }
    if constexpr (ONLY) {
        u32x4 w;
#pragma unroll
        for (int p = 0; p < 4; ++p) w[p] = E::pack(acc[2 * p], acc[2 * p + 1]);
        *reinterpret_cast<u32x4*>(sum + col) = w;
    } else {
        store8(part + rg * F + col, acc);
    }
}
