// tfx_fft16k.hip -- overlap-save FIR with 16384-point FFTs (filters of up to
// 8193 taps).
//
// With V the filter's memory (M - 1 rounded up to a multiple of 64) a block of
// 16384 samples gives T = 16384 - V outputs.  A workgroup filters two
// neighbouring tiles of one channel, one in the real and one in the imaginary
// part of the transform (the taps are real, so the two outputs separate
// exactly, and channels never mix).  Convolution: a tile's block starts V
// samples before it, and the last T outputs of the circular convolution are
// the tile.  Correlation (the FIR adjoint, gx[n] = sum_k h[k] g[n + k]): the
// block starts at the tile, the spectrum is conjugated, and the first T
// outputs are the tile.
//
// Bound by its vector arithmetic and LDS traffic, not by HBM: per block two
// transforms (tfx_fft16k.h) and the product, about 1700 lane operations per
// 16 points.
#include <hip/hip_runtime.h>

#include "tfx_fft16k.h"

namespace tfx {

using namespace f16k;

namespace {

struct F16Args {
    const float *x;
    float *y;
    int64_t C, N, ldx, ldy;
    uint32_t nunits, per_ch;  // units (pairs of tiles), units per channel
    int32_t V;                // filter memory, a multiple of 64
    const float2 *tw;
    const float2 *hs;   // tap spectrum / 16384 in the transform's output order
    const float *hist;  // streaming: [C][hlen] inputs before the block (convolution only), or null
    int64_t hlen;
    int32_t correlate;
};

__global__ __launch_bounds__(WGB, 4) void fir16k_kernel(F16Args a) {
    __shared__ __align__(16) float P[PLANE];
    __shared__ __align__(16) float2 twl[TW_FLOAT2];
    const int t = threadIdx.x;
    tw_stage(twl, a.tw, t);
    const uint32_t u = xcd_unit(blockIdx.x, a.nunits);
    const int64_t ch = u / a.per_ch;
    const int T = NB - a.V;
    const int64_t n0 = (int64_t)(u - (uint32_t)ch * a.per_ch) * 2 * T, n1 = n0 + T;
    const int lead = a.correlate ? 0 : a.V;
    const float *xc = a.x + ch * a.ldx;
    const float *hc = a.hist ? a.hist + ch * a.hlen : nullptr;
    float zr[R], zi[R];
    load_block(zr, xc, n0 - lead, a.N, hc, a.hlen, t);
    load_block(zi, xc, n1 - lead, a.N, hc, a.hlen, t);
    __syncthreads();  // the twiddle rows
    forward(zr, zi, P, twl, t);
    spec_mul(zr, zi, a.hs, t, a.correlate ? -1.f : 1.f);
    inverse(zr, zi, P, twl, t);
    float *yc = a.y + ch * a.ldy;
    store_block(zr, yc, n0, lead, T, a.N, t);
    if (n1 < a.N) store_block(zi, yc, n1, lead, T, a.N, t);
}

// Twiddle rows and tap spectrum / 16384, in FP64 and rounded once.  A block of
// 256 threads covers 16 bins: lane (kk, jj) sums the taps j = jj (mod 16) of
// bin k = 16 blk + kk by Horner's rule in w^16, the 16 partial sums are added
// by a fixed shuffle tree.  The taps are real: bins 0..8192 are computed, the
// others are their conjugates.  (Per prepare of an 8191-tap filter this spreads
// over the chip what one workgroup's fp32 transform did in 17 us.)
__global__ __launch_bounds__(256) void fft16k_prepare_kernel(const float *h, int32_t M, float2 *tw, float2 *hs) {
    extern __shared__ double ht[];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int steps = (M + 15) / 16;
    for (int j = tid; j < 16 * steps; j += 256) ht[j] = j < M ? (double)h[j] : 0.0;
    const int i = b * 256 + tid;
    if (i < TW_FLOAT2) {
        const int row = i / TWS, k = i % TWS;
        const int m = k < R ? ((row < 32 ? 16 * row : row - 32) * k) & (NB - 1) : 0;
        double s, c;
        sincospi(-2.0 * (double)m / NB, &s, &c);
        tw[i] = k < R ? make_float2((float)c, (float)s) : make_float2(0.f, 0.f);
    }
    __syncthreads();
    const int kk = tid >> 4, jj = tid & 15;
    const int k = 16 * b + kk;
    double wr, wi, pr, pi;
    sincospi(-2.0 * (double)((16 * k) & (NB - 1)) / NB, &wi, &wr);
    sincospi(-2.0 * (double)((jj * k) & (NB - 1)) / NB, &pi, &pr);
    double ar = 0.0, ai = 0.0;
#pragma unroll 4
    for (int m = steps - 1; m >= 0; --m) {
        const double nr = fma(ar, wr, fma(-ai, wi, ht[jj + 16 * m]));
        ai = fma(ar, wi, ai * wr);
        ar = nr;
    }
    double hr = ar * pr - ai * pi, hi = fma(ar, pi, ai * pr);
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
        hr += __shfl_xor(hr, d);
        hi += __shfl_xor(hi, d);
    }
    if (jj == 0 && k <= NB / 2) {
        const float2 v = make_float2((float)(hr / NB), (float)(hi / NB));
        hs[spec_at(k)] = v;
        if (k > 0 && k < NB / 2) hs[spec_at(NB - k)] = make_float2(v.x, -v.y);
    }
}
constexpr int PREP_BLOCKS = NB / 2 / 16 + 1;
static_assert(PREP_BLOCKS * 256 >= TW_FLOAT2, "the prepare grid covers the twiddle rows");

}  // namespace

size_t fft16k_table_bytes() { return (size_t)TW_FLOAT2 * sizeof(float2) + (size_t)NB * sizeof(float2); }

hipError_t launch_fft16k_prepare(const float *h, int32_t M, void *tab, hipStream_t st) {
    float2 *tw = static_cast<float2 *>(tab);
    hipLaunchKernelGGL(fft16k_prepare_kernel, dim3(PREP_BLOCKS), dim3(256), (size_t)((M + 15) / 16 * 16) * sizeof(double),
                       st, h, M, tw, tw + TW_FLOAT2);
    return hipGetLastError();
}

hipError_t launch_fft16k(const float *x, float *y, int64_t C, int64_t N, int64_t ldx, int64_t ldy, int32_t M,
                         const void *tab, bool correlate, const float *hist, hipStream_t st) {
    if (N == 0) return hipSuccess;
    F16Args a{};
    a.x = x;
    a.y = y;
    a.C = C;
    a.N = N;
    a.ldx = ldx;
    a.ldy = ldy;
    a.V = (M - 1 + 63) / 64 * 64;
    const int64_t T2 = 2 * (int64_t)(NB - a.V);
    a.per_ch = (uint32_t)((N + T2 - 1) / T2);
    a.nunits = (uint32_t)(C * a.per_ch);
    a.tw = static_cast<const float2 *>(tab);
    a.hs = a.tw + TW_FLOAT2;
    a.hist = (!correlate && M > 1) ? hist : nullptr;
    a.hlen = M > 1 ? M - 1 : 0;
    a.correlate = correlate ? 1 : 0;
    hipLaunchKernelGGL(fir16k_kernel, dim3(a.nunits), dim3(WGB), 0, st, a);
    return hipGetLastError();
}

}  // namespace tfx
