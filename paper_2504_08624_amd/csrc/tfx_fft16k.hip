// tfx_fft16k.hip -- overlap-save FIR with 16384-point FFTs (filters of up to
// 8193 taps).
//
// With V the filter's memory (M - 1 rounded up to a multiple of 64) a block of
// 16384 samples gives T = 16384 - V outputs.  A workgroup filters two tiles,
// neighbours in one channel or, of many short rows, two rows of one tile each,
// one in the real and one in the imaginary part of the transform (the taps are
// real, so the two outputs separate).  Convolution: a tile's block starts V
// samples before it, and the last T outputs of the circular convolution are
// the tile.  Correlation (the FIR adjoint, gx[n] = sum_k h[k] g[n + k]): the
// block starts at the tile, the spectrum is conjugated, and the first T
// outputs are the tile.
//
// Bound by its vector arithmetic, not by HBM: per block two transforms
// (tfx_fft16k.h) and the product.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tfx_fft16k.h"

namespace tfx {

using namespace f16k;

namespace {

struct F16Args {
    const float *x;
    float *y;
    int64_t C, N, ldx, ldy;
    uint32_t nunits, tpc;     // units (pairs of tiles), tiles per channel
    int32_t V;                // filter memory, a multiple of 64
    const float2 *tw;
    const float2 *hs;   // tap spectrum / 16384 in the transform's output order
    const float *hist;  // streaming: [C][hlen] inputs before the block (convolution only), or null
    int64_t hlen;
    int32_t correlate;
    const uint32_t *gate;  // workspace header of a chain whose short-memory kernel ran before, or null
};

// Whether an output of the block is not finite: a NaN or an infinity in a block's
// input reaches every output as a NaN; an overflow in the last pass may be in any
// one of them.
__device__ __forceinline__ bool not_finite(const float (&zr)[R], const float (&zi)[R]) {
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < R; ++k) m = fmaxf(fmaxf(fabsf(zr[k]), fabsf(zi[k])), m);
    return !(m < INFINITY) || zr[0] != zr[0] || zi[0] != zi[0];
}

// A block with an output that is not finite is done again, a tile at a time and in
// runs of at most 8192 outputs up to the next multiple of 8192, from their own
// inputs alone: a bad sample then reaches no other tile and at most two such
// runs of its own (with 8191 taps no more can be told apart: the filter is
// as long).  A run that is still not finite is done once more at 2^-24 of its
// size, for sums that overflow on the way to outputs that do not.
constexpr int NARROW = 8192;
constexpr float NARROW_SCALE = 0x1p-24f;

// The run [lo, lo + cnt) of a tile alone.
__device__ __forceinline__ bool narrow_run(const F16Args &a, const float *xc, float *yc, const float *hc, int64_t lo,
                                           int cnt, float scale, float *P, const float2 *twl, int *s_bad, int t) {
    const int lead = a.correlate ? 0 : a.V, tail = a.V - lead;
    float zr[R], zi[R];
    load_block(zr, xc, lo - lead, min(a.N, lo + cnt + tail), hc, a.hlen, opaque(t));
#pragma unroll
    for (int k = 0; k < R; ++k) {
        zr[k] *= scale;
        zi[k] = 0.f;
    }
    if (t == 0) *s_bad = 0;
    __syncthreads();  // the run before: its reads of P and of s_bad
    convolve(zr, zi, a.hs, a.correlate ? -1.f : 1.f, P, twl, a.tw, t);
    if (not_finite(zr, zi)) *s_bad = 1;
    const float back = 1.f / scale;
#pragma unroll
    for (int k = 0; k < R; ++k) zr[k] *= back;
    store_block(zr, yc, lo, lead, cnt, a.N, opaque(t));
    __syncthreads();
    const bool bad = *s_bad != 0;
    __syncthreads();
    return bad;
}

// The unit's tiles again in narrow runs.  Everything is formed anew from the
// kernel's arguments: kept across the transform before, it would cost that
// registers (44 scalar ones spilled: 110 us over 4096 x 4096 samples, 109 so).
__device__ __forceinline__ void redo_unit(uint32_t block, int wave, float *P, const float2 *twl, int *s_bad) {
    typedef __attribute__((address_space(4))) const F16Args KernArgs;
    KernArgs *ka = (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka), "+s"(block), "+s"(wave));
    F16Args a{};
    a.x = ka->x;
    a.y = ka->y;
    a.C = ka->C;
    a.N = ka->N;
    a.ldx = ka->ldx;
    a.ldy = ka->ldy;
    a.nunits = ka->nunits;
    a.tpc = ka->tpc;
    a.V = ka->V;
    a.tw = ka->tw;
    a.hs = ka->hs;
    a.hist = ka->hist;
    a.hlen = ka->hlen;
    a.correlate = ka->correlate;
    const int t = 64 * wave + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), T = NB - a.V;
    const TilePair p = tile_pair(xcd_unit(block, a.nunits), (uint32_t)a.C, a.tpc, T);
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < (p.two ? 2 : 1); ++s) {
        const int64_t ch = s ? p.chB : p.chA, first = s ? p.nB : p.nA, last = min(first + T, a.N);
        const float *xc = a.x + ch * a.ldx, *hc = a.hist ? a.hist + ch * a.hlen : nullptr;
        float *yc = a.y + ch * a.ldy;
        for (int64_t lo = first; lo < last;) {
            const int64_t end = min(first + T, (lo / NARROW + 1) * NARROW);
            const int cnt = (int)(end - lo);
#pragma unroll 1
            for (float scale = 1.f; narrow_run(a, xc, yc, hc, lo, cnt, scale, P, twl, s_bad, opaque(t)) && scale == 1.f;)
                scale = NARROW_SCALE;
            lo = end;
        }
    }
}

__global__ __launch_bounds__(WGB, 4) void fir16k_kernel(F16Args a) {
    __shared__ __align__(16) float P[PLANE];
    __shared__ __align__(16) float2 twl[TW_LDS];
    __shared__ int s_bad;
    if (a.gate && short_done(a.gate)) return;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    tw_stage(twl, a.tw, t);
    if (t == 0) s_bad = 0;
    const int T = NB - a.V;
    const TilePair p = tile_pair(xcd_unit(blockIdx.x, a.nunits), (uint32_t)a.C, a.tpc, T);
    const int lead = a.correlate ? 0 : a.V;
    {
        float zr[R], zi[R];
        load_block(zr, a.x + p.chA * a.ldx, p.nA - lead, a.N, a.hist ? a.hist + p.chA * a.hlen : nullptr, a.hlen, t);
        load_block(zi, a.x + p.chB * a.ldx, p.nB - lead, p.two ? a.N : 0,
                   a.hist && p.two ? a.hist + p.chB * a.hlen : nullptr, a.hlen, t);
        __syncthreads();  // the twiddle rows
        convolve(zr, zi, a.hs, a.correlate ? -1.f : 1.f, P, twl, a.tw, t);
        if (not_finite(zr, zi)) s_bad = 1;
        store_block(zr, a.y + p.chA * a.ldy, p.nA, lead, T, a.N, t);
        if (p.two) store_block(zi, a.y + p.chB * a.ldy, p.nB, lead, T, a.N, t);
    }
    __syncthreads();
    if (s_bad) redo_unit(blockIdx.x, wave, P, twl, &s_bad);
}

// A short-memory chain (FIR and cascade as one filter of memory V; the grid is
// sized for the longest memory).  The same two
// transforms a block as above.  A value that is not finite marks the run, and
// the general kernels behind this one do it again.
struct ShortArgs {
    const float *x;
    float *y;
    int64_t C, N, ldx, ldy;
    const float2 *tw, *hs;
    const ShortTab *st;
    uint32_t *hdr;
    int32_t M;
    uint32_t max_units;
};

// A value as the FIR's operand type holds it: the matrix-core modes round their
// operands to bf16 or fp16 and add in fp32; the FIR here is linear in them, so
// rounded operands through the fp32 transform are that same product sum.
template <int CMP>
__device__ __forceinline__ float operand(float v) {
    if constexpr (CMP == TFX_COMPUTE_BF16) return (float)(__bf16)v;
    if constexpr (CMP == TFX_COMPUTE_F16) return (float)(_Float16)v;
    return v;
}

template <int CMP>
__global__ __launch_bounds__(WGB, 4) void short16k_kernel(ShortArgs a) {
    __shared__ __align__(16) float P[PLANE];
    __shared__ __align__(16) float2 twl[TW_LDS];
    const uint32_t tabs = a.hdr[HDR_TABS];
    int V = short_memory(a.st, a.M, threadIdx.x & 63);
    const int T = NB - V;
    const uint32_t tpc = tiles_per_row(a.N, T), nunits = tile_units((uint32_t)a.C, tpc);
    if (!tabs || unit_work((uint32_t)a.C, tpc) > units_with_memory(a.max_units, V)) V = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.hdr[HDR_SHORT] = V > 0 ? (uint32_t)(V | 1) : 0u;
    if (V == 0) return;
    if (blockIdx.x >= nunits) return;
    const int t = threadIdx.x;
    tw_stage(twl, a.tw, t);
    const uint32_t u = xcd_unit(blockIdx.x, nunits);
    const TilePair p = tile_pair(u, (uint32_t)a.C, tpc, T);
    float zr[R], zi[R];
    load_block(zr, a.x + p.chA * a.ldx, p.nA - V, a.N, nullptr, 0, t);
    load_block(zi, a.x + p.chB * a.ldx, p.nB - V, p.two ? a.N : 0, nullptr, 0, t);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        zr[k] = operand<CMP>(zr[k]);
        zi[k] = operand<CMP>(zi[k]);
    }
    __syncthreads();  // the twiddle rows
    convolve(zr, zi, a.hs, 1.f, P, twl, a.tw, t);
    store_block(zr, a.y + p.chA * a.ldy, p.nA, V, T, a.N, t);
    if (p.two) store_block(zi, a.y + p.chB * a.ldy, p.nB, V, T, a.N, t);
    if (not_finite(zr, zi))
        __hip_atomic_store(a.hdr + HDR_BAD, a.hdr[HDR_EPOCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

size_t fft16k_table_bytes() { return (size_t)TW_FLOAT2 * sizeof(float2) + (size_t)NB * sizeof(float2); }

hipError_t launch_fft16k(const float *x, float *y, int64_t C, int64_t N, int64_t ldx, int64_t ldy, int32_t M,
                         const void *tab, bool correlate, const float *hist, const uint32_t *hdr, hipStream_t st) {
    if (N == 0) return hipSuccess;
    F16Args a{};
    a.x = x;
    a.y = y;
    a.C = C;
    a.N = N;
    a.ldx = ldx;
    a.ldy = ldy;
    a.V = (M - 1 + 63) / 64 * 64;
    const int64_t T = NB - a.V;
    a.tpc = (uint32_t)((N + T - 1) / T);
    a.nunits = tile_units((uint32_t)C, a.tpc);
    a.tw = static_cast<const float2 *>(tab);
    a.hs = a.tw + TW_FLOAT2;
    a.hist = (!correlate && M > 1) ? hist : nullptr;
    a.hlen = M > 1 ? M - 1 : 0;
    a.correlate = correlate ? 1 : 0;
    a.gate = hdr;
    hipLaunchKernelGGL(fir16k_kernel, dim3(a.nunits), dim3(WGB), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_short16k(const float *x, float *y, int64_t C, int64_t N, int64_t ldx, int64_t ldy, int32_t M,
                           int32_t cmp, uint32_t max_units, const void *tab, const void *tw, uint32_t *hdr,
                           hipStream_t st) {
    ShortArgs a{};
    a.x = x;
    a.y = y;
    a.C = C;
    a.N = N;
    a.ldx = ldx;
    a.ldy = ldy;
    a.tw = static_cast<const float2 *>(tw);
    a.hs = static_cast<const float2 *>(tab) + TW_FLOAT2;
    a.st = reinterpret_cast<const ShortTab *>(static_cast<const char *>(tab) + fft16k_table_bytes());
    a.hdr = hdr;
    a.M = M;
    a.max_units = max_units;
    const int64_t T = NB - FFT16_MEM;  // the shortest tiles: the most blocks
    const dim3 grid(std::min(std::max(units_with_memory(max_units, FFT16_MEM), (uint32_t)C),
                             tile_units((uint32_t)C, (uint32_t)((N + T - 1) / T))));
    switch (cmp) {
        case TFX_COMPUTE_BF16: hipLaunchKernelGGL(short16k_kernel<TFX_COMPUTE_BF16>, grid, dim3(WGB), 0, st, a); break;
        case TFX_COMPUTE_F16: hipLaunchKernelGGL(short16k_kernel<TFX_COMPUTE_F16>, grid, dim3(WGB), 0, st, a); break;
        default: hipLaunchKernelGGL(short16k_kernel<TFX_COMPUTE_F32>, grid, dim3(WGB), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace tfx
