// tfx_short_bwd.hip -- the adjoint of a short-memory chain (FIR and cascade as
// one FIR of memory V, see tfx_internal.h).
//
// With H the chain's response, h its impulse response and g the upstream
// gradient:  dL/dx = correlation of g with h, and dL/dh[k] = r[k] = sum over
// channels and n of x[n] g[n + k], k <= V.  Every coefficient enters through h,
// so with R the spectrum whose inverse transform's real part is r,
//   dL/dtheta = sum_k r[k] dh[k]/dtheta = Re sum_f R(f) conj(dH/dtheta(f)) / N
// (dh/dtheta has died out beyond V as h has, so the lags above V, which R also
// holds, do not count).  No section signal is formed and no adjoint state
// scanned: per tile three transforms, where the cascade adjoint rebuilt every
// section's input in S (S - 1) / 2 chunk passes and took a look-back per
// section.  All that depends on the coefficients is done once per call, on 16384
// bins, in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tfx_fft16k.h"
#include "tfx_grads.h"

namespace tfx {

using namespace f16k;

namespace {

struct ShortBwdArgs {
    const float *x, *g;
    float *gx;
    int64_t C, N, ldx, ldg, ldgx;
    const float2 *tw, *hs;  // twiddle rows, combined spectrum / 16384
    const ShortTab *st;
    uint32_t *hdr;
    int32_t M;
    uint32_t max_units;
    int32_t want;   // coefficient gradients wanted
    float4 *spart;  // [run of SB_RUN units][workgroup][16][512] summed spectra, two bins of thread t at [j / 2][t]
};

// Units (two neighbouring tiles, see TilePair) of a workgroup: with B the
// transform of the gradient's blocks [n0, n0 + 16384) and X that of the input's
// tiles [n0, n0 + T), zero-padded, gx = IFFT(conj(H) B) over the tiles and
// conj(X) B sums over a run of units in registers; both products use the one B.
// 192 data registers a thread: one workgroup a CU.
__global__ __launch_bounds__(WGB, 2) void short_bwd_kernel(ShortBwdArgs a) {
    __shared__ __align__(16) float P[PLANE];
    __shared__ __align__(16) float2 twl[TW_LDS];
    const int t = threadIdx.x;
    int V = short_memory(a.st, a.M, t & 63);
    const int T = NB - V;
    const uint32_t tpc = tiles_per_row(a.N, T), nunits = tile_units((uint32_t)a.C, tpc);
    if (unit_work((uint32_t)a.C, tpc) > units_with_memory(a.max_units, V)) V = 0;
    if (blockIdx.x == 0 && t == 0) a.hdr[HDR_SHORT] = V > 0 ? (uint32_t)(V | 1) : 0u;
    if (V == 0) return;
    tw_stage(twl, a.tw, t);
    float m = 0.f;
#pragma unroll 1
    for (uint32_t run = 0, i = blockIdx.x; i < nunits; ++run) {
        float ar[R], ai[R];
#pragma unroll
        for (int k = 0; k < R; ++k) ar[k] = ai[k] = 0.f;
#pragma unroll 1
        for (uint32_t n = 0; n < SB_RUN && i < nunits; ++n, i += gridDim.x) {
            const uint32_t u = xcd_unit(i, nunits);
            const TilePair p = tile_pair(u, (uint32_t)a.C, tpc, T);
            const int64_t limB = p.two ? a.N : 0;
            float zr[R], zi[R];
            load_block(zr, a.g + p.chA * a.ldg, p.nA, a.N, nullptr, 0, t);
            load_block(zi, a.g + p.chB * a.ldg, p.nB, limB, nullptr, 0, t);
            __syncthreads();  // the twiddle rows; the last unit's reads of P
            forward(zr, zi, P, twl, a.tw, t);
            if (a.want) {
                float xr[R], xi[R];
                load_tile(xr, a.x + p.chA * a.ldx, p.nA, T, a.N, t);
                load_tile(xi, a.x + p.chB * a.ldx, p.nB, T, limB, t);
                __syncthreads();  // the other waves' reads of their rows of P
                forward(xr, xi, P, twl, a.tw, t);
#pragma unroll
                for (int k = 0; k < R; ++k) {  // += conj(X) B
                    ar[k] = fmaf(xr[k], zr[k], fmaf(xi[k], zi[k], ar[k]));
                    ai[k] = fmaf(xr[k], zi[k], fmaf(-xi[k], zr[k], ai[k]));
                }
            }
            product_inverse(zr, zi, a.hs, -1.f, P, twl, a.tw, t);
            store_block(zr, a.gx + p.chA * a.ldgx, p.nA, 0, T, a.N, t);
            if (p.two) store_block(zi, a.gx + p.chB * a.ldgx, p.nB, 0, T, a.N, t);
#pragma unroll
            for (int k = 0; k < R; ++k) m = fmaxf(fmaxf(fabsf(zr[k]), fabsf(zi[k])), m);
            if (zr[0] != zr[0] || zi[0] != zi[0]) m = INFINITY;
        }
        if (a.want) {
            float4 *o = a.spart + ((int64_t)run * gridDim.x + blockIdx.x) * (NB / 2) + t;
#pragma unroll
            for (int p = 0; p < R / 2; ++p) {
                o[p * WGB] = make_float4(ar[2 * p], ai[2 * p], ar[2 * p + 1], ai[2 * p + 1]);
                if (!(fabsf(ar[2 * p]) + fabsf(ai[2 * p]) + fabsf(ar[2 * p + 1]) + fabsf(ai[2 * p + 1]) < INFINITY))
                    m = INFINITY;
            }
        }
    }
    if (!(m < INFINITY))
        __hip_atomic_store(a.hdr + HDR_BAD, a.hdr[HDR_EPOCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

// Units of the adjoint at most (the shortest tiles), its workgroups (one a CU).
int64_t short_bwd_units(int64_t C, int64_t N) {
    const int64_t T = NB - FFT16_MEM;
    return tile_units((uint32_t)C, (uint32_t)((N + T - 1) / T));
}
int64_t short_bwd_wgs(int64_t C, int64_t N) { return std::min<int64_t>(short_bwd_units(C, N), 256); }

struct Lay {
    size_t hf, spart, sum1, colsum, part, total;
};
Lay short_lay(int64_t C, int64_t N) {
    Lay l{};
    size_t off = 0;
    l.hf = off;
    off += al256((size_t)NB * sizeof(double2));
    l.spart = off;
    const int64_t nwg = short_bwd_wgs(C, N);
    off += al256((size_t)((short_bwd_units(C, N) + SB_RUN * nwg - 1) / (SB_RUN * nwg) * nwg) * NB * sizeof(float2));
    l.sum1 = off;
    off += al256((size_t)SB_SPLITS * NB * sizeof(double2));
    l.colsum = off;
    off += al256((size_t)128 * 128 * sizeof(double2));
    l.part = off;
    off += al256((size_t)128 * 5 * CASC_MAX * sizeof(double));
    l.total = off;
    return l;
}

}  // namespace

size_t short_bwd_bytes(int64_t C, int64_t N) { return short_lay(C, N).total; }
void *short_bwd_hf(void *area) { return area; }

hipError_t launch_short_bwd(const BwdPlan &bp, int32_t M, uint32_t max_units, const void *tab, const void *tw,
                            void *area, bool want, uint32_t *hdr) {
    const ChainPlan &p = bp.fwd;
    const Lay l = short_lay(p.C, p.N);
    char *w = static_cast<char *>(area);
    hipStream_t st = p.stream;
    ShortBwdArgs a{};
    a.x = p.x;
    a.g = bp.gy;
    a.gx = bp.gx;
    a.C = p.C;
    a.N = p.N;
    a.ldx = p.ldx;
    a.ldg = bp.ldg;
    a.ldgx = bp.ldgx;
    a.tw = static_cast<const float2 *>(tw);
    a.hs = static_cast<const float2 *>(tab) + TW_FLOAT2;
    a.st = reinterpret_cast<const ShortTab *>(static_cast<const char *>(tab) + fft16k_table_bytes());
    a.hdr = hdr;
    a.M = M;
    a.max_units = max_units;
    a.want = want ? 1 : 0;
    a.spart = reinterpret_cast<float4 *>(w + l.spart);
    const int64_t nwg = short_bwd_wgs(p.C, p.N);
    hipLaunchKernelGGL(short_bwd_kernel, dim3((unsigned)nwg), dim3(WGB), 0, st, a);
    return hipGetLastError();
}

ShortGradArgs short_grad_args(const BwdPlan &bp, int32_t M, void *area, float *gH, const uint32_t *hdr) {
    const ChainPlan &p = bp.fwd;
    const Lay l = short_lay(p.C, p.N);
    char *w = static_cast<char *>(area);
    ShortGradArgs r{};
    r.spart = reinterpret_cast<const float2 *>(w + l.spart);
    r.nwg = (int32_t)short_bwd_wgs(p.C, p.N);
    r.C = p.C;
    r.N = p.N;
    r.sum1 = reinterpret_cast<double2 *>(w + l.sum1);
    r.hf = reinterpret_cast<const double2 *>(w + l.hf);
    r.sos = p.sos;
    r.S = p.S;
    r.M = M;
    r.colsum = reinterpret_cast<double2 *>(w + l.colsum);
    r.part = reinterpret_cast<double *>(w + l.part);
    r.gh = gH;
    r.hdr = hdr;
    return r;
}

}  // namespace tfx
