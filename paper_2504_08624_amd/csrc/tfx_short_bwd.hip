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

// Units that a workgroup sums in fp32, 16384 bins of sums of up to 16384
// products each; its runs of so many are added in FP64 (by short_spec_sum_kernel).
// Every unit rounds the running sum once, so without runs the error grows with
// the signal: 131072 equal rows, 256 units a workgroup, 4.4e-6 of the section
// gradients, 1.8e-7 so (8 x 5.76 M, 6 units a workgroup: the same time).
constexpr uint32_t SB_RUN = 8;

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

// sum1[split][pos] = sum of the spectra q = split, split + SPLITS, ... of spart in
// that order, in FP64.  Only the first of them are written: by the workgroups of
// the whole rounds, and in the last round by those that have a unit left.
constexpr int SB_SPLITS = 16;
__global__ __launch_bounds__(256) void short_spec_sum_kernel(const float2 *spart, int32_t nwg, int64_t C, int64_t N,
                                                             double2 *sum1, const uint32_t *hdr) {
    if (!short_done(hdr)) return;
    const int T = NB - (int)(hdr[HDR_SHORT] & ~1u);
    const uint32_t nunits = tile_units((uint32_t)C, tiles_per_row(N, T)), round = SB_RUN * nwg;
    const uint32_t full = (nunits - 1) / round, nq = full * nwg + min((uint32_t)nwg, nunits - full * round);
    const int pos = blockIdx.x * 256 + threadIdx.x;
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (uint32_t q = blockIdx.y; q < nq; q += SB_SPLITS) {
        const float2 v = spart[(int64_t)q * NB + pos];
        sr += (double)v.x;
        si += (double)v.y;
    }
    sum1[(int64_t)blockIdx.y * NB + pos] = make_double2(sr, si);
}

__device__ __forceinline__ double2 cm(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cmc(double2 a, double2 b) {  // a conj(b)
    return make_double2(fma(a.x, b.x, a.y * b.y), fma(a.y, b.x, -a.x * b.y));
}

struct ShortGradArgs {
    const double2 *sum1;
    const double2 *hf;  // FIR response, bin k
    StageList sos;
    int32_t S, M;
    double2 *colsum;  // [128][128] B[k1][j1] of the tap gradient
    double *part;     // [128][5 CASC_MAX] section sums of the blocks
    const uint32_t *hdr;
    GradList gsos;
    float *gh;
};

// Block k1: bins k = k1 + 128 k2.  With R the summed spectrum, Hf the
// FIR's response and H_s = B_s / A_s the sections', T_s = R conj(Hf prod_{t != s}
// H_t / A_s) gives the bin's shares of section s's gradients: Re T_s conj(z^i)
// for b_i, -Re T_s conj(H_s z^i) for a_i (z = e^{-2 pi i k / N}).  The tap
// gradient is the inverse transform of Q = R conj(prod H_t); its first half, for
// j = j1 + 128 j2, B[k1][j1] = sum_k2 Q(k) e^{2 pi i k2 j1 / 128}, is done here.
//
// 16384 bins are few for the chip, so the time is one wave's instructions: four
// threads share a bin (two sections each, a quarter of the sums over k2), the
// sums over the bins go through LDS, a row a wave (64 x 192000, 8 sections: 17.7
// us with one thread a bin and every sum in every wave, 9.2 us so).
__global__ __launch_bounds__(512) void short_grad_kernel(ShortGradArgs a) {
    __shared__ double co[CASC_MAX][5];
    __shared__ double2 q[128], sH[CASC_MAX][128];
    __shared__ double sv[5 * CASC_MAX][128];  // first the splits' sums, [4][128] double2, at the end the parts of B
    if (!short_done(a.hdr)) return;
    const int tid = threadIdx.x, t = tid & 127, g = tid >> 7;  // bin k2 = t, share g
    const int k1 = blockIdx.x, k = k1 + 128 * t;
    const int S = a.S;
    const int pos = spec_at(k);
    static_assert(SB_SPLITS % 4 == 0 && CASC_MAX == 8, "shares of the four threads of a bin");
    double2 Rk = make_double2(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < SB_SPLITS / 4; ++w) {
        const double2 v = a.sum1[(int64_t)(4 * w + g) * NB + pos];
        Rk.x += v.x;
        Rk.y += v.y;
    }
    const double2 hf = a.hf[k];
    if (tid < 5 * S) {
        int s = tid / 5, st = 0;
        while (s >= a.sos.len[st]) {
            s -= a.sos.len[st];
            ++st;
        }
        co[tid / 5][tid % 5] = (double)a.sos.ptr[st][5 * s + tid % 5];
    }
    double2 *part = reinterpret_cast<double2 *>(&sv[0][0]);
    part[128 * g + t] = Rk;
    double2 z;
    sincospi(-2.0 * (double)k / NB, &z.y, &z.x);
    const double2 z2 = cm(z, z);
    __syncthreads();
    double2 iA[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int s = g + 4 * u;
        if (s < S) {
            const double2 n = make_double2(co[s][0] + co[s][1] * z.x + co[s][2] * z2.x, co[s][1] * z.y + co[s][2] * z2.y);
            const double2 d = make_double2(1.0 + co[s][3] * z.x + co[s][4] * z2.x, co[s][3] * z.y + co[s][4] * z2.y);
            const double r = 1.0 / fma(d.x, d.x, d.y * d.y);
            iA[u] = make_double2(d.x * r, -d.y * r);
            sH[s][t] = cm(n, iA[u]);
        }
    }
    Rk = part[t];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
        Rk.x += part[128 * w + t].x;
        Rk.y += part[128 * w + t].y;
    }
    __syncthreads();
    double2 pr[2] = {make_double2(1.0, 0.0), make_double2(1.0, 0.0)}, all = make_double2(1.0, 0.0);  // without s; all
#pragma unroll
    for (int s = 0; s < CASC_MAX; ++s) {
        if (s < S) {
            const double2 h = sH[s][t];
            if (s != g) pr[0] = cm(pr[0], h);
            if (s != g + 4) pr[1] = cm(pr[1], h);
            if (g == 0) all = cm(all, h);
        }
    }
    if (g == 0) q[t] = cmc(Rk, all);
    const double2 X = cmc(Rk, hf);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int s = g + 4 * u;
        if (s < S) {
            const double2 T = cmc(X, cm(pr[u], iA[u]));
            const double2 U = cmc(T, sH[s][t]);
            sv[5 * s][t] = T.x;
            sv[5 * s + 1][t] = fma(T.x, z.x, T.y * z.y);
            sv[5 * s + 2][t] = fma(T.x, z2.x, T.y * z2.y);
            sv[5 * s + 3][t] = -fma(U.x, z.x, U.y * z.y);
            sv[5 * s + 4][t] = -fma(U.x, z2.x, U.y * z2.y);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) {  // row 8 i + wave
        const int r = 8 * i + (tid >> 6);
        if (r < 5 * S) {
            double v = sv[r][tid & 63] + sv[r][64 + (tid & 63)];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
            if ((tid & 63) == 0) a.part[k1 * 5 * CASC_MAX + r] = v;
        }
    }
    // first half of the tap gradient's inverse transform: j1 = t, k2 from 32 g on,
    // whose first factor e^{2 pi i 32 g j1 / 128} is i^(g j1)
    double2 st, w, b = make_double2(0.0, 0.0);
    sincospi((double)t / 64.0, &st.y, &st.x);
    const int quarter = (g * t) & 3;
    w.x = quarter == 0 ? 1.0 : quarter == 2 ? -1.0 : 0.0;
    w.y = quarter == 1 ? 1.0 : quarter == 3 ? -1.0 : 0.0;
#pragma unroll 4
    for (int k2 = 32 * g; k2 < 32 * g + 32; ++k2) {
        const double2 v = q[k2];
        b.x = fma(v.x, w.x, fma(-v.y, w.y, b.x));
        b.y = fma(v.x, w.y, fma(v.y, w.x, b.y));
        w = cm(w, st);
    }
    __syncthreads();  // the rows are summed
    part[128 * g + t] = b;
    __syncthreads();
    if (g == 0) {
#pragma unroll
        for (int u = 1; u < 4; ++u) {
            b.x += part[128 * u + t].x;
            b.y += part[128 * u + t].y;
        }
        a.colsum[k1 * 128 + t] = b;
    }
}

// Blocks < nj: dL/dh[j] = Re sum_k1 e^{2 pi i k1 j / N} B[k1][j mod 128] / N for
// 8 lags, 32 lanes each; the last block: the section sums over the 128 blocks
// in order, written to the stages' gradients.
constexpr int SB_LAGS = 8;
__global__ __launch_bounds__(256) void short_grad_out_kernel(ShortGradArgs a, int32_t nj) {
    if (!short_done(a.hdr)) return;
    const int t = threadIdx.x;
    if ((int)blockIdx.x < nj) {
        const int j = blockIdx.x * SB_LAGS + (t >> 5), l = t & 31;
        if (j >= a.M) return;
        double2 w, st;
        sincospi(2.0 * (double)((l * j) & (NB - 1)) / NB, &w.y, &w.x);
        sincospi(2.0 * (double)((32 * j) & (NB - 1)) / NB, &st.y, &st.x);
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const double2 b = a.colsum[(l + 32 * m) * 128 + (j & 127)];
            s = fma(b.x, w.x, fma(-b.y, w.y, s));
            w = cm(w, st);
        }
#pragma unroll
        for (int d = 16; d >= 1; d >>= 1) s += __shfl_xor(s, d);
        if (l == 0) a.gh[j] = (float)(s / NB);
        return;
    }
    if (t >= 5 * a.S) return;
    int s = t / 5, st = 0;
    while (s >= a.gsos.len[st]) {
        s -= a.gsos.len[st];
        ++st;
    }
    if (!a.gsos.ptr[st]) return;
    double v = 0.0;
#pragma unroll 16
    for (int b = 0; b < 128; ++b) v += a.part[b * 5 * CASC_MAX + t];
    a.gsos.ptr[st][5 * s + t % 5] = (float)(v / NB);
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
                            void *area, float *gH, uint32_t *hdr) {
    const ChainPlan &p = bp.fwd;
    const Lay l = short_lay(p.C, p.N);
    char *w = static_cast<char *>(area);
    hipStream_t st = p.stream;
    bool any = gH != nullptr;
    for (int i = 0; i < bp.gsos.n; ++i) any = any || bp.gsos.ptr[i] != nullptr;
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
    a.want = any ? 1 : 0;
    a.spart = reinterpret_cast<float4 *>(w + l.spart);
    const int64_t nwg = short_bwd_wgs(p.C, p.N);
    hipLaunchKernelGGL(short_bwd_kernel, dim3((unsigned)nwg), dim3(WGB), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !any) return e;
    ShortGradArgs r{};
    r.sum1 = reinterpret_cast<double2 *>(w + l.sum1);
    r.hf = reinterpret_cast<const double2 *>(w + l.hf);
    r.sos = p.sos;
    r.S = p.S;
    r.M = M;
    r.colsum = reinterpret_cast<double2 *>(w + l.colsum);
    r.part = reinterpret_cast<double *>(w + l.part);
    r.hdr = hdr;
    r.gsos = bp.gsos;
    r.gh = gH;
    hipLaunchKernelGGL(short_spec_sum_kernel, dim3(NB / 256, SB_SPLITS), dim3(256), 0, st,
                       reinterpret_cast<const float2 *>(w + l.spart), (int32_t)nwg, p.C, p.N,
                       reinterpret_cast<double2 *>(w + l.sum1), static_cast<const uint32_t *>(hdr));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(short_grad_kernel, dim3(128), dim3(512), 0, st, r);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int32_t nj = gH ? (M + SB_LAGS - 1) / SB_LAGS : 0;
    hipLaunchKernelGGL(short_grad_out_kernel, dim3((unsigned)(nj + 1)), dim3(256), 0, st, r, nj);
    return hipGetLastError();
}

}  // namespace tfx
