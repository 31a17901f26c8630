// tfx_grads.h -- what depends on the coefficients in the adjoint of a short-memory
// chain (tfx_short_bwd.hip), as parts of the reduction kernels that both forms of
// the adjoint share (tfx_backward.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "tfx_fft16k.h"

namespace tfx {

struct ShortGradArgs {
    const float2 *spart;  // [run of SB_RUN units][workgroup][16384] cross-spectra, short_bwd_kernel's workgroups nwg
    int32_t nwg;
    int64_t C, N;
    double2 *sum1;
    const double2 *hf;  // FIR response, bin k
    StageList sos;
    int32_t S, M;
    double2 *colsum;  // [128][128] B[k1][j1] of the tap gradient
    double *part;     // [128][5 CASC_MAX] section sums of the blocks
    float *gh;        // tap gradient (null: not wanted)
    const uint32_t *hdr;
};
ShortGradArgs short_grad_args(const BwdPlan &bp, int32_t M, void *area, float *gH, const uint32_t *hdr);

// Units that a workgroup sums in fp32, 16384 bins of sums of up to 16384
// products each; its runs of so many are added in FP64 (by short_spec_sum).
// Every unit rounds the running sum once, so without runs the error grows with
// the signal: 131072 equal rows, 256 units a workgroup, 4.4e-6 of the section
// gradients, 1.8e-7 so (8 x 5.76 M, 6 units a workgroup: the same time).
constexpr uint32_t SB_RUN = 8;

constexpr int SB_SPLITS = 16;

// sum1[split][pos] = sum of the spectra q = split, split + SPLITS, ... of spart in
// that order, in FP64.  Only the first of them are written: by the workgroups of
// the whole runs, and in the last run by those that have a unit left.
constexpr int SB_SUM_BLOCKS = FFT16_POINTS / 256 * SB_SPLITS;  // of 256 threads
__device__ __forceinline__ void short_spec_sum(const ShortGradArgs &a, int block) {
    const int T = FFT16_POINTS - (int)(a.hdr[HDR_SHORT] & ~1u), split = block / (FFT16_POINTS / 256);
    const uint32_t nwg = a.nwg, run = SB_RUN * nwg;
    const uint32_t nunits = tile_units((uint32_t)a.C, f16k::tiles_per_row(a.N, T));
    const uint32_t full = (nunits - 1) / run, nq = full * nwg + min(nwg, nunits - full * run);
    const int pos = block % (FFT16_POINTS / 256) * 256 + threadIdx.x;
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (uint32_t q = split; q < nq; q += SB_SPLITS) {
        const float2 v = a.spart[(int64_t)q * FFT16_POINTS + pos];
        sr += (double)v.x;
        si += (double)v.y;
    }
    a.sum1[(int64_t)split * FFT16_POINTS + pos] = make_double2(sr, si);
}

__device__ __forceinline__ double2 cm(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cmc(double2 a, double2 b) {  // a conj(b)
    return make_double2(fma(a.x, b.x, a.y * b.y), fma(a.y, b.x, -a.x * b.y));
}

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
constexpr int SB_GRAD_BLOCKS = 128;  // of 512 threads
__device__ __forceinline__ void short_grad(const ShortGradArgs &a, int k1) {
    constexpr int NB = FFT16_POINTS;
    __shared__ double co[CASC_MAX][5];
    __shared__ double2 q[128], sH[CASC_MAX][128];
    __shared__ double sv[5 * CASC_MAX][128];  // first the splits' sums, [4][128] double2, at the end the parts of B
    const int tid = threadIdx.x, t = tid & 127, g = tid >> 7;  // bin k2 = t, share g
    const int k = k1 + 128 * t;
    const int S = a.S;
    const int pos = f16k::spec_at(k);
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
__host__ __device__ constexpr int short_out_blocks(int M) { return (M + SB_LAGS - 1) / SB_LAGS; }  // and one, of 256 threads
__device__ __forceinline__ void short_grad_out(const ShortGradArgs &a, const GradList &gsos, int block, int nj) {
    constexpr int NB = FFT16_POINTS;
    const int t = threadIdx.x;
    if (block < nj) {
        const int j = block * SB_LAGS + (t >> 5), l = t & 31;
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
    if (block > nj || t >= 5 * a.S) return;
    int s = t / 5, st = 0;
    while (s >= gsos.len[st]) {
        s -= gsos.len[st];
        ++st;
    }
    if (!gsos.ptr[st]) return;
    double v = 0.0;
#pragma unroll 16
    for (int b = 0; b < 128; ++b) v += a.part[b * 5 * CASC_MAX + t];
    gsos.ptr[st][5 * s + t % 5] = (float)(v / NB);
}

}  // namespace tfx
