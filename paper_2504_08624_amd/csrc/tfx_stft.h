// tfx_stft.h -- what the STFT kernels share: the FFT of a workgroup's batch of
// frame pairs, the twiddles, the dealing of work units (see tfx_stft.hip), and the
// arguments.  For the two files of kernels: in one module the forward kernel kept
// one register more in scratch memory (237 -> 240 us a launch at n_fft 2048).
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

#include "tfx_internal.h"

namespace tfx {
namespace {

constexpr int SWG = 256;
constexpr int TOTMIN = 4096;  // complex values per workgroup transform batch (radix-16 passes: 1 butterfly per lane)

// LDS index with one float2 of padding after every 16: the strided Stockham
// stores of the first passes then spread over the banks.
__device__ __forceinline__ int pad(int i) { return i + (i >> 4); }

template <int LOG2N>
struct Shape {
    static constexpr int N = 1 << LOG2N;
    static constexpr int G = N >= TOTMIN ? 1 : TOTMIN / N;  // transforms per batch
    static constexpr int TOT = G * N;
    static constexpr int F = N / 2 + 1;
    static constexpr int R0 = (LOG2N % 4) ? (1 << (LOG2N % 4)) : 16;  // radix of the first pass
    static constexpr int NP = LOG2N / 4 + ((LOG2N % 4) ? 1 : 0);      // passes
    // base twiddles of the radix-16 passes after the first: pass p >= 1 has
    // sub-transform length R0 * 16^(p-1) and as many table entries
    static constexpr int TWN = N > R0 ? (N - R0) / 15 : 1;
    static constexpr int LDS_BUF = TOT + TOT / 16;
};

struct StftArgs {
    const float *x;       // [C][ldx] signal (forward)
    int64_t ldx, nx;      // row stride and length of the signal
    const float *win;     // window of wl samples at offset wleft in the frame (NULL = ones)
    int32_t wl, wleft;
    int32_t hop, off;     // frame step; left padding (n_fft/2 when centred, else 0)
    float scale;          // forward: 1 or n_fft^-1/2; inverse: (1 or n_fft^1/2) / n_fft
    int64_t T;            // frames per channel
    int64_t P;            // forward: frame pairs per channel, ceil(T/2)
    int64_t pairs;        // forward: C * P
    int64_t units;        // work units (forward: batches of G pairs; inverse: output segments)
    float2 *spec;         // [C][T][n_fft/2+1] (forward output / inverse input)
    // inverse
    int64_t C, L, total, ldy, nseg;
    float *y;
};

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }  // -i a

__device__ __forceinline__ float window_at(const StftArgs &a, int n) {
    const int j = n - a.wleft;
    if (j < 0 || j >= a.wl) return 0.f;
    return a.win ? a.win[j] : 1.f;
}

// forward DFTs of 2, 4, 8 and 16 points in registers
__device__ __forceinline__ void dft2(float2 &a, float2 &b) {
    const float2 t = a;
    a = cadd(t, b);
    b = csub(t, b);
}

__device__ __forceinline__ void dft4(float2 &a, float2 &b, float2 &c, float2 &d) {
    const float2 s02 = cadd(a, c), d02 = csub(a, c), s13 = cadd(b, d), d13 = csub(b, d);
    a = cadd(s02, s13);
    c = csub(s02, s13);
    b = cadd(d02, mul_mi(d13));
    d = csub(d02, mul_mi(d13));
}

constexpr float C8 = 0.70710678118654752f;  // cos(pi/4)
constexpr float C16 = 0.92387953251128674f; // cos(pi/8)
constexpr float S16 = 0.38268343236508977f; // sin(pi/8)

// v[n] -> V[k]: index n = 2 n1 + n2, k = k1 + 4 k2
__device__ __forceinline__ void dft8(float2 *v) {
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    // twiddles W8^(n2 k1) on the n2 = 1 row: k1 = 1, 2, 3
    v[3] = make_float2(C8 * (v[3].x + v[3].y), C8 * (v[3].y - v[3].x));
    v[5] = mul_mi(v[5]);
    v[7] = make_float2(C8 * (v[7].y - v[7].x), -C8 * (v[7].x + v[7].y));
    float2 y[8];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
        float2 a = v[2 * k1], b = v[2 * k1 + 1];
        dft2(a, b);
        y[k1] = a;
        y[k1 + 4] = b;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = y[k];
}

// v[n] -> V[k]: index n = 4 n1 + n2, k = k1 + 4 k2
__device__ __forceinline__ void dft16(float2 *v) {
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[4 + n2], v[8 + n2], v[12 + n2]);
    // element (n1 -> k1, n2) now sits at v[4 k1 + n2]; multiply by W16^(n2 k1)
    const float2 w1 = make_float2(C16, -S16), w2 = make_float2(C8, -C8), w3 = make_float2(S16, -C16);
    const float2 w6 = make_float2(-C8, -C8), w9 = make_float2(-C16, S16);
    v[5] = cmul(v[5], w1);
    v[6] = cmul(v[6], w2);
    v[7] = cmul(v[7], w3);
    v[9] = cmul(v[9], w2);
    v[10] = mul_mi(v[10]);
    v[11] = cmul(v[11], w6);
    v[13] = cmul(v[13], w3);
    v[14] = cmul(v[14], w6);
    v[15] = cmul(v[15], w9);
    float2 y[16];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
        float2 a = v[4 * k1], b = v[4 * k1 + 1], c = v[4 * k1 + 2], d = v[4 * k1 + 3];
        dft4(a, b, c, d);
        y[k1] = a;
        y[k1 + 4] = b;
        y[k1 + 8] = c;
        y[k1 + 12] = d;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = y[k];
}

template <int R>
__device__ __forceinline__ void dft_r(float2 *v) {
    if constexpr (R == 2) dft2(v[0], v[1]);
    else if constexpr (R == 4) dft4(v[0], v[1], v[2], v[3]);
    else if constexpr (R == 8) dft8(v);
    else dft16(v);
}

// Powers w^r, r = 1..15, of the base twiddle w by a product tree (each
// power is at most four products from w).
__device__ __forceinline__ void twiddle16(float2 *v, float2 w1) {
    const float2 w2 = cmul(w1, w1), w3 = cmul(w2, w1), w4 = cmul(w2, w2);
    const float2 w5 = cmul(w4, w1), w6 = cmul(w4, w2), w7 = cmul(w4, w3), w8 = cmul(w4, w4);
    v[1] = cmul(v[1], w1);
    v[2] = cmul(v[2], w2);
    v[3] = cmul(v[3], w3);
    v[4] = cmul(v[4], w4);
    v[5] = cmul(v[5], w5);
    v[6] = cmul(v[6], w6);
    v[7] = cmul(v[7], w7);
    v[8] = cmul(v[8], w8);
    v[9] = cmul(v[9], cmul(w8, w1));
    v[10] = cmul(v[10], cmul(w8, w2));
    v[11] = cmul(v[11], cmul(w8, w3));
    v[12] = cmul(v[12], cmul(w8, w4));
    v[13] = cmul(v[13], cmul(w8, w5));
    v[14] = cmul(v[14], cmul(w8, w6));
    v[15] = cmul(v[15], cmul(w8, w7));
}

// One self-sorting pass: radix R over sub-transforms of length NS, on the G
// rows of N points in buf (padded).  tw = base twiddles exp(-2 pi i k/(NS R)).
template <int LOG2N, int R, int NS>
__device__ __forceinline__ void fft_pass(float2 *buf, const float2 *tw, int tid) {
    constexpr int N = 1 << LOG2N, TOT = Shape<LOG2N>::TOT, M = N / R, NB = TOT / R / SWG;
    static_assert(NB >= 1, "every lane holds at least one butterfly");
    static_assert(NS == 1 || R == 16, "twiddled passes are radix 16");
    float2 v[NB][R];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int i = tid + q * SWG, g = i / M, j = i - g * M;
        if constexpr (M % 16 == 0) {  // r * M keeps the padding phase: one pad per butterfly
            const int b = pad(g * N + j);
#pragma unroll
            for (int r = 0; r < R; ++r) v[q][r] = buf[b + r * (M + M / 16)];
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[q][r] = buf[pad(g * N + j + r * M)];
        }
        if constexpr (NS > 1) twiddle16(v[q], tw[j & (NS - 1)]);
        dft_r<R>(v[q]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int i = tid + q * SWG, g = i / M, j = i - g * M;
        const int o = g * N + (j / NS) * NS * R + (j & (NS - 1));
        if constexpr (NS % 16 == 0) {
            const int b = pad(o);
#pragma unroll
            for (int r = 0; r < R; ++r) buf[b + r * (NS + NS / 16)] = v[q][r];
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) buf[pad(o + r * NS)] = v[q][r];
        }
    }
    __syncthreads();
}

// In-place forward DFT of the G rows; entry and exit with the workgroup in step.
template <int LOG2N>
__device__ __forceinline__ void fft_rows(float2 *buf, const float2 *tw, int tid) {
    using S = Shape<LOG2N>;
    fft_pass<LOG2N, S::R0, 1>(buf, tw, tid);
    if constexpr (S::NP > 1) fft_pass<LOG2N, 16, S::R0>(buf, tw, tid);
    if constexpr (S::NP > 2) fft_pass<LOG2N, 16, S::R0 * 16>(buf, tw + S::R0, tid);
}

// Base twiddles of the radix-16 passes: pass with sub-transform length ns
// at offset ns - R0 (R0, R0 + 16 R0, ...: the tables follow one another),
// entry k = exp(-2 pi i k / (16 ns)), in FP64 then rounded.
template <int LOG2N>
__device__ __forceinline__ void fill_twiddles(float2 *tw, int tid) {
    using S = Shape<LOG2N>;
    for (int ns = S::R0, base = 0; ns * 16 <= S::N; base += ns, ns *= 16) {
        for (int k = tid; k < ns; k += SWG) {
            double sn, cs;
            sincospi(2.0 * (double)k / (16.0 * (double)ns), &sn, &cs);
            tw[base + k] = make_float2((float)cs, (float)-sn);
        }
    }
}

// Units of this workgroup: XCD b % 8 owns a contiguous range of units, which
// its workgroups take in turn.
struct UnitRange {
    int64_t first, end, step;
};

__device__ __forceinline__ UnitRange unit_range(int64_t units) {
    const int64_t per_xcd = (units + 7) / 8;
    const int64_t xcd = blockIdx.x & 7, k = gridDim.x >> 3;
    const int64_t lo = xcd * per_xcd;
    const int64_t hi = lo + per_xcd < units ? lo + per_xcd : units;
    return UnitRange{lo + (int64_t)(blockIdx.x >> 3), hi, k};
}

// a wave-uniform 64-bit value moved to scalar registers
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t reflect(int64_t q, int64_t n) {
    return q < 0 ? -q : (q >= n ? 2 * (n - 1) - q : q);
}

inline StftArgs make_args(const StftPlan &sp) {
    StftArgs a{};
    const int N = 1 << sp.log2n;
    a.x = sp.x;
    a.ldx = sp.ldx;
    a.nx = sp.nx;
    a.win = sp.win;
    a.wl = sp.win_length;
    a.wleft = (N - sp.win_length) / 2;
    a.hop = sp.hop;
    a.off = sp.center ? N / 2 : 0;
    a.T = sp.T;
    a.C = sp.C;
    return a;
}

inline int batch_of(int log2n) { return (1 << log2n) >= TOTMIN ? 1 : TOTMIN >> log2n; }
inline dim3 unit_grid(int64_t units, int per_cu) {
    // enough workgroups for per_cu resident per CU, in eight equal XCD shares
    const int64_t per_xcd = (units + 7) / 8;
    const int64_t cap = 32 * (int64_t)per_cu;
    const int64_t k = per_xcd < cap ? per_xcd : cap;
    return dim3((unsigned)(8 * (k > 0 ? k : 1)));
}

// Arguments of an inverse (sp.length > 0).
inline StftArgs inverse_args(const StftPlan &sp) {
    const int N = 1 << sp.log2n;
    StftArgs a = make_args(sp);
    a.scale = (float)((sp.normalized ? std::sqrt((double)N) : 1.0) / (double)N);
    a.spec = reinterpret_cast<float2 *>(const_cast<float *>(sp.spec_in));
    a.L = sp.length;
    a.total = (int64_t)N + (int64_t)sp.hop * (sp.T - 1);
    a.ldy = sp.ldy;
    a.y = sp.y;
    return a;
}

}  // namespace

// The inverse for hops of 256 H samples (tfx_istft.hip); *done says whether it took the call.
hipError_t launch_istft_slide(const StftPlan &sp, bool *done);

}  // namespace tfx
