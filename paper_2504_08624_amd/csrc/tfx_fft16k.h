// tfx_fft16k.h -- the 16384-point complex FFT of one 512-thread workgroup.
//
// 16384 = 32 x 32 x 16.  With n = 512 a + t (a < 32, t < 512), t = 16 b + c
// (b < 32, c < 16), k = k1 + 32 k2 + 1024 k3 (k1, k2 < 32, k3 < 16) and
// W = e^{-2 pi i / 16384}:
//   pass A  (thread t, over a):        32-point DFT, then * W^(t k1)
//   pass B  (thread (k1, c), over b):  32-point DFT, then * W^(32 c k2)
//   pass C  (thread (k1, k2 mod 16), twice, over c): 16-point DFT
// A thread holds 32 complex values (64 data registers), so two workgroups
// share a CU (four waves per SIMD).
//
// Exchanges: one LDS plane P of 32 rows (k1) of 512 values, the real parts
// first, then the imaginary parts.  A row is padded to 528 floats, so the 4
// rows a wave touches at once lie 16 banks apart.  Threads (k1, .) are the 16
// lanes t >> 4 = k1, so a row is read by one wave only and the exchange
// between passes B and C stays inside a wave: it needs no barrier.  Inside a
// row, pass B's value (k2, c) sits at 16 k2 + 4 ((c / 4 + k2 / 4) mod 4) +
// c mod 4: the rotation of the 4-float groups spreads pass C's 16-byte reads
// over all banks.  Every address is a lane constant plus an immediate.
//
// Per block that leaves 3 barriers a transform; the former 16 x 16 x 16 x 4
// form passed three exchanges through the workgroup (11 barriers a transform)
// and spent a select on most LDS addresses.
#pragma once
#include <hip/hip_runtime.h>

#include "tfx_device.h"
#include "tfx_internal.h"

namespace tfx {
namespace f16k {

constexpr int NB = FFT16_POINTS;   // 16384
constexpr int WGB = 512;           // threads per workgroup
constexpr int R = 32;              // complex values per thread
constexpr int ROW = 528;           // floats per LDS row (512 + 16)
constexpr int PLANE = R * ROW;     // floats of the exchange plane

// Twiddle rows of 32 entries, padded to TWS float2 (16 lanes reading 16
// different rows hit 64 different banks): row p < 32 holds W^(16 p k), row
// 32 + q (q < 16) holds W^(q k).  W^(t k) = row[t >> 4][k] row[32 + (t & 15)][k]
// and W^(32 c k) = row[2 c][k].
constexpr int TWS = 34, TW_ROWS = 48;
constexpr int TW_FLOAT2 = TW_ROWS * TWS;

// Bin k of the transform's output is value spec_j(k) of thread spec_t(k).
// Spectra are stored as pairs of bins per thread, [j / 2][t][j % 2].
__host__ __device__ constexpr int spec_t(int k) { return (k & 31) * 16 + ((k >> 5) & 15); }
__host__ __device__ constexpr int spec_j(int k) { return 16 * ((k >> 9) & 1) + (k >> 10); }
__host__ __device__ constexpr int spec_at(int k) { return ((spec_j(k) >> 1) * WGB + spec_t(k)) * 2 + (spec_j(k) & 1); }

// cos / sin of 2 pi m / 32
__device__ constexpr float c32[16] = {1.f, 0.98078528040323044913f, 0.92387953251128675613f, 0.83146961230254523708f,
                                      0.70710678118654752440f, 0.55557023301960222474f, 0.38268343236508977173f,
                                      0.19509032201612826785f, 0.f, -0.19509032201612826785f,
                                      -0.38268343236508977173f, -0.55557023301960222474f, -0.70710678118654752440f,
                                      -0.83146961230254523708f, -0.92387953251128675613f, -0.98078528040323044913f};
__device__ constexpr float s32[16] = {0.f, 0.19509032201612826785f, 0.38268343236508977173f, 0.55557023301960222474f,
                                      0.70710678118654752440f, 0.83146961230254523708f, 0.92387953251128675613f,
                                      0.98078528040323044913f, 1.f, 0.98078528040323044913f,
                                      0.92387953251128675613f, 0.83146961230254523708f, 0.70710678118654752440f,
                                      0.55557023301960222474f, 0.38268343236508977173f, 0.19509032201612826785f};

// In-register 32-point DFT, X_k = sum_n v_n e^{SIGN 2 pi i n k / 32}: two
// 16-point DFTs of the even and odd values and one butterfly level.
template <int SIGN>
__device__ __forceinline__ void dft32(float (&zr)[R], float (&zi)[R]) {
    float er[16], ei[16], qr[16], qi[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        er[m] = zr[2 * m];
        ei[m] = zi[2 * m];
        qr[m] = zr[2 * m + 1];
        qi[m] = zi[2 * m + 1];
    }
    dft16<SIGN>(er, ei);
    dft16<SIGN>(qr, qi);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float tr, ti;
        if (k == 0) {
            tr = qr[k];
            ti = qi[k];
        } else if (k == 8) {  // -i or i
            tr = SIGN < 0 ? qi[k] : -qi[k];
            ti = SIGN < 0 ? -qr[k] : qr[k];
        } else {
            const float c = c32[k], s = SIGN < 0 ? -s32[k] : s32[k];
            tr = qr[k] * c - qi[k] * s;
            ti = qr[k] * s + qi[k] * c;
        }
        zr[k] = er[k] + tr;
        zi[k] = ei[k] + ti;
        zr[k + 16] = er[k] - tr;
        zi[k + 16] = ei[k] - ti;
    }
}

// Multiplies the thread's 32 values by a twiddle row (or its conjugate; entry
// 0 is 1), the row's 16-byte pieces read from LDS as they are used.
template <bool CONJ>
__device__ __forceinline__ void twiddle_row(float (&zr)[R], float (&zi)[R], const float2 *row) {
    const float4 *r4 = reinterpret_cast<const float4 *>(row);
#pragma unroll
    for (int g = 0; g < R / 2; ++g) {
        const float4 w = r4[g];
        if (g > 0) cmul_tw<CONJ>(zr[2 * g], zi[2 * g], make_float2(w.x, w.y));
        cmul_tw<CONJ>(zr[2 * g + 1], zi[2 * g + 1], make_float2(w.z, w.w));
    }
}
template <bool CONJ>
__device__ __forceinline__ void twiddle_a(float (&zr)[R], float (&zi)[R], const float2 *tw, int t) {
    twiddle_row<CONJ>(zr, zi, tw + (t >> 4) * TWS);
    twiddle_row<CONJ>(zr, zi, tw + (32 + (t & 15)) * TWS);
}

// A copy of the thread index the compiler cannot see through: addresses
// derived from it are formed where they are used instead of being held in
// registers across the transform (128 registers a thread, 64 of them data).
__device__ __forceinline__ int opaque(int t) {
    asm volatile("" : "+v"(t));
    return t;
}

// Copies the twiddle rows into the workgroup's LDS copy (every load issued
// before the first store; the caller passes a barrier before the first use).
__device__ __forceinline__ void tw_stage(float2 *twl, const float2 *tw, int t) {
    constexpr int N4 = TW_FLOAT2 / 2, P = (N4 + WGB - 1) / WGB;
    const float4 *src = reinterpret_cast<const float4 *>(tw);
    float4 *dst = reinterpret_cast<float4 *>(twl);
    float4 w[P];
#pragma unroll
    for (int r = 0; r < P; ++r) w[r] = src[min(t + r * WGB, N4 - 1)];
#pragma unroll
    for (int r = 0; r < P; ++r)
        if (t + r * WGB < N4) dst[t + r * WGB] = w[r];
}

// Address bases of the exchanges (floats): rows are read back by the threads
// t >> 4, c = t & 15; pass C's threads are (k1, k2 mod 16) = (t >> 4, t & 15).
__device__ __forceinline__ int row_base(int t) { return ROW * (t >> 4) + (t & 15); }
__device__ __forceinline__ int rot_base(int t, int r) {  // pass B's value k2 at rot_base((k2 / 4) mod 4) + 16 k2
    const int c = t & 15;
    return ROW * (t >> 4) + 4 * (((c >> 2) + r) & 3) + (c & 3);
}
__device__ __forceinline__ int grp_base(int t, int g) {  // pass C's values c = 4 g .. 4 g + 3 of k2 = t & 15 (+ 16 h)
    const int q = t & 15;
    return ROW * (t >> 4) + 16 * q + 4 * ((g + (q >> 2)) & 3);
}

__device__ __forceinline__ void put_cols(const float (&z)[R], float *P, int t) {
#pragma unroll
    for (int k = 0; k < R; ++k) P[t + ROW * k] = z[k];
}
__device__ __forceinline__ void get_cols(float (&z)[R], const float *P, int t) {
#pragma unroll
    for (int k = 0; k < R; ++k) z[k] = P[t + ROW * k];
}
__device__ __forceinline__ void put_row(const float (&z)[R], float *P, int t) {
    float *p = P + row_base(t);
#pragma unroll
    for (int b = 0; b < R; ++b) p[16 * b] = z[b];
}
__device__ __forceinline__ void get_row(float (&z)[R], const float *P, int t) {
    const float *p = P + row_base(t);
#pragma unroll
    for (int b = 0; b < R; ++b) z[b] = p[16 * b];
}
// the B <-> C exchange of one plane, inside a wave (its LDS accesses complete
// in order; the fences keep the compiler from moving them across each other)
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void b_to_c(float (&z)[R], float *P, int t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float *p = P + rot_base(t, r);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k2 = 16 * (j >> 2) + 4 * r + (j & 3);
            p[16 * k2] = z[k2];
        }
    }
    wave_fence();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 *p = reinterpret_cast<const float4 *>(P + grp_base(t, g));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 w = p[64 * h];
            z[16 * h + 4 * g] = w.x;
            z[16 * h + 4 * g + 1] = w.y;
            z[16 * h + 4 * g + 2] = w.z;
            z[16 * h + 4 * g + 3] = w.w;
        }
    }
    wave_fence();
}
__device__ __forceinline__ void c_to_b(float (&z)[R], float *P, int t) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        float4 *p = reinterpret_cast<float4 *>(P + grp_base(t, g));
#pragma unroll
        for (int h = 0; h < 2; ++h)
            p[64 * h] = make_float4(z[16 * h + 4 * g], z[16 * h + 4 * g + 1], z[16 * h + 4 * g + 2],
                                    z[16 * h + 4 * g + 3]);
    }
    wave_fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float *p = P + rot_base(t, r);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k2 = 16 * (j >> 2) + 4 * r + (j & 3);
            z[k2] = p[16 * k2];
        }
    }
    wave_fence();
}

template <int SIGN>
__device__ __forceinline__ void dft16_halves(float (&zr)[R], float (&zi)[R]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float ar[16], ai[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            ar[c] = zr[16 * h + c];
            ai[c] = zi[16 * h + c];
        }
        dft16<SIGN>(ar, ai);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            zr[16 * h + c] = ar[c];
            zi[16 * h + c] = ai[c];
        }
    }
}

// Forward transform.  In: thread t holds z[512 a + t] at a.  Out: bin
// k1 + 32 (t & 15) + 512 h + 1024 k3 (k1 = t >> 4) at 16 h + k3.  The caller
// has passed a barrier since the last access to P by another wave; the
// transform ends with accesses to the wave's own rows only.
__device__ __forceinline__ void forward(float (&zr)[R], float (&zi)[R], float *P, const float2 *tw, int t) {
    dft32<-1>(zr, zi);
    twiddle_a<false>(zr, zi, tw, opaque(t));
    put_cols(zr, P, opaque(t));
    __syncthreads();
    get_row(zr, P, opaque(t));
    __syncthreads();
    put_cols(zi, P, opaque(t));
    __syncthreads();
    get_row(zi, P, opaque(t));
    dft32<-1>(zr, zi);
    twiddle_row<false>(zr, zi, tw + 2 * (opaque(t) & 15) * TWS);
    wave_fence();
    b_to_c(zr, P, opaque(t));
    b_to_c(zi, P, opaque(t));
    dft16_halves<-1>(zr, zi);
}

// Inverse of forward without the 1/16384 factor: from its output layout back
// to its input layout.  Starts on the wave's own rows of P (no barrier needed
// after forward); ends with reads of every row.
__device__ __forceinline__ void inverse(float (&zr)[R], float (&zi)[R], float *P, const float2 *tw, int t) {
    dft16_halves<1>(zr, zi);
    c_to_b(zr, P, opaque(t));
    c_to_b(zi, P, opaque(t));
    twiddle_row<true>(zr, zi, tw + 2 * (opaque(t) & 15) * TWS);
    dft32<1>(zr, zi);
    put_row(zr, P, opaque(t));
    __syncthreads();
    get_cols(zr, P, opaque(t));
    __syncthreads();
    put_row(zi, P, opaque(t));
    __syncthreads();
    get_cols(zi, P, opaque(t));
    twiddle_a<true>(zr, zi, tw, opaque(t));
    dft32<1>(zr, zi);
}

// z *= H, or z *= conj(H): the spectrum's pairs of bins in the thread's order,
// a quarter of the loads issued at a time (registers; the lane index laundered
// per quarter so the next loads are not hoisted above the products).
__device__ __forceinline__ void spec_mul(float (&zr)[R], float (&zi)[R], const float2 *hs, int t, float sg) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 *h4 = reinterpret_cast<const float4 *>(hs) + opaque(t);
        float4 w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) w[g] = h4[(4 * q + g) * WGB];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int j = 8 * q + 2 * g;
            cmul_tw<false>(zr[j], zi[j], make_float2(w[g].x, sg * w[g].y));
            cmul_tw<false>(zr[j + 1], zi[j + 1], make_float2(w[g].z, sg * w[g].w));
            asm volatile("" : "+v"(zr[j]), "+v"(zi[j]), "+v"(zr[j + 1]), "+v"(zi[j + 1]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Unit u of nu (a pair of neighbouring tiles of one channel) of block id i:
// the blocks of one XCD (block i runs on XCD i mod 8) take one contiguous
// range of units, so tiles that share input are read through one L2.
__device__ __forceinline__ uint32_t xcd_unit(uint32_t i, uint32_t nu) {
    const uint32_t x = i & 7u, per = nu >> 3, rem = nu & 7u;
    return __builtin_amdgcn_readfirstlane(x * per + (x < rem ? x : rem) + (i >> 3));
}

// 32 samples x[base + 512 a + t] of a channel row, zero outside [0, lim); n < 0
// reads the history hist[hlen + n] if there is one.
__device__ __forceinline__ void load_block(float (&z)[R], const float *x, int64_t base, int64_t lim,
                                           const float *hist, int64_t hlen, int t) {
    if (base >= 0 && base + NB <= lim) {
        const float *p = x + base + t;
#pragma unroll
        for (int a = 0; a < R; ++a) z[a] = p[512 * a];
        return;
    }
#pragma unroll
    for (int a = 0; a < R; ++a) {
        const int64_t n = base + 512 * a + t;
        float v = 0.f;
        if (n >= 0 && n < lim) v = x[n];
        else if (hist && n < 0 && n >= -hlen) v = hist[hlen + n];
        z[a] = v;
    }
}

// The tile x[n0 .. n0 + cnt), up to N, zero-padded to a block (cnt a multiple of
// 64: a wave's 64 values are inside the tile or not together).
__device__ __forceinline__ void load_tile(float (&z)[R], const float *x, int64_t n0, int cnt, int64_t N, int t) {
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int c64 = cnt >> 6;
    const float *p = x + n0 + t;
    if (n0 + cnt <= N) {
#pragma unroll
        for (int a = 0; a < R; ++a) z[a] = 8 * a + w < c64 ? p[512 * a] : 0.f;
        return;
    }
#pragma unroll
    for (int a = 0; a < R; ++a) z[a] = (8 * a + w < c64 && n0 + 512 * a + t < N) ? p[512 * a] : 0.f;
}

// Memory V of the chain of an M-tap FIR and the cascade (M - 1 and the length of
// the cascade's response that the decay sums prove, rounded up to 64), or 0
// when the sums prove none up to FFT16_MEM.  By a whole wave, the same in each.
__device__ __forceinline__ int short_memory(const ShortTab *st, int32_t M, int lane) {
    const int j = lane & 3;
    const double lam = st->lam[j];
    double s = st->sum[lane >> 2][j];
#pragma unroll
    for (int d = 4; d < 64; d <<= 1) s += __shfl_xor(s, d);
    const double unit = __shfl(s, 0);
    // (false for a NaN, for an unstable cascade and for one with FP64 carry)
    float len = 1e9f;
    if (lam < 0.0 && unit < 1e300 && s < 1e300) {
        const float r = (float)(unit / s);
        if (r > 0.f) len = fmaxf((SHORT_LOG2_EPS + 0.5f * log2f(r)) / (float)lam, 0.f);
        else if (unit == 0.0) len = 0.f;
    }
#pragma unroll
    for (int d = 1; d < 4; d <<= 1) len = fminf(len, __shfl_xor(len, d));
    if (!(len <= (float)FFT16_MEM)) return 0;
    const int V = (M - 1 + (int)len + 1 + 63) & ~63;
    return __builtin_amdgcn_readfirstlane(V <= FFT16_MEM ? V : 0);
}

// Stores the block's values i in [lo, lo + cnt) to y[n0 + i - lo], up to N.
// lo and cnt are multiples of 64: a wave's 64 values are stored or not
// together (scalar tests).
__device__ __forceinline__ void store_block(const float (&z)[R], float *y, int64_t n0, int lo, int cnt, int64_t N,
                                            int t) {
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l64 = lo >> 6, c64 = cnt >> 6;
    float *p = y + (n0 - lo) + t;
    if (n0 + cnt <= N) {
#pragma unroll
        for (int a = 0; a < R; ++a)
            if ((unsigned)(8 * a + w - l64) < (unsigned)c64) p[512 * a] = z[a];
        return;
    }
#pragma unroll
    for (int a = 0; a < R; ++a)
        if ((unsigned)(8 * a + w - l64) < (unsigned)c64 && n0 - lo + 512 * a + t < N) p[512 * a] = z[a];
}

}  // namespace f16k
}  // namespace tfx
