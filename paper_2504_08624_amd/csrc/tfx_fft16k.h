// tfx_fft16k.h -- the 16384-point complex FFT of one 512-thread workgroup.
//
// 16384 = 32 x 32 x 16.  With n = 512 a + t (a < 32, t < 512), t = 16 b + c
// (b < 32, c < 16), k = k1 + 32 k2 + 1024 k3 (k1, k2 < 32, k3 < 16) and
// W = e^{-2 pi i / 16384}:
//   pass A  (thread t, over a):        32-point DFT
//   pass B  (thread (k1, c), over b):  * W^(16 b k1), 32-point DFT
//   pass C  (thread (k1, k2 mod 16), twice, over c): * W^(c (k1 + 32 k2)), 16-point DFT
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
// The transform is bound by its vector instructions, so twiddles stand where
// they cost least.  A product with e^{i phi} in front of a butterfly is two
// fused multiply-adds by tan phi; the left-over factor cos phi goes into the
// butterfly's own additions, which become fused multiply-adds (a radix-4
// butterfly with four twiddled inputs: 26 operations instead of 32).  That is
// how the constants inside the DFTs and pass B's table (in front of its 32-point
// DFT) are applied.  Pass C's row is formed once per block from four of its
// powers and serves both directions of a convolution.  With plain products
// behind every pass a convolution took 3275 operations per 32 values, now 2720;
// 64 x 5.76 M samples with 8191 taps: 1425 -> 1117 us.
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

// Twiddle table.  Rows r < 32 of 32 entries (padded to TWS float2: the 4 rows a
// wave reads lie 4 banks apart) for W^(16 r e), phi = 2 pi r e / 1024, in the
// form in which pass B's butterflies over e, e + 8, e + 16, e + 24 take them:
//   e < 8 and e = 16: (cos, sin);  8 <= e < 24: (tan, cos);  e >= 24: (tan, cos / cos of entry e - 16)
// Entry 16 of row 16 is the one quarter turn: that column takes plain products, whose
// two more operations a transform are 0.1 % (as a tangent it would be 2^28 or so and
// overflow sums from 1e30 on); the largest tangent left is 163, of 255 / 1024 of a turn.
// Behind them, per thread t, W^(m kappa), kappa = (t >> 4) + 32 (t & 15), m = 1, 2
// (first 512 float4) and m = 4, 8 (second).
constexpr int TWS = 34, TW_ROWS = 32;
constexpr int TW_LDS = TW_ROWS * TWS;           // float2 copied into LDS
constexpr int TW_FLOAT2 = TW_LDS + 4 * WGB;

// Bin k of the transform's output is value spec_j(k) of thread spec_t(k).
// Spectra are stored as pairs of bins per thread, [j / 2][t][j % 2].
__host__ __device__ constexpr int spec_t(int k) { return (k & 31) * 16 + ((k >> 5) & 15); }
__host__ __device__ constexpr int spec_j(int k) { return 16 * ((k >> 9) & 1) + (k >> 10); }
__host__ __device__ constexpr int spec_at(int k) { return ((spec_j(k) >> 1) * WGB + spec_t(k)) * 2 + (spec_j(k) & 1); }

// cos and tan of 2 pi k / 32
__device__ constexpr float c32[16] = {1.f, 0.98078528f, 0.923879533f, 0.831469612f, 0.707106781f, 0.555570233f, 0.382683432f, 0.195090322f, 0.f, -0.195090322f, -0.382683432f, -0.555570233f, -0.707106781f, -0.831469612f, -0.923879533f, -0.98078528f};
__device__ constexpr float t32[16] = {0.f, 0.198912367f, 0.414213562f, 0.668178638f, 1.f, 1.49660576f, 2.41421356f, 5.02733949f, 0.f, -5.02733949f, -2.41421356f, -1.49660576f, -1.f, -0.668178638f, -0.414213562f, -0.198912367f};

// x (1 -+ i t): a product with e^{SIGN i phi} over cos phi, t = tan phi
template <int SIGN>
__device__ __forceinline__ void turn(float &r, float &i, float t) {
    const float nr = SIGN < 0 ? fmaf(i, t, r) : fmaf(i, -t, r);
    i = SIGN < 0 ? fmaf(r, -t, i) : fmaf(r, t, i);
    r = nr;
}

// 4-point DFT of z0, e^{i phi_1} z1, e^{i phi_2} z2, e^{i phi_3} z3, where z1, z2,
// z3 have been turned: c1, c2 = cos phi_1, cos phi_2, q = cos phi_3 / cos phi_1.
template <int SIGN>
__device__ __forceinline__ void dft4_tw(float &r0, float &i0, float &r1, float &i1, float &r2, float &i2, float &r3,
                                        float &i3, float c1, float c2, float q) {
    const float ar = fmaf(c2, r2, r0), ai = fmaf(c2, i2, i0), br = fmaf(-c2, r2, r0), bi = fmaf(-c2, i2, i0);
    const float pr = fmaf(q, r3, r1), pi = fmaf(q, i3, i1), mr = fmaf(-q, r3, r1), mi = fmaf(-q, i3, i1);
    r0 = fmaf(c1, pr, ar);
    i0 = fmaf(c1, pi, ai);
    r2 = fmaf(-c1, pr, ar);
    i2 = fmaf(-c1, pi, ai);
    if (SIGN < 0) {  // b -+ i c1 m
        r1 = fmaf(c1, mi, br);
        i1 = fmaf(-c1, mr, bi);
        r3 = fmaf(-c1, mi, br);
        i3 = fmaf(c1, mr, bi);
    } else {
        r1 = fmaf(-c1, mi, br);
        i1 = fmaf(c1, mr, bi);
        r3 = fmaf(c1, mi, br);
        i3 = fmaf(-c1, mr, bi);
    }
}

// Second level of a 16-point DFT (element (k1, n2) at 4 k1 + n2 on entry,
// natural order on return).
template <int SIGN>
__device__ __forceinline__ void dft16_tail(float (&zr)[16], float (&zi)[16]) {
    constexpr float T8 = 0.41421356237309504880f, T38 = 2.41421356237309504880f;  // tan(pi / 8), tan(3 pi / 8)
    constexpr float C1 = c32[2], C2 = c32[4], C3 = c32[6];
    dft4<SIGN>(zr[0], zi[0], zr[1], zi[1], zr[2], zi[2], zr[3], zi[3]);
    turn<SIGN>(zr[5], zi[5], T8);
    turn<SIGN>(zr[6], zi[6], 1.f);
    turn<SIGN>(zr[7], zi[7], T38);
    dft4_tw<SIGN>(zr[4], zi[4], zr[5], zi[5], zr[6], zi[6], zr[7], zi[7], C1, C2, C3 / C1);
    {   // angles 2, 4 (a quarter turn: z2 -> -+ i z2), 6 sixteenths
        turn<SIGN>(zr[9], zi[9], 1.f);
        turn<SIGN>(zr[11], zi[11], -1.f);
        const float t = SIGN < 0 ? zi[10] : -zi[10], u = SIGN < 0 ? -zr[10] : zr[10];
        zr[10] = t;
        zi[10] = u;
        const float ar = zr[8] + zr[10], ai = zi[8] + zi[10], br = zr[8] - zr[10], bi = zi[8] - zi[10];
        const float pr = zr[9] - zr[11], pi = zi[9] - zi[11], mr = zr[9] + zr[11], mi = zi[9] + zi[11];
        zr[8] = fmaf(C2, pr, ar);
        zi[8] = fmaf(C2, pi, ai);
        zr[10] = fmaf(-C2, pr, ar);
        zi[10] = fmaf(-C2, pi, ai);
        zr[9] = SIGN < 0 ? fmaf(C2, mi, br) : fmaf(-C2, mi, br);
        zi[9] = SIGN < 0 ? fmaf(-C2, mr, bi) : fmaf(C2, mr, bi);
        zr[11] = SIGN < 0 ? fmaf(-C2, mi, br) : fmaf(C2, mi, br);
        zi[11] = SIGN < 0 ? fmaf(C2, mr, bi) : fmaf(-C2, mr, bi);
    }
    turn<SIGN>(zr[13], zi[13], T38);
    turn<SIGN>(zr[14], zi[14], -1.f);
    turn<SIGN>(zr[15], zi[15], T8);
    dft4_tw<SIGN>(zr[12], zi[12], zr[13], zi[13], zr[14], zi[14], zr[15], zi[15], C3, -C2, -C1 / C3);
    float tr[16], ti[16];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2) {
            tr[k1 + 4 * k2] = zr[4 * k1 + k2];
            ti[k1 + 4 * k2] = zi[4 * k1 + k2];
        }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        zr[k] = tr[k];
        zi[k] = ti[k];
    }
}

// In-register 16-point DFT, X_k = sum_n v_n e^{SIGN 2 pi i n k / 16}.
template <int SIGN>
__device__ __forceinline__ void dft16f(float (&zr)[16], float (&zi)[16]) {
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2)
        dft4<SIGN>(zr[n2], zi[n2], zr[4 + n2], zi[4 + n2], zr[8 + n2], zi[8 + n2], zr[12 + n2], zi[12 + n2]);
    dft16_tail<SIGN>(zr, zi);
}

// In-register 32-point DFT, X_k = sum_n v_n e^{SIGN 2 pi i n k / 32}: the 16-point
// DFTs of the even and odd values and one butterfly level.  TW: v_n is first
// multiplied by the twiddle row's entry n (its conjugate for SIGN > 0), the row's
// 16-byte pieces read from LDS as they are used.
template <int SIGN, bool TW>
__device__ __forceinline__ void dft32(float (&zr)[R], float (&zi)[R], const float2 *row) {
    float er[16], ei[16], qr[16], qi[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        er[m] = zr[2 * m];
        ei[m] = zi[2 * m];
        qr[m] = zr[2 * m + 1];
        qi[m] = zi[2 * m + 1];
    }
    if constexpr (TW) {
        const float4 *r4 = reinterpret_cast<const float4 *>(row);
#pragma unroll
        for (int n = 0; n < 4; ++n) {  // entries e = 2 n (even values) and 2 n + 1 (odd), e + 8, e + 16, e + 24
            const float4 w0 = r4[n], w1 = r4[n + 4], w2 = r4[n + 8], w3 = r4[n + 12];
            if (n > 0) cmul_tw<(SIGN < 0)>(er[n], ei[n], make_float2(w0.x, w0.y));
            cmul_tw<(SIGN < 0)>(qr[n], qi[n], make_float2(w0.z, w0.w));
            turn<SIGN>(er[4 + n], ei[4 + n], w1.x);
            if (n > 0) turn<SIGN>(er[8 + n], ei[8 + n], w2.x);
            else cmul_tw<(SIGN < 0)>(er[8], ei[8], make_float2(w2.x, w2.y));
            turn<SIGN>(er[12 + n], ei[12 + n], w3.x);
            dft4_tw<SIGN>(er[n], ei[n], er[4 + n], ei[4 + n], er[8 + n], ei[8 + n], er[12 + n], ei[12 + n], w1.y,
                          n > 0 ? w2.y : 1.f, w3.y);
            turn<SIGN>(qr[4 + n], qi[4 + n], w1.z);
            turn<SIGN>(qr[8 + n], qi[8 + n], w2.z);
            turn<SIGN>(qr[12 + n], qi[12 + n], w3.z);
            dft4_tw<SIGN>(qr[n], qi[n], qr[4 + n], qi[4 + n], qr[8 + n], qi[8 + n], qr[12 + n], qi[12 + n], w1.w, w2.w,
                          w3.w);
        }
        dft16_tail<SIGN>(er, ei);
        dft16_tail<SIGN>(qr, qi);
    } else {
        dft16f<SIGN>(er, ei);
        dft16f<SIGN>(qr, qi);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k == 0) {
            zr[k] = er[k] + qr[k];
            zi[k] = ei[k] + qi[k];
            zr[k + 16] = er[k] - qr[k];
            zi[k + 16] = ei[k] - qi[k];
        } else if (k == 8) {  // -+ i
            const float tr = SIGN < 0 ? qi[k] : -qi[k], ti = SIGN < 0 ? -qr[k] : qr[k];
            zr[k] = er[k] + tr;
            zi[k] = ei[k] + ti;
            zr[k + 16] = er[k] - tr;
            zi[k + 16] = ei[k] - ti;
        } else {
            turn<SIGN>(qr[k], qi[k], t32[k]);
            zr[k] = fmaf(c32[k], qr[k], er[k]);
            zi[k] = fmaf(c32[k], qi[k], ei[k]);
            zr[k + 16] = fmaf(-c32[k], qr[k], er[k]);
            zi[k + 16] = fmaf(-c32[k], qi[k], ei[k]);
        }
    }
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
    constexpr int N4 = TW_LDS / 2, P = (N4 + WGB - 1) / WGB;
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

// Pass C's twiddles W^(c kappa), c < 16, of half h (kappa + 512 h): from the
// thread's four powers (tw: the table in global memory), at most two products
// deep.
struct PowC {
    float2 u1, u2, u4, u8;
};
__device__ __forceinline__ float2 cmul2(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ PowC load_pow(const float2 *tw, int t) {
    const float4 *p = reinterpret_cast<const float4 *>(tw + TW_LDS) + t;
    const float4 a = p[0], b = p[WGB];
    return PowC{make_float2(a.x, a.y), make_float2(a.z, a.w), make_float2(b.x, b.y), make_float2(b.z, b.w)};
}
template <int H>
__device__ __forceinline__ void row_c(float2 (&w)[16], const PowC &p) {
    if constexpr (H == 0) {
        w[1] = p.u1;
        w[2] = p.u2;
        w[4] = p.u4;
        w[8] = p.u8;
    } else {  // times e^{-2 pi i c / 32}
        w[1] = cmul2(p.u1, make_float2(c32[1], -c32[7]));
        w[2] = cmul2(p.u2, make_float2(c32[2], -c32[6]));
        w[4] = make_float2(c32[4] * (p.u4.x + p.u4.y), c32[4] * (p.u4.y - p.u4.x));
        w[8] = make_float2(p.u8.y, -p.u8.x);
    }
    w[3] = cmul2(w[2], w[1]);
    w[5] = cmul2(w[4], w[1]);
    w[6] = cmul2(w[4], w[2]);
    w[7] = cmul2(w[4], w[3]);
    w[9] = cmul2(w[8], w[1]);
    w[10] = cmul2(w[8], w[2]);
    w[11] = cmul2(w[8], w[3]);
    w[12] = cmul2(w[8], w[4]);
    w[13] = cmul2(w[12], w[1]);
    w[14] = cmul2(w[12], w[2]);
    w[15] = cmul2(w[12], w[3]);
}
template <bool CONJ>
__device__ __forceinline__ void mul_row(float (&r)[16], float (&i)[16], const float2 (&w)[16]) {
#pragma unroll
    for (int c = 1; c < 16; ++c) cmul_tw<CONJ>(r[c], i[c], w[c]);
}
template <int H>
__device__ __forceinline__ void take_half(float (&a)[16], const float (&z)[R]) {
#pragma unroll
    for (int c = 0; c < 16; ++c) a[c] = z[16 * H + c];
}
template <int H>
__device__ __forceinline__ void put_half(float (&z)[R], const float (&a)[16]) {
#pragma unroll
    for (int c = 0; c < 16; ++c) z[16 * H + c] = a[c];
}

// a *= H, or conj(H) (sg < 0), for half h: the spectrum's pairs of bins in the
// thread's order, four loads at a time (registers; the lane index laundered per
// group so the next loads are not hoisted above the products).
template <int H>
__device__ __forceinline__ void spec_mul(float (&r)[16], float (&i)[16], const float2 *hs, int t, float sg) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float4 *h4 = reinterpret_cast<const float4 *>(hs) + opaque(t);
        float4 w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) w[g] = h4[(8 * H + 4 * q + g) * WGB];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int j = 8 * q + 2 * g;
            cmul_tw<false>(r[j], i[j], make_float2(w[g].x, sg * w[g].y));
            cmul_tw<false>(r[j + 1], i[j + 1], make_float2(w[g].z, sg * w[g].w));
            asm volatile("" : "+v"(r[j]), "+v"(i[j]), "+v"(r[j + 1]), "+v"(i[j + 1]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Passes A and B and the exchange in front of pass C.  In: thread t holds
// z[512 a + t] at a.  The caller has passed a barrier since the last access to P
// by another wave; ends with accesses to the wave's own rows only.
__device__ __forceinline__ void passes_ab(float (&zr)[R], float (&zi)[R], float *P, const float2 *twl, int t) {
    dft32<-1, false>(zr, zi, nullptr);
    put_cols(zr, P, opaque(t));
    __syncthreads();
    get_row(zr, P, opaque(t));
    __syncthreads();
    put_cols(zi, P, opaque(t));
    __syncthreads();
    get_row(zi, P, opaque(t));
    dft32<-1, true>(zr, zi, twl + (opaque(t) >> 4) * TWS);
    wave_fence();
    b_to_c(zr, P, opaque(t));
    b_to_c(zi, P, opaque(t));
}

// The inverse passes behind pass C's: starts on the wave's own rows of P (no
// barrier needed after passes_ab), ends with reads of every row.
__device__ __forceinline__ void passes_ba(float (&zr)[R], float (&zi)[R], float *P, const float2 *twl, int t) {
    c_to_b(zr, P, opaque(t));
    c_to_b(zi, P, opaque(t));
    dft32<1, false>(zr, zi, nullptr);
    put_row(zr, P, opaque(t));
    __syncthreads();
    get_cols(zr, P, opaque(t));
    __syncthreads();
    put_row(zi, P, opaque(t));
    __syncthreads();
    get_cols(zi, P, opaque(t));
    dft32<1, true>(zr, zi, twl + (opaque(t) >> 4) * TWS);
}

template <int H, bool FWD, bool INV>
__device__ __forceinline__ void pass_c(float (&zr)[R], float (&zi)[R], const PowC &p, const float2 *hs, int t, float sg) {
    float2 w[16];
    float r[16], i[16];
    row_c<H>(w, p);
    take_half<H>(r, zr);
    take_half<H>(i, zi);
    if constexpr (FWD) {
        mul_row<false>(r, i, w);
        dft16f<-1>(r, i);
    }
    if constexpr (INV) {
        spec_mul<H>(r, i, hs, t, sg);
        dft16f<1>(r, i);
        mul_row<true>(r, i, w);
    }
    put_half<H>(zr, r);
    put_half<H>(zi, i);
}

// Forward transform.  In: thread t holds z[512 a + t] at a.  Out: bin
// k1 + 32 (t & 15) + 512 h + 1024 k3 (k1 = t >> 4) at 16 h + k3.  (Barriers as in
// passes_ab; twl: the rows in LDS, tw: the whole table.)
__device__ __forceinline__ void forward(float (&zr)[R], float (&zi)[R], float *P, const float2 *twl, const float2 *tw,
                                        int t) {
    passes_ab(zr, zi, P, twl, t);
    const PowC p = load_pow(tw, opaque(t));
    pass_c<0, true, false>(zr, zi, p, nullptr, t, 0.f);
    pass_c<1, true, false>(zr, zi, p, nullptr, t, 0.f);
}

// z <- inverse transform (without 1/16384) of H z, or conj(H) z (sg < 0), from
// forward's output layout back to its input layout.
__device__ __forceinline__ void product_inverse(float (&zr)[R], float (&zi)[R], const float2 *hs, float sg, float *P,
                                                const float2 *twl, const float2 *tw, int t) {
    const PowC p = load_pow(tw, opaque(t));
    pass_c<0, false, true>(zr, zi, p, hs, t, sg);
    pass_c<1, false, true>(zr, zi, p, hs, t, sg);
    passes_ba(zr, zi, P, twl, t);
}

// Circular convolution with the spectrum hs (/ 16384), or correlation (sg < 0).
__device__ __forceinline__ void convolve(float (&zr)[R], float (&zi)[R], const float2 *hs, float sg, float *P,
                                         const float2 *twl, const float2 *tw, int t) {
    passes_ab(zr, zi, P, twl, t);
    const PowC p = load_pow(tw, opaque(t));
    pass_c<0, true, true>(zr, zi, p, hs, t, sg);
    pass_c<1, true, true>(zr, zi, p, hs, t, sg);
    passes_ba(zr, zi, P, twl, t);
}

// Unit u of nu (a pair of neighbouring tiles, see TilePair) of block id i:
// the blocks of one XCD (block i runs on XCD i mod 8) take one contiguous
// range of units, so tiles that share input are read through one L2.
__device__ __forceinline__ uint32_t xcd_unit(uint32_t i, uint32_t nu) {
    const uint32_t x = i & 7u, per = nu >> 3, rem = nu & 7u;
    return __builtin_amdgcn_readfirstlane(x * per + (x < rem ? x : rem) + (i >> 3));
}

// The two tiles of unit u, with tpc tiles of T samples a row: neighbours in one
// channel (the second may be missing), so that no channel's rounding reaches
// another; where rows are one tile and many, those of two channels, as half of
// every transform would be empty (4096 x 4096 samples, 8191 taps: 185 us with a
// channel a unit, 118 us so; a chain on 256 x 12000 has a CU for every row: 32.8
// and 34.4).  two: there is a second tile.
struct TilePair {
    int64_t chA, nA, chB, nB;
    bool two;
};
__device__ __forceinline__ TilePair tile_pair(uint32_t u, uint32_t C, uint32_t tpc, int T) {
    const bool rows = rows_paired(C, tpc);
    const uint32_t per = (tpc + 1) / 2, c = __builtin_amdgcn_readfirstlane(rows ? 2 * u : u / per);
    const uint32_t i = rows ? 0 : 2 * (u - c * per);
    TilePair p;
    p.two = rows ? c + 1 < C : i + 1 < tpc;
    p.chA = c;
    p.nA = (int64_t)i * T;
    p.chB = rows && p.two ? c + 1 : c;
    p.nB = rows ? 0 : p.nA + T;
    return p;
}
// tpc of a row of N < 2^38 samples (T is a multiple of 64), in scalar registers
__device__ __forceinline__ uint32_t tiles_per_row(int64_t N, int T) {
    const uint32_t t64 = (uint32_t)T >> 6;
    return __builtin_amdgcn_readfirstlane(((uint32_t)((N + 63) >> 6) + t64 - 1) / t64);
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
