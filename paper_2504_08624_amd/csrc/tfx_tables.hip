// tfx_tables.hip -- the prepare step: per-section scan tables, FFT twiddles and
// tap spectrum, merged taps, workspace initialisation.  Everything is formed
// in FP64 from the fp32 coefficients the filter kernel will see, and rounded
// once.  These kernels run once per (workspace, coefficients); the filter
// kernel (tfx_chain.hip) only reads what they leave in the workspace.
#include <hip/hip_runtime.h>

#include "tfx_fft16k.h"
#include "tfx_internal.h"

namespace tfx {

// The table builders below run one per block, in one kernel: each lays its
// arrays over the block's one LDS buffer.
constexpr int PREP_LDS = 20 * 1024;
template <class Sh>
__device__ __forceinline__ Sh &lds_as(char *raw) {
    static_assert(sizeof(Sh) <= PREP_LDS, "fits the block's LDS buffer");
    return *reinterpret_cast<Sh *>(raw);
}

__device__ void mat2_mul(const double *A, const double *B, double *C) {
    const double c0 = A[0] * B[0] + A[1] * B[2];
    const double c1 = A[0] * B[1] + A[1] * B[3];
    const double c2 = A[2] * B[0] + A[3] * B[2];
    const double c3 = A[2] * B[1] + A[3] * B[3];
    C[0] = c0;
    C[1] = c1;
    C[2] = c2;
    C[3] = c3;
}

__device__ void put4(float *f, double *d, const double *m) {
    for (int i = 0; i < 4; ++i) {
        f[i] = (float)m[i];
        if (d) d[i] = m[i];
    }
}

// R = A^e (FP64 2 x 2) by binary powering; R may alias nothing.
__device__ void mat2_pow(const double *A, int e, double *R) {
    double P[4] = {A[0], A[1], A[2], A[3]};
    R[0] = 1.0;
    R[1] = 0.0;
    R[2] = 0.0;
    R[3] = 1.0;
    while (e > 0) {
        if (e & 1) mat2_mul(R, P, R);
        e >>= 1;
        if (e > 0) mat2_mul(P, P, P);
    }
}

__device__ double mat2_maxabs(const double *M) {
    return fmax(fmax(fabs(M[0]), fabs(M[1])), fmax(fabs(M[2]), fabs(M[3])));
}

// Transition powers of one TDF-II section, built by one block of 256
// threads.  With state s = (s1, s2) the section is s' = A s + B x,
// y = s1 + b0 x, A = [[-a1, 1], [-a2, 0]], so a state s entering a chunk
// becomes Phi s = A^Lc s after Lc samples.  Thread k < 64 writes the fold
// power Phi^k, thread j < 9 the look-back power W^(2^j) of the tile
// transition W = Phi^128, and threads k < 64 test W^(k+1) for the look-back
// depth (the first d <= 64 with max |W^d| <= 2^-60, 0 if none).  Every power
// is formed by binary powering in FP64 and rounded once.
__device__ void build_section_block(SecTab *tb, const float *co, int Lc, int tid) {
    __shared__ int s_dep;
    const double a1 = co[3], a2 = co[4];
    const double A[4] = {-a1, 1.0, -a2, 0.0};
    double Phi[4], Psi[4], W[4], R[4];
    mat2_pow(A, Lc, Phi);
    mat2_pow(Phi, 64, Psi);
    mat2_pow(Psi, GWAVES, W);
    if (tid == 0) s_dep = 65;
    const bool hiq = section_hiq(a1, a2);
    __syncthreads();
    // a wave each: the folds; the look-back depth; psi and lb; the zero-input response
    const int wv = tid >> 6, l = tid & 63;
    if (wv == 0) {
        mat2_pow(Phi, l, R);
        for (int q = 0; q < 4; ++q) tb->fold[l][q] = (float)R[q];
        if (hiq)
            for (int q = 0; q < 4; ++q) tb->fold_d[l][q] = R[q];
    } else if (wv == 1) {
        mat2_pow(W, l + 1, R);
        if (mat2_maxabs(R) <= DEPTH_EPS) atomicMin(&s_dep, l + 1);
    } else if (wv == 2) {
        if (l < GWAVES) {
            mat2_pow(Psi, l, R);
            put4(tb->psi[l], tb->psi_d[l], R);
        }
        if (l < 9) {
            mat2_pow(W, 1 << l, R);
            put4(tb->lb[l], tb->lb_d[l], R);
        }
    } else if (l < 32 && !hiq) {
        mat2_pow(A, l, R);
        tb->zir[l] = (float)R[0];
    }
    __syncthreads();
    if (tid == 0) {
        for (int i = 0; i < 5; ++i) tb->coef[i] = co[i];
        tb->pad = 0;
        tb->depth = s_dep > 64 ? 0 : s_dep;
        tb->hiq = hiq ? 1 : 0;
    }
}

// Element (i, j) of the cascade's one-sample transition F under zero input
// (D = 2S state components, section s at 2s, 2s + 1): block (s, s) is the
// section's A; block (s, t), t < s, is B_s (prod_{t<l<s} b0_l) C, since
// section s's input is section s-1's output.
__device__ double cascade_f(const double (*co)[5], int D, int i, int j) {
    if (i >= D || j >= D) return 0.0;
    const int si = i >> 1, ri = i & 1, sj = j >> 1, cj = j & 1;
    const double b0 = co[si][0], b1 = co[si][1], b2 = co[si][2], a1 = co[si][3], a2 = co[si][4];
    if (si == sj) return ri == 0 ? (cj == 0 ? -a1 : 1.0) : (cj == 0 ? -a2 : 0.0);
    if (sj < si && cj == 0) {
        double pr = ri == 0 ? b1 - a1 * b0 : b2 - a2 * b0;
        for (int l = sj + 1; l < si; ++l) pr *= co[l][0];
        return pr;
    }
    return 0.0;
}

// Tile-transition powers of the whole cascade for the cascade-level
// look-back, in FP64, by one block of 256 threads (one matrix element
// each).  The cascade's one-sample transition F (zero input): block (i, i) =
// A_i; block (i, j), j < i = B_i (prod_{j<l<i} D_l) C, since section i's
// input is section i-1's output; Phi_T = F^(128 Lc) = (F^Lc)^128.
// A block's time is these products one after another, and a product's is its
// reads of LDS: only the first D of 16 rows and columns hold anything, and A's
// row comes two values a read (101 taps and 2 sections: prepare 9.6 us with all
// 16, one value a read and the section's powers in turn, 6.9 us so; 6 sections
// whose depth is searched for to the end: 13.6 and 12.9).
template <int D>
__device__ __forceinline__ double mm_dot_n(const double (*A)[16], const double (*B)[16], int i, int j) {
    double2 r[D / 2];
    double b[D];
#pragma unroll
    for (int k = 0; k < D / 2; ++k) r[k] = reinterpret_cast<const double2 *>(A[i])[k];
#pragma unroll
    for (int k = 0; k < D; ++k) b[k] = B[k][j];
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k) acc += (k & 1 ? r[k / 2].y : r[k / 2].x) * b[k];
    return acc;
}
__device__ __forceinline__ double mm_dot(const double (*A)[16], const double (*B)[16], int i, int j, int D) {
    if (D <= 4) return mm_dot_n<4>(A, B, i, j);
    if (D <= 8) return mm_dot_n<8>(A, B, i, j);
    if (D <= 12) return mm_dot_n<12>(A, B, i, j);
    return mm_dot_n<16>(A, B, i, j);
}
__device__ void mm16(const double (*A)[16], const double (*B)[16], double (*R)[16], int i, int j, int D) {
    const double acc = mm_dot(A, B, i, j, D);
    __syncthreads();  // every read of A and B done (R may alias either)
    R[i][j] = acc;
    __syncthreads();
}
// P = P F (if mul) and F = F F in one round
__device__ void mm16_step(double (*P)[16], double (*F)[16], bool mul, int i, int j, int D) {
    const double p = mul ? mm_dot(P, F, i, j, D) : 0.0, f = mm_dot(F, F, i, j, D);
    __syncthreads();
    if (mul) P[i][j] = p;
    F[i][j] = f;
    __syncthreads();
}

// Whether max |M| over the block is within the depth bound (every thread gets it).
__device__ bool block_within(double m) { return __syncthreads_and(fabs(m) <= DEPTH_EPS) != 0; }

// co(s, k): coefficient k of section s; Lc: the chunk length (tile 128 Lc).
template <class Co>
__device__ void casc_table_block(char *raw, Co co_at, int32_t S, int Lc, CascTab *out, int tid) {
    struct Sh {
        alignas(16) double M0[16][16], M1[16][16], Pw[7][16][16], co[CASC_MAX][5];
    };
    Sh &sh = lds_as<Sh>(raw);
    auto &co = sh.co;
    auto &M0 = sh.M0, &M1 = sh.M1;
    auto &Pw = sh.Pw;
    const int i = tid >> 4, j = tid & 15, D = 2 * S;
    if (tid < S * 5) co[tid / 5][tid % 5] = co_at(tid / 5, tid % 5);
    __syncthreads();
    M1[i][j] = cascade_f(co, D, i, j);
    Pw[0][i][j] = i == j ? 1.0 : 0.0;
    __syncthreads();
    for (int e = Lc; e > 0; e >>= 1) {  // Pw[0] = F^Lc by binary powering
        if (e > 1) mm16_step(Pw[0], M1, e & 1, i, j, D);
        else mm16(Pw[0], M1, Pw[0], i, j, D);
    }
    for (int t = 0; t < 7; ++t) mm16(Pw[0], Pw[0], Pw[0], i, j, D);  // F^(128 Lc), the tile transition
    for (int t = 1; t < 7; ++t) mm16(Pw[t - 1], Pw[t - 1], Pw[t], i, j, D);  // Phi_T^(2^t)
    out->T[0][i][j] = (float)Pw[0][i][j];
    out->T[1][i][j] = (float)Pw[1][i][j];
    out->T[2][i][j] = (float)Pw[2][i][j];
    // look-back depth: a d <= 64 with max |Phi_T^d| <= 2^-60 (0 if none),
    // found by doubling, then bisection between the last failing power of
    // two and the first passing one; every accepted d is checked directly
    int first = -1;
    for (int t = 0; t < 7 && first < 0; ++t)
        if (block_within(Pw[t][i][j])) first = t;
    int dep = 0;
    if (first == 0) {
        dep = 1;
    } else if (first > 0) {
        int lo = 1 << (first - 1), hi = 1 << first;
        M0[i][j] = Pw[first - 1][i][j];  // Phi_T^lo
        __syncthreads();
        for (int t = first - 2; t >= 0; --t) {
            mm16(M0, Pw[t], M1, i, j, D);  // Phi_T^(lo + 2^t)
            if (block_within(M1[i][j])) {
                hi = lo + (1 << t);
            } else {
                lo += 1 << t;
                M0[i][j] = M1[i][j];
                __syncthreads();
            }
        }
        dep = hi;
    }
    if (tid == 0) out->depth = dep;
}

// Zero-input response tables of the cascade (CascZir), in FP64 then
// rounded, one block of 256 threads (one matrix element each) per entry:
// k < ZIR_B gives F^(Lc k), ZIR_B <= k < ZIR_B + ZIR_A gives F^(16 Lc a),
// a = k - ZIR_B, by binary powering; k == ZIR_B + ZIR_A gives the output rows
// G[r] = c F^r, r < Lc, where c[2s] = prod_{t>s} b0_t (the s1 register of
// section s reaches the output through the b0 of every later section) and
// c[2s+1] = 0.
template <class Co>
__device__ void zir_block(char *raw, Co co_at, int32_t S, int Lc, int k, CascZir *out, int tid) {
    struct Sh {
        alignas(16) double Fm[16][16], P[16][16], G[32][16], co[CASC_MAX][5];
    };
    Sh &sh = lds_as<Sh>(raw);
    auto &co = sh.co;
    auto &Fm = sh.Fm, &P = sh.P;
    auto &G = sh.G;
    const int i = tid >> 4, j = tid & 15;
    if (tid < S * 5) co[tid / 5][tid % 5] = co_at(tid / 5, tid % 5);
    __syncthreads();
    const int D = 2 * S;
    Fm[i][j] = cascade_f(co, D, i, j);
    P[i][j] = i == j ? 1.0 : 0.0;
    __syncthreads();
    if (k < ZIR_B + ZIR_A) {
        const int e0 = k < ZIR_B ? Lc * k : ZIR_B * Lc * (k - ZIR_B);
        for (int e = e0; e > 0; e >>= 1) {
            if (e > 1) mm16_step(P, Fm, e & 1, i, j, D);
            else mm16(P, Fm, P, i, j, D);
        }
        if (k < ZIR_B) out->Mb[i][j][k] = (float)P[i][j];
        else out->MaT[k - ZIR_B][j][i] = (float)P[i][j];
        return;
    }
    if (tid < 16) {
        double c = 0.0;
        if (tid < D && (tid & 1) == 0) {
            c = 1.0;
            for (int t = (tid >> 1) + 1; t < S; ++t) c *= co[t][0];
        }
        G[0][tid] = c;
    }
    __syncthreads();
    for (int m = 1; m < Lc; m *= 2) {  // rows m .. 2 m - 1 are rows 0 .. m - 1 times F^m
        const double acc = i < m ? mm_dot(G, Fm, i, j, D) : 0.0, f = mm_dot(Fm, Fm, i, j, D);
        __syncthreads();
        if (i < m) G[m + i][j] = acc;
        Fm[i][j] = f;
        __syncthreads();
    }
    for (int e = tid; e < 16 * Lc; e += 256) out->G[e & 15][e >> 4] = (float)G[e >> 4][e & 15];
}

// Matrix-core cascade tables (McTab), in FP64 then rounded, one block of
// 256 threads: the chunk's impulse response h, the input columns F^m b, the
// output rows c F^r, the chunk transition Fc = F^32 and the segment
// transition Fc^12, each laid out as the kernel's operands.
template <class Co>
__device__ void mc_block(char *raw, Co co_at, int32_t S, McTab *out, int tid) {
    struct Sh {
        double co[CASC_MAX][5], Pw[16][16], Q[16][16];
        double V[MC_LC][16];   // F^m b
        double Gm[MC_LC][16];  // c F^r
        double hh[MC_LC];
    };
    Sh &sh = lds_as<Sh>(raw);
    auto &co = sh.co;
    auto &Pw = sh.Pw, &Q = sh.Q;
    auto &V = sh.V, &Gm = sh.Gm;
    auto &hh = sh.hh;
    const int i = tid >> 4, j = tid & 15;
    if (tid < S * 5) co[tid / 5][tid % 5] = co_at(tid / 5, tid % 5);
    __syncthreads();
    const int D = 2 * S;
    Pw[i][j] = cascade_f(co, D, i, j);
    if (tid < 16) {
        // b: section s sees the input through the b0 of every earlier
        // section; c: the s1 register of section s reaches the output
        // through the b0 of every later one
        double bb = 0.0, cc = 0.0;
        if (tid < D) {
            const int sc = tid >> 1;
            double g = 1.0;
            for (int l = 0; l < sc; ++l) g *= co[l][0];
            bb = ((tid & 1) ? co[sc][2] - co[sc][4] * co[sc][0] : co[sc][1] - co[sc][3] * co[sc][0]) * g;
            if ((tid & 1) == 0) {
                cc = 1.0;
                for (int t = sc + 1; t < S; ++t) cc *= co[t][0];
            }
        }
        V[0][tid] = bb;
        Gm[0][tid] = cc;
    }
    __syncthreads();
    // doubling: with Pw = F^(2^l), V[2^l + v] = Pw V[v] and
    // Gm[2^l + v] = Gm[v] Pw for v < 2^l (thread (i, j): component i of
    // vector j), then Pw <- Pw^2; five levels give 32 vectors and Pw = F^32
    for (int l = 0; l < 5; ++l) {
        const int n = 1 << l;
        double vv = 0.0, gg = 0.0;
        if (j < n) {
            for (int k = 0; k < 16; ++k) {
                vv += Pw[i][k] * V[j][k];
                gg += Gm[j][k] * Pw[k][i];
            }
        }
        __syncthreads();
        if (j < n) {
            V[n + j][i] = vv;
            Gm[n + j][i] = gg;
        }
        mm16(Pw, Pw, Pw, i, j, 2 * S);
    }
    if (tid < MC_LC) {  // h[0] = d, h[n] = c F^(n-1) b
        double hv = 0.0;
        if (tid == 0) {
            hv = S > 0 ? 1.0 : 0.0;
            for (int l = 0; l < S; ++l) hv *= co[l][0];
        } else {
            for (int k = 0; k < 16; ++k) hv += Gm[tid - 1][k] * V[0][k];
        }
        hh[tid] = hv;
    }
    __syncthreads();
    for (int e = tid; e < 64 * 24; e += 256) {
        const int l = e / 24, q = e % 24, rb = q / 8, t = q % 8;
        const int row = 16 * rb + (l & 15), m = 8 * (l >> 4) + t;
        double v;
        if (row < MC_LC) v = row >= m ? hh[row - m] : 0.0;
        else v = V[MC_LC - 1 - m][row - MC_LC];  // H[:, m] = F^(31 - m) b
        out->W[l][q] = (float)v;
    }
    for (int e = tid; e < 64 * 8; e += 256) {
        const int l = e / 8, q = e % 8, rb = q / 4, k = q % 4;
        out->Gt[l][q] = (float)Gm[16 * rb + (l & 15)][4 * (l >> 4) + k];
    }
    out->Fr[i][j] = (float)Pw[i][mc_src(i, j)];  // Fc = F^32
    mm16(Pw, Pw, Q, i, j, 2 * S);  // Fc^2
    mm16(Q, Q, Q, i, j, 2 * S);    // Fc^4
    mm16(Q, Q, Pw, i, j, 2 * S);   // Fc^8
    mm16(Pw, Q, Q, i, j, 2 * S);   // Fc^12
    out->Fsr[i][j] = (float)Q[i][mc_src(i, j)];
}

struct MergeArgs {
    StageList firs;
    double *buf0, *buf1;
    float *out;
};

// Convolves the tap vectors of several FIR stages into one (FP64, one block).
__global__ void merge_taps_kernel(MergeArgs a) {
    int Mcur = a.firs.len[0];
    for (int k = threadIdx.x; k < Mcur; k += blockDim.x) a.buf0[k] = a.firs.ptr[0][k];
    __syncthreads();
    double *cur = a.buf0, *nxt = a.buf1;
    for (int st = 1; st < a.firs.n; ++st) {
        const int Mi = a.firs.len[st];
        const float *hi = a.firs.ptr[st];
        const int Mn = Mcur + Mi - 1;
        for (int k = threadIdx.x; k < Mn; k += blockDim.x) {
            const int jlo = k - Mi + 1 > 0 ? k - Mi + 1 : 0;
            const int jhi = k < Mcur - 1 ? k : Mcur - 1;
            double acc = 0.0;
            for (int j = jlo; j <= jhi; ++j) acc += cur[j] * (double)hi[k - j];
            nxt[k] = acc;
        }
        __syncthreads();
        double *t = cur;
        cur = nxt;
        nxt = t;
        Mcur = Mn;
    }
    for (int k = threadIdx.x; k < Mcur; k += blockDim.x) a.out[k] = (float)cur[k];
}

// Entry i of the twiddle tables (i < 4096), each e^{-2 pi i e / 4096} for an
// exact integer e mod 4096, in FP64 and rounded once: tw64[i] (e = i) and,
// for i < TWL_ENTRIES, the padded fp32 table TWL of the FFT kernels.
__device__ void write_twiddle(float2 *twid, double2 *tw64, int i) {
    double sn, cs;
    sincospi(-2.0 * (double)i / NFFT, &sn, &cs);
    tw64[i] = make_double2(cs, sn);
    if (i < TWL_ENTRIES) {  // TWL[r][k]: e = 16 r k (r < 16), (r - 16) k; pads zero
        const int r = i / TWL_S, k = i % TWL_S;
        const int eL = ((r < 16 ? 16 * r : r - 16) * k) & (NFFT - 1);
        sincospi(-2.0 * (double)eL / NFFT, &sn, &cs);
        twid[i] = k < 16 ? make_float2((float)cs, (float)sn) : make_float2(0.f, 0.f);
    }
}

__global__ void fft_twiddle_kernel(float2 *twid, double2 *tw64) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < NFFT) write_twiddle(twid, tw64, k);
}

// hspec[p][k] = (sum_j h[1025 p + j] e^{-2 pi i j k / 4096}) / 4096, the DFT
// of tap partition p (j < 1025, zero-padded), in FP64, stored in the FFT
// kernels' per-lane order (bin t + 256 k3 at [t][k3]).  One block of 256
// lanes covers 16 bins: lane (kk, jj) sums taps j = jj (mod 16) of bin
// k = 16 blk + kk, stepping its twiddle by e^{-2 pi i 16 k / 4096} (at most
// 65 steps from an exact start, so the FP64 twiddle error stays near
// 1e-14, far below the fp32 rounding of the result); the 16 partial sums
// are added by a fixed shuffle tree.
__device__ void spectrum_block(char *raw, const float *h_all, int32_t M_all, int part, int blk, float2 *hspec_all,
                               int tid) {
    struct Sh {
        float hs[FFT_PART + 15];
    };
    auto &hs = lds_as<Sh>(raw).hs;
    const int kk = tid >> 4, jj = tid & 15;
    const int k = blk * 16 + kk;
    const float *h = h_all + (int64_t)part * FFT_PART;
    const int rest = M_all - part * FFT_PART;
    const int M = rest < FFT_PART ? rest : FFT_PART;
    for (int j = tid; j < FFT_PART + 15; j += 256) hs[j] = j < M ? h[j] : 0.f;  // zero-padded to 16 | length
    __syncthreads();
    double wr, wi, sr, si;
    sincospi(-2.0 * (double)((jj * k) & (NFFT - 1)) / NFFT, &wi, &wr);
    sincospi(-2.0 * (double)((16 * k) & (NFFT - 1)) / NFFT, &si, &sr);
    double hr = 0.0, hi = 0.0;
#pragma unroll 5
    for (int m = 0; m < (FFT_PART + 15) / 16; ++m) {
        const double hv = (double)hs[jj + 16 * m];
        hr = fma(hv, wr, hr);
        hi = fma(hv, wi, hi);
        const double nr = wr * sr - wi * si;
        wi = fma(wr, si, wi * sr);
        wr = nr;
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
        hr += __shfl_xor(hr, d);
        hi += __shfl_xor(hi, d);
    }
    if (jj == 0)  // per-lane layout: bin t + 256 k3 at [t][k3]
        hspec_all[(int64_t)part * NFFT + 16 * (k & 255) + (k >> 8)] = make_float2((float)(hr / NFFT), (float)(hi / NFFT));
}

// Spectra of the 16384-point path, in FP64 and rounded once, each / 16384 in
// the transform's output order: the taps' (hs), and the taps' times the
// cascade's (ht); with hf the taps' spectrum also stays in FP64 (bin k at
// hf[k], unscaled).  With n = 128 n1 + n2 and k = k1 + 128 k2, block k1 forms
// A[n2] = W^(n2 k1) sum_n1 h[n] W_128^(n1 k1) and from it its 128 bins
// sum_n2 A[n2] W_128^(n2 k2), two threads a bin; everything is real in time, so
// blocks k1 <= 64 give the others' bins as conjugates.  The first blocks also
// write the twiddle rows.  (A direct sum per bin took 29 us of a prepare with
// 1023 taps, one workgroup's fp32 transform 17; this form takes none of its
// critical path.)
constexpr int SPEC16_BLOCKS = 65;
static_assert(SPEC16_BLOCKS * 256 >= f16k::TW_FLOAT2, "the spectrum blocks cover the twiddle rows");
__device__ __forceinline__ double2 cmul64(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
template <class Co>
__device__ void spec16_block(char *raw, const float *h, int32_t M, int32_t cmp, Co co_at, int32_t S, int k1, float2 *tw,
                             float2 *hs, float2 *ht, double2 *hf, int tid) {
    constexpr int NB = FFT16_POINTS;
    struct Sh {
        double2 w128[128], wq[128], A[128], part[128];
        double cs[CASC_MAX][5];
    };
    Sh &sh = lds_as<Sh>(raw);
    auto &w128 = sh.w128, &wq = sh.wq, &A = sh.A, &part = sh.part;
    auto &cs = sh.cs;
    const int q = tid & 127, hf2 = tid >> 7;
    if (ht && tid < S * 5) cs[tid / 5][tid % 5] = co_at(tid / 5, tid % 5);
    // W_128^q (threads < 128), W^(q k1) (the others), then the twiddle table's
    // entry: one loop, so that the sine's code is there once
    const int i = k1 * 256 + tid;
    int role = -1, m1 = 0, m2 = 0;  // entry's form (-1: none), its angle, the angle of the cosine it is divided by
    if (i < f16k::TW_LDS) {
        const int row = i / f16k::TWS, e = i % f16k::TWS;
        role = e == 16 ? 0 : e < f16k::R ? e >> 3 : 4;
        m1 = 16 * row * e;
        m2 = 16 * row * (e - 16);
    } else if (i < f16k::TW_FLOAT2) {  // float4 of thread t: m = 1, 2, or 4, 8
        const int f = i - f16k::TW_LDS, t = (f >> 1) & (f16k::WGB - 1);
        role = 5;
        m1 = ((t >> 4) + 32 * (t & 15)) << (2 * (f >> 10) + (f & 1));
    }
    double c1 = 0.0, s1 = 0.0;
#pragma unroll 1
    for (int r = 0; r < (role < 0 ? 1 : role == 3 ? 3 : 2); ++r) {
        const int m = r == 0 ? (hf2 == 0 ? 128 * q : q * k1) : r == 1 ? m1 : m2;
        double s, c;
        sincospi(-2.0 * (double)(m & (NB - 1)) / NB, &s, &c);
        if (r == 0) {
            (hf2 == 0 ? w128 : wq)[q] = make_double2(c, s);
            continue;
        }
        if (r == 1) {
            c1 = c;
            s1 = -s;
            const float2 v = role == 0 ? make_float2((float)c, (float)-s)
                           : role == 4 ? make_float2(0.f, 0.f)
                           : role == 5 ? make_float2((float)c, (float)s) : make_float2((float)(-s / c), (float)c);
            if (role != 3) tw[i] = v;
        } else {
            tw[i] = make_float2((float)(s1 / c1), (float)(c1 / c));
        }
    }
    __syncthreads();
    double2 acc = make_double2(0.0, 0.0);
    const int n1s = (M + 127) / 128;
#pragma unroll 4
    for (int n1 = hf2; n1 < n1s; n1 += 2) {
        const int n = 128 * n1 + q;
        float hq = h[min(n, M - 1)];
        hq = cmp == TFX_COMPUTE_BF16 ? (float)(__bf16)hq : cmp == TFX_COMPUTE_F16 ? (float)(_Float16)hq : hq;
        const double hv = n < M ? (double)hq : 0.0;
        const double2 w = w128[(n1 * k1) & 127];
        acc.x = fma(hv, w.x, acc.x);
        acc.y = fma(hv, w.y, acc.y);
    }
    if (hf2 == 1) part[q] = acc;
    __syncthreads();
    if (hf2 == 0) A[q] = cmul64(make_double2(acc.x + part[q].x, acc.y + part[q].y), wq[q]);
    __syncthreads();
    const double2 step = w128[q];
    double2 w = w128[(64 * hf2 * q) & 127];
    acc = make_double2(0.0, 0.0);
#pragma unroll 2
    for (int n2 = 64 * hf2; n2 < 64 * hf2 + 64; ++n2) {
        const double2 a = A[n2];
        acc.x = fma(a.x, w.x, fma(-a.y, w.y, acc.x));
        acc.y = fma(a.x, w.y, fma(a.y, w.x, acc.y));
        w = cmul64(w, step);
    }
    if (hf2 == 1) part[q] = acc;
    __syncthreads();
    const int k = k1 + 128 * q;
    if (hf2 == 0) acc = make_double2(acc.x + part[q].x, acc.y + part[q].y);
    double2 g = make_double2(1.0, 0.0);
    if (ht) {  // sections hf2, hf2 + 2, ...: (b0 + z (b1 + z b2)) / (1 + z (a1 + z a2))
        const double2 zz = cmul64(wq[1], w128[q]);  // W^k
#pragma unroll 1
        for (int s = hf2; s < S; s += 2) {
            const double *c = cs[s];
            double2 u = cmul64(make_double2(c[1] + zz.x * c[2], zz.y * c[2]), zz);
            double2 v = cmul64(make_double2(c[3] + zz.x * c[4], zz.y * c[4]), zz);
            u.x += c[0];
            v.x += 1.0;
            const double r = 1.0 / fma(v.x, v.x, v.y * v.y);
            u = cmul64(u, make_double2(v.x, -v.y));
            g = cmul64(g, make_double2(u.x * r, u.y * r));
        }
        __syncthreads();
        if (hf2 == 1) part[q] = g;
        __syncthreads();
        if (hf2 == 0) g = cmul64(g, part[q]);
    }
    // blocks 0 and 64 hold both a bin and its mirror image: the lower one counts
    if (hf2 == 1 || (k1 == 0 && q > 64) || (k1 == 64 && q > 63)) return;
    const int km = (NB - k) & (NB - 1), at = f16k::spec_at(k), am = f16k::spec_at(km);
    const bool both = km != k;
    if (hs) {
        const float2 v = make_float2((float)(acc.x / NB), (float)(acc.y / NB));
        hs[at] = v;
        if (both) hs[am] = make_float2(v.x, -v.y);
    }
    if (ht) {
        const double2 t = cmul64(acc, g);
        const float2 v = make_float2((float)(t.x / NB), (float)(t.y / NB));
        ht[at] = v;
        if (both) ht[am] = make_float2(v.x, -v.y);
    }
    if (hf) {
        hf[k] = acc;
        if (both) hf[km] = make_double2(acc.x, -acc.y);
    }
}

// Decay of the cascade's response (ShortTab), CIRC_BLOCKS blocks, FP64: thread
// p of block blk sums |H|^2 at angle (256 blk + tid + 1/2) pi / (256
// CIRC_BLOCKS) on the unit circle and on circles of radius rho_j between the
// largest pole radius r and 1.  By Parseval the mean of |H|^2 on a circle of
// radius rho is sum_n h[n]^2 rho^(-2 n), so the response beyond sample L has a
// 2-norm of at most rho^L times its root.  (Exact decays by powers of the
// transition took 19 us in one block; this needs no chain of dependent steps
// and overstates the memory by 15 - 20 %.)
template <class Co>
__device__ void circle_block(char *raw, Co co_at, int32_t S, int blk, ShortTab *out, int tid) {
    struct Sh {
        double co[CASC_MAX][5], r[CASC_MAX], w[4][4];
    };
    Sh &sh = lds_as<Sh>(raw);
    if (tid < S * 5) sh.co[tid / 5][tid % 5] = co_at(tid / 5, tid % 5);
    __syncthreads();
    if (tid < S) sh.r[tid] = section_radius(sh.co[tid][3], sh.co[tid][4]);
    __syncthreads();
    double rm = 0.0;
    for (int s = 0; s < S; ++s) rm = rm == rm && !(sh.r[s] <= rm) ? sh.r[s] : rm;  // (a NaN stays)
    double sn, cs;
    sincospi(-((double)(256 * blk + tid) + 0.5) / (256.0 * CIRC_BLOCKS), &sn, &cs);
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
        const double rho = j == 0 ? 1.0 : rm + (1.0 - rm) * (j == 1 ? 0.0625 : j == 2 ? 0.125 : 0.25);
        const double zr = cs / rho, zi = sn / rho;
        double num = 1.0, den = 1.0;
#pragma unroll 1
        for (int s = 0; s < S; ++s) {
            const double *c = sh.co[s];
            const double ur = fma(zr, c[2], c[1]), ui = zi * c[2], vr = fma(zr, c[4], c[3]), vi = zi * c[4];
            const double nr = c[0] + zr * ur - zi * ui, ni = zr * ui + zi * ur;
            const double dr = 1.0 + zr * vr - zi * vi, di = zr * vi + zi * vr;
            num *= nr * nr + ni * ni;
            den *= dr * dr + di * di;
        }
        double v = num / den;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
        if ((tid & 63) == 0) sh.w[j][tid >> 6] = v;
        if (blk == 0 && tid == 0) out->lam[j] = rm <= 0.999 ? log2(rho) : 0.0;
    }
    __syncthreads();
    if (tid < 4) out->sum[blk][tid] = (sh.w[tid][0] + sh.w[tid][1]) + (sh.w[tid][2] + sh.w[tid][3]);
}

// The prepare step of a chain in one launch.  Blocks take roles by index:
// tap-spectrum blocks (which also write the twiddle tables), one block per
// section (scan tables), one block for the cascade's tile transition; every
// block also clears a share of the look-back records (tag 0 never matches
// an epoch), and block 0 arms the header (epoch 1, error 0, high-Q word).
struct PrepareArgs {
    const float *h;
    int32_t M, nspec;  // nspec = 256 * partitions, or 0 without an FFT FIR
    float2 *twid, *hspec;
    double2 *tw64;
    SecTab *tab;
    int32_t S, casc;
    StageList sos;
    CascTab *ctab;
    McTab *mc;     // matrix-core cascade tables (null: not wanted)
    CascZir *zir;  // zero-input response tables (null: not wanted)
    uint64_t *recs;
    int64_t nwords;
    uint32_t *hdr;
    // 16384-point path: the first n16 blocks, for a chain that may be a
    // short-memory one (ht16 set) CIRC_BLOCKS, then SPEC16_BLOCKS
    int32_t n16, cmp16;  // cmp16: operand type of the FIR's taps
    float2 *tw16, *hs16, *ht16;
    ShortTab *st16;
    double2 *hf16;
};

__global__ __launch_bounds__(256) void prepare_kernel(PrepareArgs a) {
    __shared__ __align__(16) char raw[PREP_LDS];
    const int tid = threadIdx.x;
    const int bid = blockIdx.x;
    for (int64_t i = (int64_t)bid * 256 + tid; i < a.nwords; i += (int64_t)gridDim.x * 256) a.recs[i] = 0ull;
    if (bid == 0) {  // header words; the cascade's high-Q word: one section per thread, loads in parallel
        __shared__ uint32_t s_any;
        if (tid == 0) s_any = 0u;
        __syncthreads();
        for (int q = tid; q < a.S; q += 256) {
            int sec = q, st = 0;
            while (sec >= a.sos.len[st]) {
                sec -= a.sos.len[st];
                ++st;
            }
            if (section_hiq(a.sos.ptr[st][5 * sec + 3], a.sos.ptr[st][5 * sec + 4])) atomicOr(&s_any, 1u);
        }
        __syncthreads();
        if (tid == 0) {
            a.hdr[HDR_ERROR] = 0u;
            a.hdr[HDR_EPOCH] = 1u;
            a.hdr[HDR_HIQ] = s_any;
            a.hdr[HDR_BAD] = 0u;
            a.hdr[HDR_SHORT] = 0u;
            a.hdr[HDR_DONE] = 0u;
            a.hdr[HDR_TABS] = a.ht16 ? 1u : 0u;
        }
    }
    if (bid < a.n16) {
        const StageList &sl = a.sos;
        const auto co = [&](int s, int k) {
            int st = 0;
            while (s >= sl.len[st]) {
                s -= sl.len[st];
                ++st;
            }
            return (double)sl.ptr[st][5 * s + k];
        };
        const int r = a.ht16 ? bid - CIRC_BLOCKS : bid;
        if (r < 0) circle_block(raw, co, a.S, bid, a.st16, tid);
        else spec16_block(raw, a.h, a.M, a.cmp16, co, a.S, r, a.tw16, a.hs16, a.ht16, a.hf16, tid);
        return;
    }
    const int b = bid - a.n16;
    if (b < a.nspec) {
        const int blk = b % (NFFT / 16), part = b / (NFFT / 16);
        spectrum_block(raw, a.h, a.M, part, blk, a.hspec, tid);
        if (part == 0 && tid < 16) write_twiddle(a.twid, a.tw64, blk * 16 + tid);
    } else if (b < a.nspec + a.S) {
        int s = b - a.nspec, st = 0;
        while (s >= a.sos.len[st]) {
            s -= a.sos.len[st];
            ++st;
        }
        build_section_block(&a.tab[b - a.nspec], a.sos.ptr[st] + 5 * s, L, tid);
    } else if (a.casc && b == a.nspec + a.S) {
        const StageList &sl = a.sos;
        casc_table_block(
            raw, [&](int s, int k) {
                int st = 0;
                while (s >= sl.len[st]) {
                    s -= sl.len[st];
                    ++st;
                }
                return (double)sl.ptr[st][5 * s + k];
            },
            a.S, L, a.ctab, tid);
    } else if (a.casc && a.mc && b == a.nspec + a.S + 1) {
        const StageList &sl = a.sos;
        mc_block(
            raw, [&](int s, int k) {
                int st = 0;
                while (s >= sl.len[st]) {
                    s -= sl.len[st];
                    ++st;
                }
                return (double)sl.ptr[st][5 * s + k];
            },
            a.S, a.mc, tid);
    } else if (a.casc && a.zir && b > a.nspec + a.S + 1 && b <= a.nspec + a.S + 2 + ZIR_B + ZIR_A) {
        const StageList &sl = a.sos;
        zir_block(
            raw, [&](int s, int k) {
                int st = 0;
                while (s >= sl.len[st]) {
                    s -= sl.len[st];
                    ++st;
                }
                return (double)sl.ptr[st][5 * s + k];
            },
            a.S, L, b - (a.nspec + a.S + 2), a.zir, tid);
    }
}

__global__ void state_passthrough_kernel(const float *in, float *out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in ? in[i] : 0.f;
}

// Batched clips: section tables of every clip (chunk length lc), the block
// map, cleared look-back records, epoch 1.  Thread g < nsec builds section g, found by a
// binary search over the clips' first table index.
struct BatchPrepArgs {
    const ClipDesc *desc;
    int32_t nclips;
    SecTab *tab;
    int64_t nsec;
    uint64_t *recs;
    int64_t nwords;
    uint32_t *hdr;
    int32_t lc;
    CascTab *ctab;  // per clip, or null
    McTab *mtab;    // per clip, or null
    int32_t *map;   // block id -> clip, nblocks entries
    int64_t nblocks;
};

// Blocks g < nsec build section g; blocks nsec + c build clip c's cascade
// tables (when ctab is set); every block clears a share of the records.
__global__ __launch_bounds__(256) void batch_prep_kernel(BatchPrepArgs a) {
    __shared__ __align__(16) char raw[PREP_LDS];
    const int tid = threadIdx.x;
    for (int64_t i = (int64_t)blockIdx.x * 256 + tid; i < a.nwords; i += (int64_t)gridDim.x * 256) a.recs[i] = 0ull;
    // block map: the last clip whose first block is <= b (first blocks never
    // decrease; a clip without blocks shares its first block with the next)
    for (int64_t b = (int64_t)blockIdx.x * 256 + tid; b < a.nblocks; b += (int64_t)gridDim.x * 256) {
        int lo = 0, hi = a.nclips - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (a.desc[mid].blk0 <= b) lo = mid;
            else hi = mid - 1;
        }
        a.map[b] = lo;
    }
    if (blockIdx.x == gridDim.x - 1) {  // (the first blocks have the longest roles)
        // eight threads a clip (by one thread in turn it was the kernel's length)
        uint32_t any = 0u;
        for (int c = tid >> 3; c < a.nclips; c += 32) {
            const float *co = a.desc[c].sos;
            const int S = a.desc[c].S;
            for (int s = tid & 7; s < S; s += 8) any |= section_hiq(co[5 * s + 3], co[5 * s + 4]) ? 1u : 0u;
        }
        any = __syncthreads_or(any);
        if (tid == 0) {
            a.hdr[HDR_ERROR] = 0u;
            a.hdr[HDR_EPOCH] = 1u;
            a.hdr[HDR_HIQ] = any ? 1u : 0u;
        }
    }
    const int64_t nroles = a.nsec + (a.ctab ? a.nclips : 0) + (a.mtab ? a.nclips : 0);
    for (int64_t g = blockIdx.x; g < nroles; g += gridDim.x) {
        if (g < a.nsec) {
            // the last clip with tab0 <= g: tab0 grows with the clip index by
            // S, so that clip has S > 0 and holds section g
            int lo = 0, hi = a.nclips - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) / 2;
                if (a.desc[mid].tab0 <= g) lo = mid;
                else hi = mid - 1;
            }
            build_section_block(&a.tab[g], a.desc[lo].sos + 5 * (g - a.desc[lo].tab0), a.lc, tid);
        } else if (g < a.nsec + a.nclips) {
            const ClipDesc &d = a.desc[g - a.nsec];
            if (d.S > 0) {
                const float *co = d.sos;
                casc_table_block(raw, [&](int s, int k) { return (double)co[5 * s + k]; }, d.S, a.lc,
                                 &a.ctab[g - a.nsec], tid);
            }
        } else {
            const int c = (int)(g - a.nsec - a.nclips);
            const ClipDesc &d = a.desc[c];
            if (d.S > 0) {
                const float *co = d.sos;
                mc_block(raw, [&](int s, int k) { return (double)co[5 * s + k]; }, d.S, &a.mtab[c], tid);
            }
        }
        __syncthreads();  // the role's shared memory is reused by the next one
    }
}

hipError_t launch_batch_prepare(const BatchLayout &lay, int lc, int32_t nclips, void *ws, hipStream_t st) {
    char *w = static_cast<char *>(ws);
    BatchPrepArgs a;
    a.desc = reinterpret_cast<const ClipDesc *>(w + lay.desc);
    a.nclips = nclips;
    a.tab = reinterpret_cast<SecTab *>(w + lay.tab);
    a.nsec = lay.nsec;
    a.recs = reinterpret_cast<uint64_t *>(w + lay.recs);
    a.nwords = lay.nrec * 4;
    a.hdr = reinterpret_cast<uint32_t *>(w + lay.hdr);
    a.lc = lc;
    a.ctab = lay.casc_on ? reinterpret_cast<CascTab *>(w + lay.casc) : nullptr;
    a.mtab = lay.mc_on ? reinterpret_cast<McTab *>(w + lay.mc) : nullptr;
    a.map = reinterpret_cast<int32_t *>(w + lay.map);
    a.nblocks = lay.nblocks;
    const int64_t nroles = a.nsec + (a.ctab ? nclips : 0) + (a.mtab ? nclips : 0);
    int64_t nb = (a.nwords + 255) / 256;
    if (nb > 2048) nb = 2048;
    if (nb < nroles) nb = nroles < 2048 ? nroles : 2048;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(batch_prep_kernel, dim3((unsigned)nb), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_tables(const ChainPlan &p, const WsLayout &lay, const float *h, int32_t M, void *hf) {
    char *ws = static_cast<char *>(p.ws);
    hipError_t e;
    if (p.firs.n > 1) {
        MergeArgs m;
        m.firs = p.firs;
        m.buf0 = reinterpret_cast<double *>(ws + lay.merge);
        m.buf1 = m.buf0 + M;
        m.out = reinterpret_cast<float *>(ws + lay.taps);
        hipLaunchKernelGGL(merge_taps_kernel, dim3(1), dim3(256), 0, p.stream, m);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    PrepareArgs a{};
    const bool fft = p.firs.n > 0 && p.fir_mode == FIR_FFT;
    a.h = h;
    a.M = M;
    a.nspec = fft ? (NFFT / 16) * fft_parts(M) : 0;
    a.twid = reinterpret_cast<float2 *>(ws + lay.twid);
    a.hspec = reinterpret_cast<float2 *>(ws + lay.hspec);
    a.tw64 = reinterpret_cast<double2 *>(ws + lay.tw64);
    a.tab = reinterpret_cast<SecTab *>(ws + lay.tab);
    a.S = p.S;
    a.casc = (p.S > 0 && p.S <= CASC_MAX) ? 1 : 0;
    a.sos = p.sos;
    a.ctab = reinterpret_cast<CascTab *>(ws + lay.casc);
    // cascades of up to ZIR_MAX sections take the zero-input response
    // tables, longer ones (up to CASC_MAX) the matrix-core form
    a.mc = (a.casc && p.S >= MC_MIN_SECTIONS) ? reinterpret_cast<McTab *>(ws + lay.mc) : nullptr;
    a.zir = (a.casc && p.S <= ZIR_MAX) ? reinterpret_cast<CascZir *>(ws + lay.zir) : nullptr;
    a.recs = reinterpret_cast<uint64_t *>(ws + lay.recs);
    a.nwords = p.S > 0 ? lay.cpad * lay.ntiles * p.S * REC_WORDS : 0;
    a.hdr = reinterpret_cast<uint32_t *>(ws + lay.hdr);
    int64_t nb = a.nspec + a.S + (a.casc ? 2 : 0) + (a.zir ? ZIR_B + ZIR_A + 1 : 0);
    if (p.firs.n > 0 && p.fir_mode == FIR_FFT16) {
        a.tw16 = reinterpret_cast<float2 *>(ws + lay.f16);
        a.hs16 = a.tw16 + f16k::TW_FLOAT2;
        a.n16 = SPEC16_BLOCKS;
    }
    a.cmp16 = TFX_COMPUTE_F32;
    if (short_wanted(p, lay)) {
        if (p.fir_mode == FIR_TOEPLITZ) a.cmp16 = p.cmp;
        if (!a.tw16) a.tw16 = reinterpret_cast<float2 *>(ws + lay.sh);
        a.ht16 = reinterpret_cast<float2 *>(ws + lay.sh) + f16k::TW_FLOAT2;
        a.st16 = reinterpret_cast<ShortTab *>(ws + lay.sh + fft16k_table_bytes());
        a.hf16 = static_cast<double2 *>(hf);
        a.n16 = SPEC16_BLOCKS + CIRC_BLOCKS;
    }
    nb += a.n16;
    int64_t nclear = (a.nwords + 255) / 256;
    if (nclear > 1024) nclear = 1024;
    if (nb < nclear) nb = nclear;
    // a workspace with room for the header gets its header words written
    // even when there is nothing else to build
    if (nb == 0 && p.ws && p.ws_bytes >= 256) nb = 1;
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)nb), dim3(256), 0, p.stream, a);
    return hipGetLastError();
}

// Header words of a workspace that a call uses without building anything
// (empty signals, identity cascades): error 0, epoch 1, no high-Q section.
__global__ void header_init_kernel(uint32_t *hdr) {
    hdr[HDR_ERROR] = 0u;
    hdr[HDR_EPOCH] = 1u;
    hdr[HDR_HIQ] = 0u;
    hdr[HDR_SHORT] = 0u;
    hdr[HDR_BAD] = 0u;
    hdr[HDR_DONE] = 0u;
    hdr[HDR_TABS] = 0u;
}

hipError_t launch_header_init(void *ws, size_t ws_bytes, hipStream_t st) {
    if (!ws || ws_bytes < 256) return hipSuccess;
    hipLaunchKernelGGL(header_init_kernel, dim3(1), dim3(1), 0, st, static_cast<uint32_t *>(ws));
    return hipGetLastError();
}

// Status word of a workspace: OR it into *flags (written only when a bit is
// set), then optionally clear it.  One thread; stream-ordered after the
// calls that used the workspace.
__global__ void ws_status_kernel(uint32_t *hdr, uint32_t *flags, int32_t clear) {
    const uint32_t v = __hip_atomic_load(hdr + HDR_ERROR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v) *flags |= v;
    if (clear) __hip_atomic_store(hdr + HDR_ERROR, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t launch_ws_status(void *ws, uint32_t *flags, int32_t clear, hipStream_t st) {
    hipLaunchKernelGGL(ws_status_kernel, dim3(1), dim3(1), 0, st, static_cast<uint32_t *>(ws), flags, clear);
    return hipGetLastError();
}

hipError_t launch_twiddles(float2 *twid, double2 *tw64, hipStream_t st) {
    hipLaunchKernelGGL(fft_twiddle_kernel, dim3(NFFT / 256), dim3(256), 0, st, twid, tw64);
    return hipGetLastError();
}

hipError_t launch_state_passthrough(const float *in, float *out, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(state_passthrough_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, in, out, n);
    return hipGetLastError();
}

}  // namespace tfx
