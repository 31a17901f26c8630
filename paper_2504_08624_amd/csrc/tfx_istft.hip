// tfx_istft.hip -- the inverse short-time Fourier transform for hops of 256 H
// samples (the other hops: istft_kernel in tfx_stft.hip).
#include "tfx_stft.h"

namespace tfx {
namespace {

// The inverse for hops of 256 H samples, H = 1, 2, 4, .. (n_fft >= 256): lane
// tid then owns the same residue of every frame, and the overlap-add is a
// sliding window of registers: acc[q] holds sample 256 q + tid of the current
// frame's span, a frame is added with one LDS read and one fused multiply-add a
// sample, and the H leading registers are final and stored.  (istft_kernel
// adds through LDS, three accesses a sample and a barrier a frame, and its
// accumulator leaves room for two workgroups a CU.)  A unit is a run of K hops of
// one channel; the ceil(N / hop) - 1 frames before it are inverted again.  The
// frames of a sample are added in the same order as above.
// Measured on 8 x 5.76 M samples, n_fft 2048, hop 512: 528 -> 258 us a launch (3.6 TB/s of spectrum and samples).
template <int LOG2N, int H>
__global__ __launch_bounds__(SWG, 4) void istft_slide_kernel(StftArgs a) {
    using S = Shape<LOG2N>;
    constexpr int N = S::N, G = S::G, F = S::F, NW = N / SWG, HOP = SWG * H;
    static_assert(NW >= H && LOG2N >= 8, "the hop fits in the frame");
    __shared__ float2 buf[S::LDS_BUF];
    __shared__ float2 tw[S::TWN];
    const int tid = threadIdx.x;
    fill_twiddles<LOG2N>(tw, tid);
    float wq[NW], env[H];  // window x scale; summed squared window of a sample that every frame reaches
#pragma unroll
    for (int j = 0; j < H; ++j) {
        float e = 0.f;
#pragma unroll
        for (int q = j; q < NW; q += H) {
            const float w = window_at(a, tid + q * SWG);
            e += w * w;
        }
        env[j] = e;
    }
#pragma unroll
    for (int q = 0; q < NW; ++q) wq[q] = window_at(a, tid + q * SWG) * a.scale;
    constexpr int WARM = (N + HOP - 1) / HOP - 1;
    const int64_t h0 = a.off / HOP;  // hop that holds the first output sample
    const UnitRange ur = unit_range(a.units);
    for (int64_t u = ur.first; u < ur.end; u += ur.step) {
        const int64_t c = u / a.nseg;
        const int64_t f0 = h0 + (u - c * a.nseg) * a.P;  // first hop of the unit
        const int64_t fend = (a.L + a.off + HOP - 1) / HOP;
        const int64_t f1 = f0 + a.P < fend ? f0 + a.P : fend;
        float acc[NW];
#pragma unroll
        for (int q = 0; q < NW; ++q) acc[q] = 0.f;
        float *yc = a.y + c * a.ldy;
        for (int64_t tb = f0 - WARM; tb < f1; tb += 2 * G) {
            // (laundered: the addresses formed from it are not kept across batches)
            int tl = tid;
            asm volatile("" : "+v"(tl));
            // conj of Z = Xa + i Xb as above; row g holds frames tb + 2 g and tb + 2 g + 1
            const float2 *sb = a.spec + (c * a.T + tb) * F;
            constexpr int NL = (G * F + SWG - 1) / SWG;
            float2 xa[NL], xb[NL];
#pragma unroll
            for (int q = 0; q < NL; ++q) {  // loads first
                const int i = tl + q * SWG, g = i / F;
                xa[q] = make_float2(0.f, 0.f);
                xb[q] = xa[q];
                if (i < G * F) {
                    const int64_t ta = tb + 2 * g;
                    const float2 *in = sb + i + g * F;
                    if (ta >= 0 && ta < a.T) xa[q] = in[0];
                    if (ta + 1 >= 0 && ta + 1 < a.T) xb[q] = in[F];
                }
            }
            __syncthreads();  // the previous batch's reads of buf; the twiddles
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int i = tl + q * SWG, g = i / F, k = i - g * F;
                if (i >= G * F) break;
                if (k == 0 || k == N / 2) {
                    xa[q].y = 0.f;
                    xb[q].y = 0.f;
                }
                buf[pad(g * N + k)] = make_float2(xa[q].x - xb[q].y, -(xa[q].y + xb[q].x));
                if (k > 0 && k < N / 2)
                    buf[pad(g * N + N - k)] = make_float2(xa[q].x + xb[q].y, xa[q].y - xb[q].x);
            }
            __syncthreads();
            fft_rows<LOG2N>(buf, tw, tl);
            // frame tb + f is the real (f even) or negated imaginary (f odd) part of row f / 2
#pragma unroll 1
            for (int g = 0; g < G; ++g) {
                float2 z[NW];
                const int b = pad(g * N + tid);
#pragma unroll
                for (int q = 0; q < NW; ++q) z[q] = buf[b + q * (SWG + SWG / 16)];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int64_t f = tb + 2 * g + s;
#pragma unroll
                    for (int q = 0; q < NW; ++q) acc[q] += wq[q] * (s ? -z[q].y : z[q].x);
                    if (f >= f0 && f < f1) {
                        const int64_t p0 = f * HOP, i0 = p0 - a.off;
                        float *yp = yc + i0 + tid;
                        if (p0 >= N - HOP && f <= a.T - 1 && i0 >= 0 && i0 + HOP <= a.L) {
#pragma unroll
                            for (int j = 0; j < H; ++j) yp[j * SWG] = env[j] > 1e-11f ? acc[j] / env[j] : 0.f;
                        } else {  // fewer frames than in the middle, or a hop partly outside: sums first
#pragma unroll
                            for (int j = 0; j < H; ++j)
                                if ((uint64_t)(i0 + j * SWG + tid) < (uint64_t)a.L) yp[j * SWG] = acc[j];
#pragma unroll 1
                            for (int j = 0; j < H; ++j) {
                                const int64_t p = p0 + j * SWG + tid;
                                if ((uint64_t)(p - a.off) >= (uint64_t)a.L) continue;
                                float e = 0.f;
                                for (int64_t t = f < a.T - 1 ? f : a.T - 1; t >= 0 && p - t * HOP < N; --t) {
                                    const float w = window_at(a, (int)(p - t * HOP));
                                    e += w * w;
                                }
                                yp[j * SWG] = e > 1e-11f ? yp[j * SWG] / e : 0.f;
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < NW; ++q) acc[q] = q + H < NW ? acc[q + H] : 0.f;
                }
            }
        }
    }
}

// The sliding inverse of this size and hop (null: none).
typedef void (*IstftKernel)(StftArgs);
template <int LOG2N>
IstftKernel slide_of(int32_t hop) {
    constexpr int NW = (1 << LOG2N) / SWG;
    if (hop == SWG) return istft_slide_kernel<LOG2N, 1>;
    if constexpr (NW >= 2)
        if (hop == 2 * SWG) return istft_slide_kernel<LOG2N, 2>;
    if constexpr (NW >= 4)
        if (hop == 4 * SWG) return istft_slide_kernel<LOG2N, 4>;
    if constexpr (NW >= 8)
        if (hop == 8 * SWG) return istft_slide_kernel<LOG2N, 8>;
    if constexpr (NW >= 16)
        if (hop == 16 * SWG) return istft_slide_kernel<LOG2N, 16>;
    return nullptr;
}

}  // namespace

hipError_t launch_istft_slide(const StftPlan &sp, bool *done) {
    const int N = 1 << sp.log2n;
    const IstftKernel slide = sp.log2n == 8 ? slide_of<8>(sp.hop) : sp.log2n == 9 ? slide_of<9>(sp.hop)
                        : sp.log2n == 10 ? slide_of<10>(sp.hop) : sp.log2n == 11 ? slide_of<11>(sp.hop)
                        : sp.log2n == 12 ? slide_of<12>(sp.hop) : nullptr;
    *done = slide != nullptr;
    if (!slide) return hipSuccess;
    StftArgs a = inverse_args(sp);
    // runs of K hops, at most one a resident workgroup (four a CU), whole
    // batches of frames with the ones inverted again in front of a run
    const int64_t hops = (a.L + a.off + sp.hop - 1) / sp.hop - a.off / sp.hop;
    const int64_t runs = 1024 / sp.C > 0 ? 1024 / sp.C : 1, warm = (N + sp.hop - 1) / sp.hop - 1;
    const int64_t b2 = 2 * batch_of(sp.log2n), k = (hops + runs - 1) / runs;
    a.P = (k + warm + b2 - 1) / b2 * b2 - warm;
    if (a.P < 1) a.P += b2;
    a.nseg = (hops + a.P - 1) / a.P;
    a.units = sp.C * a.nseg;
    hipLaunchKernelGGL(slide, unit_grid(a.units, 4), dim3(SWG), 0, sp.stream, a);
    return hipGetLastError();
}

}  // namespace tfx
