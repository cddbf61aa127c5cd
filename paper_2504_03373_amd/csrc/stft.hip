// Front end of the method (eq.1): the short-time Fourier transform of every channel,
//   X_m(w, t) = sum_{n < N} win[n] x_m[t hop + n] e^{-2 pi i w n / N},   w = 0 .. N/2,
// written as X [N/2 + 1][T][M] complex64, the layout the correlation reads (channels contiguous).
//
// GPU mapping (gfx950): about 10 flops per input byte at N = 512, so an FFT in LDS, not a DFT-as-GEMM.
// One workgroup per (frame, group of CH channels).  A real frame is transformed as H = N/2 complex
// points z_n = y_{2n} + i y_{2n+1} (y the windowed frame): half the butterflies, and, unlike two
// channels in one transform, no channel's rounding depends on another's level.  The points go, channel-interleaved (CH
// consecutive channels of a sample are one contiguous read of the [n_samples][M] PCM), into
// bit-reversed positions of an [H][CH] LDS array; passes of two radix-2 stages at a time follow in
// registers, a thread per (4 points, channel); then X_k = E_k + e^{-2 pi i k / N} O_k from Z_k and Z_{H-k}, and the
// N/2 + 1 bins leave as rows of CH consecutive channels.  The twiddles e^{-2 pi i k / N}, k <= H, are
// made once per workgroup by sincospif of exact dyadic fractions and shared through LDS, as is the
// window.
//   With 200 workgroups (50 frames of 60 channels) the time is one workgroup's chain of passes, which
// the whole 1024-thread workgroup shares: 7.6 us for N = 512; 45 us with 256 threads, radix-2 stages over
// all N points and a sine and cosine per butterfly.
#include "ssl_internal.h"

namespace {

// channels per workgroup: the [N/2][CH] complex frame fills at most 32 KB of LDS
constexpr int stft_ch(int logn) { return (1 << logn) >= 8192 ? 1 : (8192 >> logn) < 16 ? (8192 >> logn) : 16; }
// threads: one (4 points, channel) each, in whole waves
constexpr int stft_threads(int logn)
{
    const int n = (1 << logn) / 8 * stft_ch(logn);
    return n < 64 ? 64 : n > 1024 ? 1024 : n;
}

__device__ __forceinline__ float2 twiddled(float2 v, float2 w)           // v w
{
    return make_float2(fmaf(v.x, w.x, -v.y * w.y), fmaf(v.x, w.y, v.y * w.x));
}

template <int LOGN>
__global__ __launch_bounds__(stft_threads(LOGN)) void stft_frames(const float *__restrict__ pcm, int M,
                                                        int hop, const float *__restrict__ win,
                                                        int T, float2 *__restrict__ X)
{
    constexpr int N = 1 << LOGN, H = N / 2, LOGH = LOGN - 1;
    constexpr int CH = stft_ch(LOGN);
    constexpr int THREADS = stft_threads(LOGN);
    constexpr int PER = (H * CH + THREADS - 1) / THREADS;
    __shared__ float2 buf[H * CH];
    __shared__ float2 tw[H + 1];                    // e^{-2 pi i k / N}
    __shared__ float ws[N];
    const int t = blockIdx.x, tid = threadIdx.x;
    const int c0 = blockIdx.y * CH;
    const int nc = min(CH, M - c0);
    const float *frame = pcm + (int64_t)t * hop * M + c0;
    float2 z[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {                 // in flight under the tables
        const int e = tid + i * THREADS, n = e / CH, ch = e - n * CH;
        z[i] = make_float2(0.0f, 0.0f);
        if (n < H && ch < nc)
            z[i] = make_float2(frame[(int64_t)(2 * n) * M + ch], frame[(int64_t)(2 * n + 1) * M + ch]);
    }
    for (int k = tid; k <= H; k += THREADS) {
        float sn, cs;
        sincospif(-(float)k / (float)H, &sn, &cs);
        tw[k] = make_float2(cs, sn);
    }
    for (int n = tid; n < N; n += THREADS) {
        float w;
        if (win) {
            w = win[n];
        } else {                                    // periodic Hann: sin^2(pi n / N)
            const float s = sinpif((float)n / (float)N);
            w = s * s;
        }
        ws[n] = w;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = tid + i * THREADS, n = e / CH, ch = e - n * CH;
        if (n < H) {
            const int rn = (int)(__brev((unsigned int)n) >> (32 - LOGH));
            buf[rn * CH + ch] = make_float2(ws[2 * n] * z[i].x, ws[2 * n + 1] * z[i].y);
        }
    }
    __syncthreads();
    if constexpr (LOGH & 1) {                       // a single stage first: span 1, no twiddle
        for (int e = tid; e < (H / 2) * CH; e += THREADS) {
            const int b = e / CH, ch = e - b * CH;
            float2 *p = buf + 2 * b * CH + ch;
            const float2 u = p[0], v = p[CH];
            p[0] = make_float2(u.x + v.x, u.y + v.y);
            p[CH] = make_float2(u.x - v.x, u.y - v.y);
        }
        __syncthreads();
    }
#pragma unroll
    for (int s = LOGH & 1; s < LOGH; s += 2) {      // stages s and s + 1: spans h and 2 h
        const int h = 1 << s;
        for (int e = tid; e < (H / 4) * CH; e += THREADS) {
            const int b = e / CH, ch = e - b * CH;
            const int j = b & (h - 1);
            float2 *p = buf + (((b >> s) << (s + 2)) + j) * CH + ch;
            const float2 w1 = tw[j << (LOGN - 1 - s)], w2 = tw[j << (LOGN - 2 - s)];
            const float2 x0 = p[0], x2 = p[2 * h * CH];
            const float2 t1 = twiddled(p[h * CH], w1), t3 = twiddled(p[3 * h * CH], w1);
            const float2 a = make_float2(x0.x + t1.x, x0.y + t1.y);
            const float2 c = make_float2(x0.x - t1.x, x0.y - t1.y);
            const float2 b2 = twiddled(make_float2(x2.x + t3.x, x2.y + t3.y), w2);
            const float2 d2 = twiddled(make_float2(x2.x - t3.x, x2.y - t3.y), w2);   // times -i below
            p[0] = make_float2(a.x + b2.x, a.y + b2.y);
            p[2 * h * CH] = make_float2(a.x - b2.x, a.y - b2.y);
            p[h * CH] = make_float2(c.x + d2.y, c.y - d2.x);
            p[3 * h * CH] = make_float2(c.x - d2.y, c.y + d2.x);
        }
        __syncthreads();
    }
    for (int e = tid; e < (H + 1) * CH; e += THREADS) {
        const int k = e / CH, ch = e - k * CH;
        if (ch < nc) {
            const float2 zk = buf[(k & (H - 1)) * CH + ch], zm = buf[((H - k) & (H - 1)) * CH + ch];
            const float2 ev = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
            const float2 od = make_float2(0.5f * (zk.y + zm.y), 0.5f * (zm.x - zk.x));
            const float2 o = twiddled(od, tw[k]);
            X[((int64_t)k * T + t) * M + c0 + ch] = make_float2(ev.x + o.x, ev.y + o.y);
        }
    }
}

template <int LOGN>
hipError_t launch(const float *pcm, int M, int hop, const float *win, int T, ssl_c64 *X,
                  hipStream_t st)
{
    constexpr int CH = stft_ch(LOGN);
    hipLaunchKernelGGL((stft_frames<LOGN>), dim3(T, (M + CH - 1) / CH),
                       dim3(stft_threads(LOGN)), 0, st, pcm,
                       M, hop, win, T, reinterpret_cast<float2 *>(X));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stft(const float *pcm, int M, int nfft, int hop, const float *win, int T,
                       ssl_c64 *X, hipStream_t st)
{
    switch (nfft) {
    case 16: return launch<4>(pcm, M, hop, win, T, X, st);
    case 32: return launch<5>(pcm, M, hop, win, T, X, st);
    case 64: return launch<6>(pcm, M, hop, win, T, X, st);
    case 128: return launch<7>(pcm, M, hop, win, T, X, st);
    case 256: return launch<8>(pcm, M, hop, win, T, X, st);
    case 512: return launch<9>(pcm, M, hop, win, T, X, st);
    case 1024: return launch<10>(pcm, M, hop, win, T, X, st);
    case 2048: return launch<11>(pcm, M, hop, win, T, X, st);
    case 4096: return launch<12>(pcm, M, hop, win, T, X, st);
    default: return hipErrorInvalidValue;
    }
}
