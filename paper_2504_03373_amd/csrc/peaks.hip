// Bin integration (eq.6 of arXiv 2504.03373) and peak search (Sec. III-A, last paragraph).
//
// Pbar[d] = sum_f P[f, d].  Deterministic, atomics-free order: bins are summed in ascending order
// inside fixed chunks of SSL_BINSUM_CHUNK bins (one thread per (direction, chunk), the whole chip
// busy), then a second launch (one workgroup per block) sums the chunk partials in ascending chunk
// order and searches the peaks.  The launch boundary makes the partials visible: no device-scope
// fence per workgroup (each is an L2 write-back on this multi-XCD part) and no completion counter.
//
// Peak rule on the n_el x n_az grid (d = el * n_az + az): d is a local maximum when it beats each
// of its 8 neighbours -- azimuth circular, elevation clamped -- where "beats" means a larger value,
// or an equal value and a lower flat index.  Maxima are ranked by the same relation; the first
// Ns are returned, -1 / 0 beyond the number found.  Non-finite values never take part.
//
// The second launch is one workgroup's latency: the partials come from other XCDs' L2s, so that those
// of two directions a thread are loaded at once, and a peak costs one barrier (shuffles within a
// wave, one LDS exchange between the waves).  257 bins, 1368 directions, 2 peaks: 7.5 us; 11.6 us with loads
// in groups of 8, early exits from the neighbour tests and a barrier per halving of the maximum.
#include "ssl_internal.h"

namespace {

constexpr int kThreads = 256;         // partial sums
constexpr int kFinal = 1024;          // final sum + peak search, one workgroup per block
constexpr int kLdsPbar = 8192;        // Pbar staged in LDS when D <= this
constexpr int kPart = 16;             // chunk partials of a direction in flight

// "beats" as one comparison: value, then lower index; 0 for a value that takes no part (-0 counts
// as +0, as in a comparison of floats).
__device__ __forceinline__ unsigned long long rank_key(float v, int d)
{
    const unsigned int b = __float_as_uint(v + 0.0f);
    const unsigned int u = b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
    return isfinite(v) ? ((unsigned long long)u << 32) | ~(unsigned int)d : 0ull;
}

// The key of direction d if it is a local maximum, else 0.  All neighbours are read at once: in LDS
// the reads cost less than the branches that would leave early.
__device__ __forceinline__ unsigned long long peak_key(const float *pb, int n_el, int n_az, int d)
{
    const int el = d / n_az, az = d - el * n_az;
    const int left = az == 0 ? n_az - 1 : az - 1, right = az == n_az - 1 ? 0 : az + 1;
    const unsigned long long own = rank_key(pb[d], d);
    unsigned long long top = 0ull;
#pragma unroll
    for (int de = -1; de <= 1; ++de) {
        const int e = min(max(el + de, 0), n_el - 1);        // clamped: the own row again
#pragma unroll
        for (int da = -1; da <= 1; ++da) {
            const int nb = e * n_az + (da < 0 ? left : da > 0 ? right : az);
            const unsigned long long k = rank_key(pb[nb], nb);
            top = k > top ? k : top;                         // the direction itself included
        }
    }
    return top == own ? own : 0ull;
}

// Whole-workgroup peak search over pb[0..D) (LDS or global).  cand is an LDS flag array of size >= D
// when D <= kLdsPbar; otherwise the maxima are found again for each peak.  The key maximum goes over the
// lanes of a wave by shuffles and over the waves through LDS.
__device__ void search_peaks(const float *pb, int D, int n_az, int n_el, int Ns,
                             int32_t *__restrict__ peaks, float *__restrict__ peak_val,
                             unsigned char *cand, unsigned long long *red)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool keep = D <= kLdsPbar;
    unsigned long long below = ~0ull;                        // peaks so far have larger keys
    for (int k = 0; k < Ns; ++k) {
        unsigned long long best = 0ull;
        for (int d = tid; d < D; d += kFinal) {              // a thread's own directions each time
            unsigned long long v;
            if (keep && k > 0) {
                v = cand[d] ? rank_key(pb[d], d) : 0ull;
            } else {
                v = peak_key(pb, n_el, n_az, d);
                if (keep) cand[d] = v != 0ull;
            }
            if (v < below && v > best) best = v;
        }
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) {
            const unsigned long long o = __shfl_xor(best, s);
            best = o > best ? o : best;
        }
        if (lane == 0) red[(k & 1) * (kFinal / 64) + wave] = best;
        __syncthreads();
        best = red[(k & 1) * (kFinal / 64) + (lane & (kFinal / 64 - 1))];
#pragma unroll
        for (int s = kFinal / 128; s > 0; s >>= 1) {
            const unsigned long long o = __shfl_xor(best, s);
            best = o > best ? o : best;
        }
        below = best;                                        // 0: none left, nor for later peaks
        if (tid == 0) {
            const int d = best != 0ull ? (int)~(unsigned int)best : -1;
            peaks[k] = d;
            peak_val[k] = d >= 0 ? pb[d] : 0.0f;
        }
    }
}

// Partial sums: thread (dc, ch, tid) sums bins ch*CHUNK .. +CHUNK-1 of direction dc*kThreads+tid.
__device__ __forceinline__ void binsum_part_body(const float *__restrict__ P, int F, int D,
                                                 float *__restrict__ part, int dc, int ch)
{
    const int d = dc * kThreads + (int)threadIdx.x;
    if (d >= D) return;
    // all loads of the chunk in flight at once, then the sum in ascending bin order
    // (absent bins of a short last chunk add an exact 0)
    const int f0 = ch * SSL_BINSUM_CHUNK;
    const int nf = min(F - f0, SSL_BINSUM_CHUNK);
    float v[SSL_BINSUM_CHUNK];
#pragma unroll
    for (int i = 0; i < SSL_BINSUM_CHUNK; ++i)
        v[i] = (i < nf) ? P[(size_t)(f0 + i) * D + d] : 0.0f;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < SSL_BINSUM_CHUNK; ++i) s += v[i];
    part[(size_t)ch * D + d] = s;
}

// Final sum over the nch chunk partials (ascending) and the peak search (peaks may be null).
__device__ __forceinline__ void binsum_final_body(const float *__restrict__ part, int nch, int D,
                                                  float *__restrict__ Pbar, int n_az, int n_el,
                                                  int Ns, int32_t *__restrict__ peaks,
                                                  float *__restrict__ peak_val)
{
    __shared__ float pb_s[kLdsPbar];
    __shared__ unsigned char cand[kLdsPbar];
    __shared__ unsigned long long red[2 * kFinal / 64];
    const int tid = threadIdx.x;
    const bool lds = D <= kLdsPbar;
    // a uniform row and a 32-bit byte offset (D <= 2^24): no address registers per load
    auto at = [](const float *row, unsigned int x) {
        return reinterpret_cast<const float *>(reinterpret_cast<const char *>(row) + 4u * x);
    };
    // two directions a thread, kPart partials of both in flight (absent ones add an exact 0)
#pragma unroll 1
    for (unsigned int e = tid; e < (unsigned int)D; e += 2 * kFinal) {
        const unsigned int e1 = min(e + kFinal, (unsigned int)D - 1);  // in range; dropped below if not ours
        float s = 0.f, s1 = 0.f;
#pragma unroll 1
        for (int c0 = 0; c0 < nch; c0 += kPart) {
            float v[kPart], v1[kPart];
            const float *row = part + (size_t)c0 * D;
#pragma unroll
            for (int i = 0; i < kPart; ++i, row += D) {
                v[i] = v1[i] = 0.0f;
                if (c0 + i < nch) {                          // uniform
                    v[i] = gload(at(row, e));
                    v1[i] = gload(at(row, e1));
                }
            }
#pragma unroll
            for (int i = 0; i < kPart; ++i) {
                s += v[i];
                s1 += v1[i];
            }
        }
        gstore(Pbar + e, s);
        if (lds) pb_s[e] = s;
        if (e + kFinal < D) {
            gstore(Pbar + e1, s1);
            if (lds) pb_s[e1] = s1;
        }
    }
    __syncthreads();
    if (peaks != nullptr)
        search_peaks(lds ? pb_s : Pbar, D, n_az, n_el, Ns, peaks, peak_val, cand, red);
}

__global__ __launch_bounds__(kThreads) void binsum_part(const float *__restrict__ P, int F, int D,
                                                        float *__restrict__ part)
{
    binsum_part_body(P, F, D, part, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kFinal) void binsum_final(const float *__restrict__ part, int nch,
                                                       int D, float *__restrict__ Pbar, int n_az,
                                                       int n_el, int Ns,
                                                       int32_t *__restrict__ peaks,
                                                       float *__restrict__ peak_val)
{
    binsum_final_body(part, nch, D, Pbar, n_az, n_el, Ns, peaks, peak_val);
}

// Batch: grid z (partials) or x (final) = block; workgroups outside a block's own (direction,
// bin) chunk grid leave at once.
__global__ __launch_bounds__(kThreads) void binsum_part_batch(const BlockDev *__restrict__ blk)
{
    const BlockDev &B = blk[blockIdx.z];
    const int ndc = (B.D + kThreads - 1) / kThreads;
    const int nch = (B.F + SSL_BINSUM_CHUNK - 1) / SSL_BINSUM_CHUNK;
    if ((int)blockIdx.x >= ndc || (int)blockIdx.y >= nch) return;
    binsum_part_body(B.P, B.F, B.D, B.part, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kFinal) void binsum_final_batch(const BlockDev *__restrict__ blk,
                                                             unsigned int *__restrict__ clear, int n_clear)
{
    if (blockIdx.x == 0 && (int)threadIdx.x < n_clear) clear[threadIdx.x] = 0u;
    const BlockDev &B = blk[blockIdx.x];
    const int nch = (B.F + SSL_BINSUM_CHUNK - 1) / SSL_BINSUM_CHUNK;
    binsum_final_body(B.part, nch, B.D, B.Pbar, B.n_az, B.n_el, B.Ns, B.peaks, B.peak_val);
}

__global__ __launch_bounds__(kFinal) void peaks_only(const float *__restrict__ Pbar, int D,
                                                     int n_az, int n_el, int Ns,
                                                     int32_t *__restrict__ peaks,
                                                     float *__restrict__ peak_val)
{
    __shared__ float pb_s[kLdsPbar];
    __shared__ unsigned char cand[kLdsPbar];
    __shared__ unsigned long long red[2 * kFinal / 64];
    const bool lds = D <= kLdsPbar;
    if (lds)
        for (int e = threadIdx.x; e < D; e += kFinal) pb_s[e] = Pbar[e];
    __syncthreads();
    search_peaks(lds ? pb_s : Pbar, D, n_az, n_el, Ns, peaks, peak_val, cand, red);
}

}  // namespace

hipError_t launch_binsum_peaks(const float *P, int F, int D, float *Pbar, float *part,
                               int n_az, int n_el, int Ns, int32_t *peaks, float *peak_val,
                               hipStream_t st)
{
    const int nch = (F + SSL_BINSUM_CHUNK - 1) / SSL_BINSUM_CHUNK;
    hipLaunchKernelGGL(binsum_part, dim3((D + kThreads - 1) / kThreads, nch), dim3(kThreads), 0,
                       st, P, F, D, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(binsum_final, dim3(1), dim3(kFinal), 0, st, part, nch, D, Pbar, n_az, n_el,
                       Ns, peaks, peak_val);
    return hipGetLastError();
}

int binsum_threads() { return kThreads; }

hipError_t launch_binsum_batch(const BlockDev *blk, int nblocks, int max_dchunks, int max_fchunks,
                               unsigned int *clear, int n_clear, hipStream_t st)
{
    if (nblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(binsum_part_batch, dim3(max_dchunks, max_fchunks, nblocks),
                       dim3(kThreads), 0, st, blk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(binsum_final_batch, dim3(nblocks), dim3(kFinal), 0, st, blk, clear, n_clear);
    return hipGetLastError();
}

hipError_t launch_peaks(const float *Pbar, int n_az, int n_el, int Ns, int32_t *peaks,
                        float *peak_val, hipStream_t st)
{
    hipLaunchKernelGGL(peaks_only, dim3(1), dim3(kFinal), 0, st, Pbar, n_az * n_el, n_az, n_el,
                       Ns, peaks, peak_val);
    return hipGetLastError();
}
