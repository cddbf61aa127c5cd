// Noise whitening for eq.4 of arXiv 2504.03373 (GSVD of K^{-1} R), all in FP64.
//
// The paper inverts the preset noise correlation K by Gaussian elimination and then forms
// A = K^{-1} R with a matrix product (Sec. III-B).  K is Hermitian positive definite and fixed per
// stream (or slowly updated), so here K^{-1} is computed once per noise set by in-place
// Gauss-Jordan elimination in FP64 and kept resident; each block then needs only the FP64 product
// A = K^{-1} R, rounded to complex64 for the FP32 Jacobi SVD.  Without pivoting on a Hermitian
// positive definite matrix the elimination pivots are the Schur-complement diagonals, i.e. the
// squared diagonal of the Cholesky factor, so they double as the positive-definiteness test.
#include "ssl_internal.h"

#include <atomic>
#include <utility>

namespace {

constexpr double kPdRel = 9.094947017729282e-13;   // 2^-40: pivot floor relative to max_i K_ii

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Lane L of each row of 16 lanes, to the whole row (DPP row_newbcast).
template <int L>
__device__ __forceinline__ double row_bcast(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x150 + L, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x150 + L, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// K^{-1} of one bin by in-place Gauss-Jordan elimination in blocks of 16 pivots, NW waves (M <= 16 NW),
// wave w holding rows 16 w .. 16 w + 15 as NW tiles in the FP64 MFMA result layout (element e of lane l:
// row l / 16 + 4 e, column l % 16).  Block step k with P = W_kk, after which W_kk = P^{-1}:
//   W_kj = P^{-1} W_kj,  W_ij -= W_ik W_kj,  W_ik = -W_ik P^{-1}    (i, j != k).
// Every wave posts its tile of block column k and wave k its rows; wave k inverts P alone (16 scalar
// steps, one wave, no barrier: row and column of the pivot by lane broadcasts), wave j forms
// W_kj and its W_jk, and each wave updates its tiles on v_mfma_f64_16x16x4f64 (four real products
// per complex one).  A product with the explicit P^{-1} has an error of 2^-53 cond(P) that the update's
// W_ik (large where P is) would amplify once more, so P^{-1} W_kj is corrected once by its residual
// W_kj - P (P^{-1} W_kj), which leaves the error of a backward stable solve (P-bar error at cond(K) =
// 1e8: 6e-3 without the correction, 2e-7 with it and with scalar pivots).  The scalar pivots are the Schur-complement diagonals d_k = L_kk^2 as without blocks; one
// that is <= 2^-40 max_i K_ii or not finite marks the bin NOT_PD (the inverse is then zero).
// Padding rows and columns (>= M) are zero and stay zero.
//   Bound by the 16-step chain of the pivot blocks (about half of the cycles) and the FP64 matrix cores.
// 257 bins of 60 channels: 52 us, five such sets in one launch 148 us, 11 of 16 and 8 channels 14 us
// (122, 346 and 31 us with one barrier per scalar pivot and rank-1 updates on the vector ALU).
template <int NW> struct FactorCfg {
    static constexpr int THREADS = 64 * NW;
    static constexpr int LD = 16 * NW + 1;         // LDS row stride, complex128
};

// One scalar step (pivot KK of the block) on a 16 x 16 tile of one wave.
template <int KK>
__device__ __forceinline__ void pivot_step(double2 (&a)[4], int lane, double thr, int m, bool &bad)
{
    constexpr int E = KK >> 2, G = (KK & 3) << 4;
    if (KK >= m || bad) return;                        // uniform
    const double2 rowk = make_double2(__shfl(a[E].x, G | (lane & 15)), __shfl(a[E].y, G | (lane & 15)));
    const long long pb = __builtin_bit_cast(long long, a[E].x);
    const int lo = __builtin_amdgcn_readlane((int)pb, G | KK);
    const int hi = __builtin_amdgcn_readlane((int)(pb >> 32), G | KK);
    const double p = __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
    if (!(p > thr && p < 1.7e308)) {                   // NaN and Inf too
        bad = true;
        return;
    }
    double ip = __builtin_amdgcn_rcp(p);
    ip = fma(ip, fma(-p, ip, 1.0), ip);
    ip = fma(ip, fma(-p, ip, 1.0), ip);
    const double2 wk = make_double2(rowk.x * ip, rowk.y * ip);      // the pivot row, scaled
    const bool colk = (lane & 15) == KK;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double2 c = make_double2(row_bcast<KK>(a[e].x), row_bcast<KK>(a[e].y));   // W_ik
        // selects by component: on whole double2 values the compiler goes through scratch memory
        const double gx = fma(-c.x, wk.x, fma(c.y, wk.y, a[e].x));
        const double gy = fma(-c.x, wk.y, fma(-c.y, wk.x, a[e].y));
        double nx = colk ? -c.x * ip : gx, ny = colk ? -c.y * ip : gy;
        if (e == E) {
            const bool rowe = (lane & 48) == G;
            nx = rowe ? (colk ? ip : wk.x) : nx;
            ny = rowe ? (colk ? 0.0 : wk.y) : ny;
        }
        a[e].x = nx;
        a[e].y = ny;
    }
}
template <int... KK>
__device__ __forceinline__ void invert_tile(std::integer_sequence<int, KK...>, double2 (&a)[4],
                                            int lane, double thr, int m, bool &bad)
{
    (pivot_step<KK>(a, lane, thr, m, bad), ...);
}

// out = init + sign * X y on one 16 x 16 complex tile, K = 16: x(q) the A operand of k-step q (row
// lane % 16, column 4 q + lane / 16), y and out in the result layout, which is the B operand's too.
template <class Init, class X>
__device__ __forceinline__ void mul_add(Init &&init, X &&x, const double2 (&y)[4], double sign,
                                        double2 (&out)[4])
{
    doublex4 re, im;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double2 v = init(e);
        re[e] = v.x;
        im[e] = v.y;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double2 v = x(q);
        const double vx = sign * v.x, vy = sign * v.y;
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(vx, y[q].x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(vx, y[q].y, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-vy, y[q].y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(vy, y[q].x, im, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = make_double2(re[e], im[e]);
}

template <int NW>
__device__ __forceinline__ void noise_factor_bin(const double2 *__restrict__ Kf,
                                                 double2 *__restrict__ Wf,
                                                 int32_t *__restrict__ stf, int M)
{
    typedef FactorCfg<NW> C;
    __shared__ double2 rowp[16 * C::LD];           // [pivot][column]: block row k, then P^{-1} of it
    __shared__ double2 colp[16 * C::LD];           // [pivot][row]: block column k
    __shared__ double dmax_s[NW];
    __shared__ int bad_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kl = lane >> 4, cl = lane & 15;

    double2 a[NW][4];
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 16 * wave + kl + 4 * e, c = 16 * j + cl;
            a[j][e] = r < M && c < M ? gload(Kf + (size_t)r * M + c) : make_double2(0.0, 0.0);
        }
    // the largest diagonal entry (NaN if one is not finite: no pivot then passes)
    double dm = 0.0;
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j == wave && kl + 4 * e == cl && !(a[j][e].x <= dm)) dm = a[j][e].x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double v = __shfl_xor(dm, o);
        if (dm == dm && !(v <= dm)) dm = v;            // a NaN on either side stays
    }
    if (lane == 0) dmax_s[wave] = dm;
    if (tid == 0) bad_s = 0;
    __syncthreads();
    dm = 0.0;
    bool fin = true;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        fin = fin && isfinite(dmax_s[w]);
        dm = fmax(dm, dmax_s[w]);
    }
    const double thr = kPdRel * dm;
    bool bad = !fin || !(dm > 0.0);
    const int nb = (M + 15) >> 4;
    // In step k register tile j is column tile (j + k) mod NW: the loop stays rolled (straight-line code
    // for every k would not fit the instruction cache), and the tiles are back in place at its end.
#pragma unroll 1
    for (int k = 0; k < NW; ++k) {
        if (k < nb && !bad) {                          // uniform
            const int ow = 16 * wave, ok = 16 * k;
            // block column k from every wave, block row k from wave k
#pragma unroll
            for (int e = 0; e < 4; ++e) colp[cl * C::LD + ow + kl + 4 * e] = a[0][e];
            if (wave == k) {
                invert_tile(std::make_integer_sequence<int, 16>(), a[0], lane, thr, M - ok, bad);
                if (bad && lane == 0) bad_s = 1;
#pragma unroll
                for (int j = 0; j < NW; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        rowp[(kl + 4 * e) * C::LD + 16 * ((j + k) % NW) + cl] = a[j][e];
            }
            __syncthreads();
            bad = bad_s != 0;
            double2 v[4];                              // V^T, element e: (pivot kl + 4 e, row cl)
            if (wave != k && !bad) {
                // W_kj = P^{-1} W_kj (j = wave), corrected by its residual
                double2 r0[4], w[4], r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r0[e] = rowp[(kl + 4 * e) * C::LD + ow + cl];
                auto inv = [&](int q) { return rowp[cl * C::LD + ok + 4 * q + kl]; };
                mul_add([](int) { return make_double2(0.0, 0.0); }, inv, r0, 1.0, w);
                mul_add([&](int e) { return r0[e]; },
                        [&](int q) { return colp[(4 * q + kl) * C::LD + ok + cl]; }, w, -1.0, r);
                mul_add([&](int e) { return w[e]; }, inv, r, 1.0, w);
#pragma unroll
                for (int e = 0; e < 4; ++e)            // tile `wave` of the panel: read by this wave alone
                    rowp[(kl + 4 * e) * C::LD + ow + cl] = w[e];
                // V = W_ik P^{-1} (i = wave) as V^T = P^{-T} W_ik^T
#pragma unroll
                for (int e = 0; e < 4; ++e) r0[e] = colp[(kl + 4 * e) * C::LD + ow + cl];
                auto invt = [&](int q) { return rowp[(4 * q + kl) * C::LD + ok + cl]; };
                mul_add([](int) { return make_double2(0.0, 0.0); }, invt, r0, 1.0, v);
            }
            __syncthreads();
            if (wave == k) {
#pragma unroll
                for (int j = 1; j < NW; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        a[j][e] = rowp[(kl + 4 * e) * C::LD + 16 * ((j + k) % NW) + cl];
            } else if (!bad) {
                auto cop = [&](int q) { return colp[(4 * q + kl) * C::LD + ow + cl]; };
#pragma unroll
                for (int j = 1; j < NW; ++j) {         // W_ij -= W_ik W_kj
                    double2 y[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        y[q] = rowp[(4 * q + kl) * C::LD + 16 * ((j + k) % NW) + cl];
                    mul_add([&](int e) { return a[j][e]; }, cop, y, -1.0, a[j]);
                }
                // W_ik = -V: the transpose through this wave's part of colp
#pragma unroll
                for (int e = 0; e < 4; ++e) colp[(kl + 4 * e) * C::LD + ow + cl] = v[e];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double2 x = colp[cl * C::LD + ow + kl + 4 * e];
                    a[0][e] = make_double2(-x.x, -x.y);
                }
            }
            __syncthreads();                           // rowp and colp have been read
        }
        if constexpr (NW > 1) {
            double2 t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = a[0][e];
#pragma unroll
            for (int j = 0; j + 1 < NW; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) a[j][e] = a[j + 1][e];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[NW - 1][e] = t[e];
        }
    }
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 16 * wave + kl + 4 * e, c = 16 * j + cl;
            if (r < M && c < M)
                gstore(Wf + (size_t)r * M + c, bad ? make_double2(0.0, 0.0) : a[j][e]);
        }
    if (tid == 0) gstore(stf, (int32_t)(bad ? SSL_BIN_NOT_PD : SSL_BIN_OK));
}

template <int MP>
__global__ __launch_bounds__((FactorCfg<MP / 16>::THREADS)) void noise_factor(const double2 *__restrict__ K,
                                                                    double2 *__restrict__ Kinv,
                                                                    int32_t *__restrict__ status,
                                                                    int M)
{
    const int f = blockIdx.x;
    noise_factor_bin<MP / 16>(K + (size_t)f * M * M, Kinv + (size_t)f * M * M, status + f, M);
}

// Item (handle, bin) of a batched noise update.
template <int MP>
__global__ __launch_bounds__((FactorCfg<MP / 16>::THREADS)) void noise_factor_batch(
    const NoiseUpdDev *__restrict__ h, const int2 *__restrict__ items)
{
    const int2 it = items[blockIdx.x];
    const NoiseUpdDev &H = h[it.x];
    const int M = H.M, f = it.y;
    noise_factor_bin<MP / 16>(H.K + (size_t)f * M * M, H.Kinv + (size_t)f * M * M, H.status + f, M);
}

// K <- alpha K + (1 - alpha) Khat
__global__ void noise_blend_c128(double2 *__restrict__ K, const double2 *__restrict__ Kh,
                                 double alpha, size_t n)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const double2 a = K[e], b = Kh[e];
        K[e] = make_double2(fma(alpha, a.x, (1.0 - alpha) * b.x), fma(alpha, a.y, (1.0 - alpha) * b.y));
    }
}
__global__ void noise_blend_c64(double2 *__restrict__ K, const float2 *__restrict__ Kh,
                                double alpha, size_t n)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const double2 a = K[e];
        const float2 b = Kh[e];
        K[e] = make_double2(fma(alpha, a.x, (1.0 - alpha) * (double)b.x),
                            fma(alpha, a.y, (1.0 - alpha) * (double)b.y));
    }
}

// K <- Kin (complex128 copy or complex64 widened)
__global__ void noise_load_c128(double2 *__restrict__ K, const double2 *__restrict__ Kin, size_t n)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x)
        K[e] = Kin[e];
}
__global__ void noise_load_c64(double2 *__restrict__ K, const float2 *__restrict__ Kin, size_t n)
{
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const float2 v = Kin[e];
        K[e] = make_double2((double)v.x, (double)v.y);
    }
}

// A = K^{-1} R per bin in FP64 on the matrix cores (v_mfma_f64_16x16x4f64: FP64 inputs, FP64
// accumulation).  The complex product takes three real ones (Gauss's trick), W = K^{-1}:
//   P1 = Wr Rr,  P2 = Wi Ri,  P3 = (Wr + Wi)(Rr + Ri);   Re A = P1 - P2,  Im A = P3 - P1 - P2,
// over k-steps of 4: a quarter fewer matrix-core cycles than the four-product form, for an FP64
// rounding error at most a small constant times larger (the sums it rounds are bounded by
// (|Wr| + |Wi|)(|Rr| + |Ri|) instead of |Wr||Ri| + |Wi||Rr|).  A workgroup takes one bin of a noise set for a run of blocks that share it:
// NT = MP / 16 waves, wave w owning rows 16 w .. 16 w + 15 and all NT column tiles.  Its A
// operands (W's rows, FP64) are loaded into registers once and reused for every block of the
// run; each block's R (complex64) is staged in LDS -- the next block's R is loaded into
// registers under the current block's products -- and read as B operands, widened to FP64.
// Padding rows, columns and k-steps (beyond M) are zero on both operands and never stored.

template <int MP> struct WhCfg {
    static constexpr int NT = MP / 16;          // row tiles = column tiles = waves
    static constexpr int THREADS = 64 * NT;
    static constexpr int KQ = MP / 4;           // k-steps at M = MP
    static constexpr int RS = MP + 16;          // LDS row stride (complex64 elements)
    static constexpr int NIT = MP * MP / THREADS;
};

// Thread t stages R elements (k0 + 4u, j), k0 = t / MP, j = t % MP, u < NIT (THREADS = 4 MP).
template <int MP>
__device__ __forceinline__ void load_r(const float2 *__restrict__ Rf, int M, int tid,
                                       float2 (&v)[WhCfg<MP>::NIT])
{
    const int k0 = tid / MP, j = tid % MP;
    const float2 *src = Rf + (size_t)k0 * M + j;
#pragma unroll
    for (int u = 0; u < WhCfg<MP>::NIT; ++u)
        v[u] = (j < M && k0 + 4 * u < M) ? gload(src + (size_t)u * 4 * M) : make_float2(0.f, 0.f);
}

template <int MP>
__device__ __forceinline__ void store_r(const float2 (&v)[WhCfg<MP>::NIT], float2 *Rs, int tid)
{
    const int k0 = tid / MP, j = tid % MP;
#pragma unroll
    for (int u = 0; u < WhCfg<MP>::NIT; ++u) Rs[(k0 + 4 * u) * WhCfg<MP>::RS + j] = v[u];
}

// One workgroup: bin `Wf` (K^{-1} of the bin, [M][M] FP64) for nb blocks; blk(i, Rf, Af) gives
// block i's R and A of the bin.
template <int MP, class BlockAt>
__device__ __forceinline__ void whiten_run(const double2 *__restrict__ Wf, int M, int nb,
                                           BlockAt &&blk)
{
    typedef WhCfg<MP> C;
    __shared__ float2 Rs[MP * C::RS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int KQ = (M + 3) >> 2;
    const int row = 16 * wave + (lane & 15);     // A-operand row of this lane
    const int kl = lane >> 4;                    // k within a k-step (A and B operands)

    double2 w[C::KQ];
#pragma unroll
    for (int q = 0; q < C::KQ; ++q) {
        const int k = 4 * q + kl;
        w[q] = (row < M && k < M) ? gload(Wf + (size_t)row * M + k) : make_double2(0.0, 0.0);
    }

    const float2 *Rf;
    float2 *Af;
    blk(0, Rf, Af);
    {
        float2 v[C::NIT];
        load_r<MP>(Rf, M, tid, v);
        store_r<MP>(v, Rs, tid);
    }
    __syncthreads();
    for (int i = 0; i < nb; ++i) {
        float2 *const cur_A = Af;
        const bool more = i + 1 < nb;
        float2 v[C::NIT];
        if (more) {
            blk(i + 1, Rf, Af);
            load_r<MP>(Rf, M, tid, v);
        }
        doublex4 p1[C::NT], p2[C::NT], p3[C::NT];
#pragma unroll
        for (int ct = 0; ct < C::NT; ++ct) {
            p1[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
            p2[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
            p3[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
        }
#pragma unroll
        for (int q = 0; q < C::KQ; ++q) {
            if (q < KQ) {                        // uniform; w[] stays register-indexed
                const float2 *rrow = Rs + (4 * q + kl) * C::RS + (lane & 15);
                const double ws = w[q].x + w[q].y;
#pragma unroll
                for (int ct = 0; ct < C::NT; ++ct) {
                    const float2 r = rrow[16 * ct];
                    const double br = (double)r.x, bi = (double)r.y;
                    p1[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[q].x, br, p1[ct], 0, 0, 0);
                    p2[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[q].y, bi, p2[ct], 0, 0, 0);
                    p3[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(ws, br + bi, p3[ct], 0, 0, 0);
                }
            }
        }
        doublex4 ar[C::NT], ai[C::NT];
#pragma unroll
        for (int ct = 0; ct < C::NT; ++ct) {
            ar[ct] = p1[ct] - p2[ct];
            ai[ct] = p3[ct] - p1[ct] - p2[ct];
        }
        // FP64 result layout: accumulator element e of lane l is row l / 16 + 4 e, column l % 16
        // of the 16 x 16 tile (rows interleaved, unlike the FP32 16x16x4 layout)
#pragma unroll
        for (int ct = 0; ct < C::NT; ++ct) {
            const int j = 16 * ct + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 16 * wave + kl + 4 * e;
                if (r < M && j < M)
                    gstore(cur_A + (size_t)r * M + j, make_float2((float)ar[ct][e], (float)ai[ct][e]));
            }
        }
        __syncthreads();                         // every wave has read Rs
        if (more) store_r<MP>(v, Rs, tid);
        __syncthreads();
    }
}

template <int MP>
__global__ __launch_bounds__(WhCfg<MP>::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void whiten(const double2 *__restrict__ Kinv,
                                                              const float2 *__restrict__ R,
                                                              float2 *__restrict__ A, int M)
{
    const size_t o = (size_t)blockIdx.x * M * M;
    whiten_run<MP>(Kinv + o, M, 1, [&](int, const float2 *&Rf, float2 *&Af) {
        Rf = R + o;
        Af = A + o;
    });
}

// Batched: item = (chunk, bin); chunks[c] = (first, count) into cblocks, a run of blocks that
// share one noise set (the same K^{-1}).
template <int MP>
__global__ __launch_bounds__(WhCfg<MP>::THREADS) __attribute__((amdgpu_waves_per_eu(2))) void whiten_batch(const BlockDev *__restrict__ blk,
                                                                    const int2 *__restrict__ items,
                                                                    const int2 *__restrict__ chunks,
                                                                    const int *__restrict__ cblocks)
{
    const int2 it = items[blockIdx.x];
    const int2 ch = chunks[it.x];
    const BlockDev &B0 = blk[cblocks[ch.x]];
    const int M = B0.M;
    const size_t o = (size_t)it.y * M * M;
    whiten_run<MP>(B0.Kinv + o, M, ch.y, [&](int i, const float2 *&Rf, float2 *&Af) {
        const BlockDev &B = blk[cblocks[ch.x + i]];
        Rf = B.R + o;
        Af = B.A + o;
    });
}

int grid_for(size_t n) { return (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096); }

}  // namespace

hipError_t launch_noise_factor(ssl_c128 *K, ssl_c128 *Kinv, int32_t *status, int F, int M,
                               hipStream_t st)
{
    const double2 *Kp = reinterpret_cast<const double2 *>(K);
    double2 *Wp = reinterpret_cast<double2 *>(Kinv);
    if (M <= 16)
        hipLaunchKernelGGL(noise_factor<16>, dim3(F), dim3(FactorCfg<1>::THREADS), 0, st, Kp, Wp,
                           status, M);
    else if (M <= 32)
        hipLaunchKernelGGL(noise_factor<32>, dim3(F), dim3(FactorCfg<2>::THREADS), 0, st, Kp, Wp,
                           status, M);
    else
        hipLaunchKernelGGL(noise_factor<64>, dim3(F), dim3(FactorCfg<4>::THREADS), 0, st, Kp, Wp,
                           status, M);
    return hipGetLastError();
}

hipError_t launch_noise_factor_batch(const NoiseUpdDev *h, const int2 *items, int n_items,
                                     int cls, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    if (cls == 16)
        hipLaunchKernelGGL(noise_factor_batch<16>, dim3(n_items), dim3(FactorCfg<1>::THREADS), 0, st,
                           h, items);
    else if (cls == 32)
        hipLaunchKernelGGL(noise_factor_batch<32>, dim3(n_items), dim3(FactorCfg<2>::THREADS), 0, st,
                           h, items);
    else
        hipLaunchKernelGGL(noise_factor_batch<64>, dim3(n_items), dim3(FactorCfg<4>::THREADS), 0, st,
                           h, items);
    return hipGetLastError();
}

hipError_t launch_noise_load(ssl_c128 *K, const void *Kin, ssl_prec kprec, int F, int M,
                             hipStream_t st)
{
    const size_t n = (size_t)F * M * M;
    if (kprec == SSL_FP64)
        hipLaunchKernelGGL(noise_load_c128, dim3(grid_for(n)), dim3(256), 0, st,
                           reinterpret_cast<double2 *>(K), static_cast<const double2 *>(Kin), n);
    else
        hipLaunchKernelGGL(noise_load_c64, dim3(grid_for(n)), dim3(256), 0, st,
                           reinterpret_cast<double2 *>(K), static_cast<const float2 *>(Kin), n);
    return hipGetLastError();
}

hipError_t launch_noise_blend(ssl_c128 *K, const void *Khat, ssl_prec kprec, double alpha, int F,
                              int M, hipStream_t st)
{
    const size_t n = (size_t)F * M * M;
    if (kprec == SSL_FP64)
        hipLaunchKernelGGL(noise_blend_c128, dim3(grid_for(n)), dim3(256), 0, st,
                           reinterpret_cast<double2 *>(K), static_cast<const double2 *>(Khat),
                           alpha, n);
    else
        hipLaunchKernelGGL(noise_blend_c64, dim3(grid_for(n)), dim3(256), 0, st,
                           reinterpret_cast<double2 *>(K), static_cast<const float2 *>(Khat),
                           alpha, n);
    return hipGetLastError();
}

hipError_t launch_whiten(const ssl_c128 *Kinv, const ssl_c64 *R, ssl_c64 *A, int F, int M,
                         hipStream_t st)
{
    const double2 *Wp = reinterpret_cast<const double2 *>(Kinv);
    const float2 *Rp = reinterpret_cast<const float2 *>(R);
    float2 *Ap = reinterpret_cast<float2 *>(A);
    switch (whiten_class(M)) {
    case 16:
        hipLaunchKernelGGL(whiten<16>, dim3(F), dim3(WhCfg<16>::THREADS), 0, st, Wp, Rp, Ap, M);
        break;
    case 32:
        hipLaunchKernelGGL(whiten<32>, dim3(F), dim3(WhCfg<32>::THREADS), 0, st, Wp, Rp, Ap, M);
        break;
    default:
        hipLaunchKernelGGL(whiten<64>, dim3(F), dim3(WhCfg<64>::THREADS), 0, st, Wp, Rp, Ap, M);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_whiten_batch(const BlockDev *blk, const int2 *items, int n_items,
                               const int2 *chunks, const int *cblocks, int cls, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    switch (cls) {
    case 16:
        hipLaunchKernelGGL(whiten_batch<16>, dim3(n_items), dim3(WhCfg<16>::THREADS), 0, st, blk,
                           items, chunks, cblocks);
        break;
    case 32:
        hipLaunchKernelGGL(whiten_batch<32>, dim3(n_items), dim3(WhCfg<32>::THREADS), 0, st, blk,
                           items, chunks, cblocks);
        break;
    default:
        hipLaunchKernelGGL(whiten_batch<64>, dim3(n_items), dim3(WhCfg<64>::THREADS), 0, st, blk,
                           items, chunks, cblocks);
        break;
    }
    return hipGetLastError();
}

int whiten_wg_per_cu(int cls)
{
    // resident workgroups per CU of the batched kernel (registers and LDS decide), cached
    static std::atomic<int> cache[3];
    const int i = cls == 16 ? 0 : cls == 32 ? 1 : 2;
    int n = cache[i].load(std::memory_order_relaxed);
    if (n > 0) return n;
    hipError_t e;
    if (cls == 16)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, whiten_batch<16>, WhCfg<16>::THREADS, 0);
    else if (cls == 32)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, whiten_batch<32>, WhCfg<32>::THREADS, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, whiten_batch<64>, WhCfg<64>::THREADS, 0);
    if (e != hipSuccess || n < 1) return 1;
    cache[i].store(n, std::memory_order_relaxed);
    return n;
}
