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
    const long long r = __builtin_amdgcn_update_dpp(0ll, b, 0x150 + L, 0xF, 0xF, true);
    return __builtin_bit_cast(double, r);
}

// K^{-1} of one bin by in-place Gauss-Jordan elimination in blocks of 16 pivots, NW waves (M <= 16 NW),
// wave w holding rows 16 w .. 16 w + 15 as NW tiles in the FP64 MFMA result layout (element e of lane l:
// row l / 16 + 4 e, column l % 16).  Block step k with P = W_kk = L U (L lower triangular with the
// Schur-complement pivots on its diagonal, U upper with ones):
//   wave k    factors P, 16 scalar steps in one wave (row and column of the pivot by lane exchanges);
//   wave j    takes its tiles of the block row and the block column through the same steps by substitution,
//             W~_j = L^{-1} W_kj and C~_j = W_jk U^{-1}; wave k the identity: L^{-1}, U^{-1};
//   then, on v_mfma_f64_16x16x4f64 (four real products per complex one),
//             W_ij -= C~_i W~_j,  W_kj = U^{-1} W~_j,  W_jk = -C~_j L^{-1},  W_kk = U^{-1} L^{-1}.
// These are the scalar elimination's own sums, 16 pivots at a time.  No product is formed with an explicit
// P^{-1}, whose error of 2^-53 cond(P) the large W_jk would multiply once more: |K^{-1} K - I| is about 2^-53
// cond(K), as with scalar pivots (17 to 64 channels, one to three directional noises or a diffuse one, cond(K)
// up to 1e11; with W_kj = P^{-1} W_kj, corrected once by its residual, 1e6 times as much at 1e8).  A pivot
// that is <= 2^-40 max_i K_ii or not finite marks the bin NOT_PD (the inverse is then zero).  Padding rows
// and columns (>= M) are zero and stay zero, but for ones on the diagonal (their pivots count as 1).
//   Bound by the two chains of 16 steps (of P and of the substitution) and the FP64 matrix cores, about a third
// each.  257 bins of 60 channels: 54 us, five such sets in one launch 150 us (122 and 346 us with one barrier per
// scalar pivot and rank-1 updates on the vector ALU); 257 bins of up to 16 channels 8 us, of 32 channels 20 us.
template <int NW> struct FactorCfg {
    static constexpr int THREADS = 64 * NW;
    static constexpr int LD = 16 * NW + 1;         // LDS row stride, complex128
};

// The factors of a pivot block, [pivot s][i], zero elsewhere: column s of L below the diagonal over -p_s and
// row s of U right of it, for the substitution; the inverses L^{-1} (row s) and U^{-1} (column s); 1 / p_s.
constexpr int kPivLd = 17;
struct PivotBlock {
    double2 low[16 * kPivLd], up[16 * kPivLd], linv[16 * kPivLd], uinv[16 * kPivLd];
    double ip[16];
};

// Lane group G (of 16 lanes) of a wave to all four.
template <int G>
__device__ __forceinline__ int group_bcast(int v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const int h = (G & 1) ? a[1] : a[0];               // groups (0, 0, 2, 2) or (1, 1, 3, 3)
    const auto b = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return (G & 2) ? b[1] : b[0];
}
template <int G>
__device__ __forceinline__ double group_bcast(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = group_bcast<G>((int)b), hi = group_bcast<G>((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Step S of the factorization on the tile of one wave: the entries below and right of pivot S; its column
// and (unscaled) row stay as they are.  No branches, so that the steps overlap: a pivot that fails clears
// ok, those of padding rows (S >= m) count as 1.  ipl: lane l's is that of pivot l % 16, inverted.
template <int S>
__device__ __forceinline__ void pivot_step(double2 (&a)[4], int lane, double thr, int m, bool &ok,
                                           double &ipl)
{
    constexpr int E = S >> 2, G = S & 3;
    const long long pb = __builtin_bit_cast(long long, a[E].x);
    const int lo = __builtin_amdgcn_readlane((int)pb, 16 * G + S);
    const int hi = __builtin_amdgcn_readlane((int)(pb >> 32), 16 * G + S);
    double p = __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
    p = S < m ? p : 1.0;
    ok = ok && (S >= m || (p > thr && p < 1.7e308));   // not NaN or Inf either
    double ip = __builtin_amdgcn_rcp(p);
    ip = fma(ip, fma(-p, ip, 1.0), ip);
    ip = fma(ip, fma(-p, ip, 1.0), ip);
    ipl = (lane & 15) == S ? ip : ipl;
    if constexpr (S < 15) {
        const bool right = (lane & 15) > S;
        const double w = right ? ip : 0.0;
        // the pivot row over -p, zero up to the pivot
        const double wx = -group_bcast<G>(a[E].x) * w, wy = -group_bcast<G>(a[E].y) * w;
#pragma unroll
        for (int e = E; e < 4; ++e) {
            double cx = row_bcast<S>(a[e].x), cy = row_bcast<S>(a[e].y);       // W_is
            if (e == E) {
                const bool below = (lane >> 4) > G;
                cx = below ? cx : 0.0;
                cy = below ? cy : 0.0;
            }
            a[e].x = fma(cx, wx, fma(-cy, wy, a[e].x));
            a[e].y = fma(cx, wy, fma(cy, wx, a[e].y));
        }
    }
}
template <int... S>
__device__ __forceinline__ void factor_tile(std::integer_sequence<int, S...>, double2 (&a)[4],
                                            int lane, double thr, int m, bool &ok, double &ipl)
{
    (pivot_step<S>(a, lane, thr, m, ok, ipl), ...);
}

// Step S of the substitution on b, a tile of the block row transposed (element e: column l / 16 + 4 e, pivot
// l % 16), and c, one of the block column (row l / 16 + 4 e, pivot l % 16): only the pivots after S change.
template <int S>
__device__ __forceinline__ void panel_step(double2 (&b)[4], double2 (&c)[4], int cl, const PivotBlock &pv)
{
    const double2 m = pv.low[S * kPivLd + cl], w = pv.up[S * kPivLd + cl];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double2 r = make_double2(row_bcast<S>(b[e].x), row_bcast<S>(b[e].y));
        const double2 u = make_double2(row_bcast<S>(c[e].x), row_bcast<S>(c[e].y));
        b[e].x = fma(r.x, m.x, fma(-r.y, m.y, b[e].x));
        b[e].y = fma(r.x, m.y, fma(r.y, m.x, b[e].y));
        c[e].x = fma(u.x, w.x, fma(-u.y, w.y, c[e].x));
        c[e].y = fma(u.x, w.y, fma(u.y, w.x, c[e].y));
    }
}
template <int... S>
__device__ __forceinline__ void panel_steps(std::integer_sequence<int, S...>, double2 (&b)[4],
                                            double2 (&c)[4], int cl, const PivotBlock &pv)
{
    (panel_step<S>(b, c, cl, pv), ...);
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
    constexpr int kPanel = NW > 1 ? 16 * C::LD : 1;
    __shared__ double2 rowp[kPanel];               // [pivot][column]: block row k, then W~
    __shared__ double2 colp[kPanel];               // [pivot][row]: C~, each wave its own rows
    __shared__ PivotBlock pv;
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
    for (int i = tid; i < 16 * kPivLd; i += C::THREADS) pv.low[i] = pv.up[i] = make_double2(0.0, 0.0);
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
            const int ow = 16 * wave;
            if (wave == k) {
#pragma unroll
                for (int j = 1; j < NW; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        rowp[(kl + 4 * e) * C::LD + 16 * ((j + k) % NW) + cl] = a[j][e];
                bool ok = true;
                double ipc = 0.0;                      // 1 / p of pivot cl
                factor_tile(std::make_integer_sequence<int, 16>(), a[0], lane, thr, M - 16 * k, ok, ipc);
                if (!ok && lane == 0) bad_s = 1;
                if (lane < 16) pv.ip[lane] = ipc;
#pragma unroll
                for (int e = 0; e < 4; ++e) {          // entry (i, cl): of L below, of U right of the diagonal
                    const int i = kl + 4 * e;
                    const double sc = i > cl ? -ipc : i < cl ? -pv.ip[i] : 0.0;
                    double2 *to = i > cl ? pv.low + cl * kPivLd + i : pv.up + i * kPivLd + cl;
                    *to = make_double2(a[0][e].x * sc, a[0][e].y * sc);
                }
            }
            __syncthreads();
            bad = bad_s != 0;
            double2 b[4], c[4];
            if (!bad) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double one = kl + 4 * e == cl ? 1.0 : 0.0;
                    b[e] = c[e] = make_double2(one, 0.0);
                    if (NW > 1 && wave != k) {
                        b[e] = rowp[cl * C::LD + ow + kl + 4 * e];
                        c[e] = a[0][e];
                    }
                }
                panel_steps(std::make_integer_sequence<int, 15>(), b, c, cl, pv);
                // tile `wave` of the panels is read by this wave alone so far
                const double ip = pv.ip[cl];
                double2 *lb = wave == k ? pv.linv + cl * kPivLd : rowp + cl * C::LD + ow;
                double2 *cb = wave == k ? pv.uinv + cl * kPivLd : colp + cl * C::LD + ow;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    lb[kl + 4 * e] = make_double2(b[e].x * ip, b[e].y * ip);
                    cb[kl + 4 * e] = c[e];
                }
            }
            __syncthreads();
            if (!bad) {
                const bool own = wave == k;
                auto row = [&](int j, double2 (&y)[4]) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        y[q] = rowp[(4 * q + kl) * C::LD + 16 * ((j + k) % NW) + cl];
                };
                const double2 *op = own ? pv.uinv + kl * kPivLd + cl : colp + kl * C::LD + ow + cl;
                const int step = 4 * (own ? kPivLd : C::LD);
                const double sign = own ? 1.0 : -1.0;
                double2 x[4], y[4];                    // U^{-1} or C~
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = op[q * step];
                auto left = [&](int q) { return x[q]; };
#pragma unroll
                for (int j = 1; j < NW; ++j) {
                    row(j, y);
                    mul_add([&](int e) { return own ? make_double2(0.0, 0.0) : a[j][e]; }, left, y, sign, a[j]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) y[q] = pv.linv[(4 * q + kl) * kPivLd + cl];
                mul_add([](int) { return make_double2(0.0, 0.0); }, left, y, sign, a[0]);
            }
            __syncthreads();                           // rowp and the pivot block have been read
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
