// The signal subspace of eq.4 (arXiv 2504.03373) without the full SVD: block subspace iteration on
// A = K^{-1} R, for the signal-subspace form of eq.5 (p = 2, Ns <= 3).
//
// eq.5 then reads only the span of the Ns dominant left singular vectors of A, the invariant
// subspace of A A^H for its Ns largest eigenvalues theta_1 >= theta_2 >= .. (theta = sigma^2).  A
// block of 8 vectors is taken through A A^H and orthonormalised:
//   Y_0 = A Omega (a fixed dense block), V_k = orth(Y_{k-1}), Y_k = A (A^H V_k).
// Every step shrinks what is left of direction j > 8 against direction s <= Ns by theta_j / theta_s,
// so the number of steps depends on theta_9 / theta_Ns: 2 to 4 in nearly every bin of the 60-channel
// workload (median sigma_2 / sigma_3 about 50), more where the sources are not resolved.  Y_0 and
// Y_1 are computed on the FP32 matrix cores (they only have to point the block the right way),
// all else in FP64.
//   From Y_2 on each step is tested: with the Ritz vectors q_S of T = V^H Y to first order and their
// Rayleigh quotient M, r = Y q_S - V q_S M bounds the angle between span V q_S and the wanted subspace
// by the root of sum_s (|r_s| / (theta_s - theta_{Ns+1}))^2, and Y q_S, the result, is nearer by theta_{Ns+1} /
// theta_Ns.  A bin is done once (sum_s (|r_s| / theta_s)^2)^1/2 theta_{Ns+1} <= 2^-24 theta_Ns: its subspace is that
// of A perturbed by the FP32 roundoff of sigma_Ns at most (the Jacobi solve stops at the roundoff of sigma_1).
// Where the first-order vectors do not apply (close singular values across the split), the block is
// rotated to its Ritz vectors by a Jacobi solve of the 8 x 8 Gram matrix; where three steps did not
// suffice, the block is filtered by a Chebyshev polynomial of A A^H before the next, of the degree that the error
// asks for.  The result is stored as complex64 vectors E_s of about unit length with the inverse Cholesky factor
// of their FP64 Gram matrix, as the Jacobi solve does.
//
// A bin that this cannot decide -- theta_Ns below 1e-11 theta_1 (sigma 3e-6: at the numerical rank), no gap behind
// theta_Ns, convergence not in sight of kBudget applications, anything not finite -- is marked
// SSL_BIN_PENDING and its A stored: the Jacobi solve, launched next, takes those bins alone.  It is given up as soon
// as that shows, zero and rank-deficient bins before the first application, since the time spent on it is
// lost.  The magnitude of A does not matter: it is scaled by a power of two first, and the result has unit
// length.
//   One 60-channel block, two sources asked for, us with the whitening and Jacobi launches / with this (257 bins,
// 72 directions, no noise set): one source over a floor 20 dB below 559 / 175, 40 dB below 508 / 689, no source and 50
// frames 476 / 154, 5000 frames 1249 / 934, silence 72 / 73, one source alone 74 / 88, R = I 187 / 241.  Up to 16
// channels long averages of noise alone take longer than before (16 channels, 500 frames: 104 / 148).
//
// What bounds it: the FP64 matrix cores (64 cycles per v_mfma_f64_16x16x4f64 and SIMD: about 11.5k
// for A, 1.9k per FP64 product, 1.3k per step for the small matrices) and, with one block per launch,
// the latency of the 8 x 8 work between products.  One workgroup per bin, NW = ceil(M / 16) waves,
// wave w owning rows 16 w .. 16 w + 15: it forms its rows of A (the whitening product of noise.hip,
// rounded to complex64 through LDS), then keeps its strips of A and A^H in registers as MFMA A
// operands for the whole solve.  Only the block travels through LDS between products, as the real M x 16
// matrix [Re | Im], so that the complex product is two real ones with full 16-column tiles,
//   P = Re(Op) [Vr | Vi],  S = Im(Op) [Vr | Vi];   Yr = P_r - S_i,  Yi = P_i + S_r
// (S moves by 8 lanes: one DPP row rotation).  The FP64 result layout (element e of lane l is row
// l / 16 + 4 e, column l % 16) is at the same time the operand layout of k-step e, so the Gram matrices
// of a wave's rows take four MFMAs straight from the result registers.  The 8 x 8 work runs on one
// complex element per lane, wave 1 (orthonormalisation) beside wave 0 (test).
//   Measured, 128 60-channel blocks per launch (32896 bins): 2.5 ms, where the whitening launch (0.98 ms)
// and the Jacobi launch (6.8 ms) stood before; one block (257 bins): 84 to 105 us by
// input, 18.7 + 505 us before.
//   Up to 16 channels one wave does all of a bin, tests before it orthonormalises, and with up to 8
// starts from the whole range of A, so that one Jacobi solve of the 8 x 8 matrix and one application decide.
// 8 channels, 257 bins: 17.5 us; the whitening and Jacobi launches took 2.5 + 23.5 us.  24 blocks each of 8 and
// of 16 channels with 257 and 513 bins: 0.126 and 0.108 ms (Jacobi: 0.175 and 0.25 ms, whitening 0.017).
#include "signal_out.h"

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kBlk = 8;              // vectors of the block
constexpr int kLd = 18;              // LDS row stride of a block, doubles (16 used: re | im)
constexpr int kMaxSteps = 64;        // applications of A A^H before the Jacobi solve takes the bin
constexpr int kFirstTest = 2;        // first application tested for convergence
constexpr int kSolved = -1, kLeft = -2;                // verdicts besides a filter's degree
constexpr int kMaxSweeps = 12;       // Jacobi sweeps over the 8 x 8 Gram matrix
constexpr double kCouple = 1e-7;     // (S-rest coupling / gap)^2 that the first-order test copes with,
constexpr double kCoupleAll = 1e-9;  // and where the block is the whole space: nothing else is to converge
constexpr int kAccel = 3;            // first step followed by a Chebyshev filter when not done
// A filter of degree d multiplies what V's columns hold of direction 1 (2^-53) by about (4 theta_1 / theta_C)^d, where
// the weakest keeps its length; orth_factor drops a column that is 2^-21 of its own length from the ones before it.
// So d log2(4 theta_1 / theta_C) <= kWideFresh, and kWide where V itself comes from a filtered block and holds more.
constexpr float kWide = 45.0f, kWideFresh = 68.0f;
// Applications that a bin may take: what the Jacobi solve takes in a large batch is about 60 (17 channels and more)
template <int NW> constexpr float kBudget = NW > 1 ? 60.0f : 46.0f;
constexpr double kTol = 5.9604644775390625e-08;      // 2^-24
// theta_Ns / theta_1 below this: left to the Jacobi solve (Y_0 and Y_1 in FP32 no longer hold direction Ns)
constexpr double kRange = 1e-11;

// NW waves, KQ k-steps of 4: M <= 16 NW and M <= 4 KQ
template <int NW, int KQ> struct SubCfg {
    static constexpr int THREADS = 64 * NW;
    static constexpr int MP = 16 * NW;
};

// LDS of a bin.  Before the iteration: R, then A, as complex64 rows of kAs elements.  During it: the
// block V of the step, W = A^H V (and, once W has been read, the 8 x 8 factors in real form: the
// next V = Y B, the test's r = Y BY - V BV), Y (each wave its own rows).
template <int NW> struct SubShared {
    static constexpr int kAs = 16 * NW + 1;
    static constexpr int kN = 16 * NW * kLd;           // doubles of a block
    static constexpr int kMat = 16 * 16;
    union {
        float2 A[16 * NW * kAs];
        struct {
            double V[kN], Y[kN];
            union {
                double W[kN > 3 * kMat ? kN : 3 * kMat];
                struct {
                    double B[kMat], BY[kMat], BV[kMat];
                };
            };
            double part[NW][2][128];     // per wave: its rows' share of Y^H Y and V^H Y (re, im)
        };
    };
    float amax[NW];
    double rpart[NW];                // per wave: its rows' share of |r|^2
    double unit[kBlk];               // scale of the result vectors: 1 / T_ss
    double weight[kBlk];             // of their residuals
    double th1, thS, thR;            // T_00, bounds of theta_Ns (below) and theta_{Ns+1} (above)
    double thC, thD;                 // smallest diagonal entry of T, and among the leading Ns
    int coupled;                     // the first-order Ritz vectors do not apply
    int lost;                        // the start block has fewer than Ns independent columns
};

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
// the value 8 lanes away in the row of 16
__device__ __forceinline__ double ror8(double v) { return dpp_f64<0x128>(v); }

// 1/sqrt(x) for normal x > 0: hardware estimate and two Newton steps
__device__ __forceinline__ double rsqrt64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}

__device__ __forceinline__ double readlane64(double v, int l)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Entry (k, c) of the start block Omega: a fixed number in [-1, 1), the fractional part of n^2 times the root of
// two (in units of 2^-32), n = 16 k + c + 1, which is equidistributed (Weyl).  Dense and unstructured, so that no
// bin's dominant directions are orthogonal to it: condition 2 to 8, and 1.1 at least of the median 2.3 of its
// products with the unit vectors and with waves of any frequency (9 to 64 channels).
__device__ __forceinline__ double omega(int k, int c)
{
    const unsigned int n = (unsigned int)(k * 16 + c + 1);
    return (double)(int)(n * n * 0x6A09E667u) * 4.656612873077393e-10;
}

// One product of a wave's 16-row strip with a block: y[e] = row l / 16 + 4 e, real column l % 16.
// op(q): this lane's operand element (row l % 16, column 4 q + l / 16); in(q): the block's real
// element (row 4 q + l / 16, column l % 16).
template <int KQ, class Op, class In>
__device__ __forceinline__ void strip_product(Op &&op, In &&in, double sgn, double (&y)[4])
{
    doublex4 p = {0.0, 0.0, 0.0, 0.0}, s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        const double2 w = op(q);
        const double b = in(q);
        p = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, b, p, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, b, s, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = fma(sgn, ror8(s[e]), p[e]);
}

// The same on v_mfma_f32_16x16x4f32, for the first applications: y[e] = row 4 (l / 16) + e.
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <int KQ, class Op, class In>
__device__ __forceinline__ void strip_product32(Op &&op, In &&in, double sgn, double (&y)[4])
{
    floatx4 p = {0.f, 0.f, 0.f, 0.f}, s = p;
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        const float2 w = op(q);
        const float b = (float)in(q);
        p = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, b, p, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, b, s, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(
            0, __float_as_int(s[e]), 0x128, 0xF, 0xF, false));
        y[e] = (double)fmaf((float)sgn, o, p[e]);
    }
}

// Coefficients of a Jacobi rotation of the Hermitian 8 x 8 matrix for one column index: the pair
// (lo, hi), lo < hi, of diagonal a, b and entry g = G[lo][hi] becomes
//   x_lo' = v+, x_hi' = v-  with the larger eigenvalue in lo;
// a column c of the pair becomes own * x_c + oth * x_partner.  B = sqrt((1 + |d| / h) / 2), z = g /
// (h B), d = a - b, h = sqrt(d^2 + 4 |g|^2): v+ = (B, conj z), v- = (-z, B) for d >= 0 and v+ = (z, B),
// v- = (B, -conj z) otherwise.  B and z are rounded to FP32: the rotated matrix and the accumulated
// Q see the same coefficients, and orth_factor makes up for their departure from a unitary pair.
struct Rot {
    double2 own, oth;
};
__device__ __forceinline__ Rot rotation(double a, double b, double2 g, bool lower)
{
    const double d = a - b;
    // to FP32 range by a power of two
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fmax(fabs(g.x), fabs(g.y))));
    const float df = (float)__builtin_amdgcn_ldexp(d, ex);
    const float gx = (float)__builtin_amdgcn_ldexp(g.x, ex), gy = (float)__builtin_amdgcn_ldexp(g.y, ex);
    const float g2 = fmaf(gx, gx, gy * gy), h2 = fmaf(df, df, 4.0f * g2);
    float B = 1.0f, zs = 0.0f;
    if (g2 > 0.0f) {
        const float rh = __builtin_amdgcn_rsqf(h2);
        const float B2 = fmaf(0.5f * fabsf(df), rh, 0.5f);
        const float rB = __builtin_amdgcn_rsqf(B2);
        B = B2 * rB;
        zs = rh * rB;
    }
    const double2 z = make_double2((double)(gx * zs), (double)(gy * zs));
    Rot r;
    const double2 Br = make_double2((double)B, 0.0);
    if (d >= 0.0) {
        r.own = Br;
        r.oth = lower ? make_double2(z.x, -z.y) : make_double2(-z.x, -z.y);
    } else {
        r.own = lower ? z : make_double2(-z.x, z.y);
        r.oth = Br;
    }
    return r;
}
__device__ __forceinline__ double2 lin(double2 a, double2 x, double2 b, double2 y)   // a x + b y
{
    return make_double2(fma(a.x, x.x, fma(-a.y, x.y, fma(b.x, y.x, -b.y * y.y))),
                        fma(a.x, x.y, fma(a.y, x.x, fma(b.x, y.y, b.y * y.x))));
}
__device__ __forceinline__ double2 shfl2(double2 v, int l)
{
    return make_double2(__shfl(v.x, l), __shfl(v.y, l));
}
__device__ __forceinline__ double2 conjd(double2 v) { return make_double2(v.x, -v.y); }

// Cyclic Jacobi on the Hermitian 8 x 8 matrix held one element per lane (row l / 8, column l % 8), the
// rotations accumulated into Q, if the first-order Ritz vectors of the test would not do (a squared
// coupling of more than `first` of the gap's square): until the leading Ns indices are decoupled from
// the rest to `couple` (in order) and the rest among themselves enough for the test's bound, or to rounding (`noise`:
// an absolute level of it for G's squared entries; `lost`: the share of the first diagonal entry below which one of
// the leading Ns is not worth it).  The pairs of a round are (i, i ^ m), m = 1 .. 7.
__device__ __forceinline__ void ritz(double2 &G, double2 &Q, int Ns, double first, double couple, double noise,
                                     double lost, int lane)
{
    const int i = lane >> 3, j = lane & 7;
    for (int sw = 0; sw < kMaxSweeps; ++sw) {
        const double di = __shfl(G.x, 9 * i), dj = __shfl(G.x, 9 * j);
        const double g2 = G.x * G.x + G.y * G.y, d = di - dj;
        // the first look decides whether to rotate at all, the later ones when to stop
        const double lim = sw == 0 ? first : couple;
        // columns of numerically orthogonal or vanishing Y_i, Y_j have nothing to rotate
        const bool none = g2 <= 2.0e-28 * fabs(di * dj) || g2 <= noise;
        double ds = readlane64(G.x, 0);                // smallest of the leading diagonal
        if (Ns > 1) ds = fmin(ds, readlane64(G.x, 9));
        if (Ns > 2) ds = fmin(ds, readlane64(G.x, 18));
        if (ds <= lost * readlane64(G.x, 0)) return;   // theta below kRange: it will be given up
        const double below = fmax(ds - di, 0.0);
        bool bad = false;
        if (i < Ns && j >= Ns) bad = !none && !(g2 <= lim * d * d && d > 0.0);
        else if (i >= Ns && j >= Ns && i != j) bad = !none && !(64.0 * g2 <= below * below);
        if (!__any(bad)) return;
#pragma unroll 1
        for (int m = 1; m < 8; ++m) {
            const int jp = j ^ m;
            const int jl = min(j, jp), jh = max(j, jp);
            const Rot c = rotation(__shfl(G.x, 9 * jl), __shfl(G.x, 9 * jh), shfl2(G, 8 * jl + jh),
                                   j < jp);
            Rot r;                                     // index i's, from a lane of column i
            r.own = shfl2(c.own, 9 * i);
            r.oth = shfl2(c.oth, 9 * i);
            const double2 gp = shfl2(G, lane ^ m), qp = shfl2(Q, lane ^ m);
            G = lin(c.own, G, c.oth, gp);
            Q = lin(c.own, Q, c.oth, qp);
            G = lin(conjd(r.own), G, conjd(r.oth), shfl2(G, lane ^ (8 * m)));
            if (i == j) G.y = 0.0;
        }
    }
}

// 1/x for normal x > 0: hardware estimate and one Newton step (about 2^-46)
__device__ __forceinline__ double rcp64(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}

// B = Q L^{-H} with Q^H G Q = L L^H (its rotated form in G), so that Y B is orthonormal: Gaussian
// elimination of [G | Q^H], the rows scaled by the pivots' roots at the end, to L^{-1} Q^H = B^H.  A
// column that depends on the ones before it to 1e-13 of its squared norm is dropped (zero in B).
// Returns element (i, j) of B^H.
__device__ __forceinline__ double2 orth_factor(double2 G, double2 Q, int lane)
{
    const int i = lane >> 3, j = lane & 7;
    double2 a = conjd(shfl2(Q, 8 * j + i));
    const double d0 = G.x;
    double piv = 0.0;                                  // row i's pivot (0: dropped)
#pragma unroll
    for (int k = 0; k < kBlk; ++k) {
        const double2 gk = shfl2(G, 8 * k + j), ak = shfl2(a, 8 * k + j);
        double2 mk = shfl2(G, 8 * i + k);
        const double dk = readlane64(G.x, 9 * k), ok = readlane64(d0, 9 * k);
        const double inv = dk > 1e-13 * ok && dk > 0.0 ? rcp64(dk) : 0.0;
        mk = make_double2(mk.x * inv, mk.y * inv);
        if (i == k) piv = inv > 0.0 ? dk : 0.0;
        if (i > k) {
            G = make_double2(fma(-mk.x, gk.x, fma(mk.y, gk.y, G.x)),
                             fma(-mk.x, gk.y, fma(-mk.y, gk.x, G.y)));
            a = make_double2(fma(-mk.x, ak.x, fma(mk.y, ak.y, a.x)),
                             fma(-mk.x, ak.y, fma(-mk.y, ak.x, a.y)));
        }
    }
    const double sc = piv > 0.0 ? rsqrt64(piv) : 0.0;
    return make_double2(a.x * sc, a.y * sc);
}

// Element (k, c) of a complex 8 x 8 matrix into the real 16 x 16 form [re, im; -im, re]
__device__ __forceinline__ void put_real(double *B, int k, int c, double2 v)
{
    B[16 * k + c] = v.x;
    B[16 * k + c + 8] = v.y;
    B[16 * (k + 8) + c] = -v.y;
    B[16 * (k + 8) + c + 8] = v.x;
}

// Sum over the 16 lanes of a row (all lanes get it) and over the wave
__device__ __forceinline__ double row_sum(double v)
{
    v += dpp_f64<0x128>(v);
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x122>(v);
    v += dpp_f64<0x121>(v);
    return v;
}

// The test's Ritz vectors to first order, from T = V^H Y (one element per lane): with S = the leading
// Ns indices, q_S = [I; X], X_js = T_js / (T_ss - T_jj) on the others, M = the leading rows of T q_S,
// so that r = Y q_S - V q_S M is the residual of the subspace V q_S.  Writes q_S and q_S M (real
// form, zero in the other columns), bounds on theta and whether the coupling is too large for this.
template <class Sh>
__device__ __forceinline__ void prepare_test(double2 t, int Ns, int lane, Sh &sh)
{
    const int i = lane >> 3, j = lane & 7;
    const double di = __shfl(t.x, 9 * i), dj = __shfl(t.x, 9 * j);
    const bool cross = i >= Ns && j < Ns;
    const double gap = dj - di;
    const double ig = cross && gap > 0.0 ? rcp64(gap) : 0.0;
    double2 q = make_double2(t.x * ig, t.y * ig);
    const bool big = cross && !(gap > 0.0 && fma(q.x, q.x, q.y * q.y) <= 0.01);
    if (!cross) q = make_double2(i == j && j < Ns ? 1.0 : 0.0, 0.0);
    double2 w = make_double2(0.0, 0.0);                // T q_S
#pragma unroll 2
    for (int k = 0; k < kBlk; ++k) {
        const double2 a = shfl2(t, 8 * i + k), b = shfl2(q, 8 * k + j);
        w = make_double2(fma(a.x, b.x, fma(-a.y, b.y, w.x)), fma(a.x, b.y, fma(a.y, b.x, w.y)));
    }
    double2 v = make_double2(0.0, 0.0);                // q_S M
    for (int k = 0; k < Ns; ++k) {
        const double2 a = shfl2(q, 8 * i + k), b = shfl2(w, 8 * k + j);
        v = make_double2(fma(a.x, b.x, fma(-a.y, b.y, v.x)), fma(a.x, b.y, fma(a.y, b.x, v.y)));
    }
    put_real(sh.BY, i, j, q);
    put_real(sh.BV, i, j, v);
    // Gershgorin: theta_{Ns+1} <= max of the absolute row sums over the other indices; theta_Ns >= the
    // smallest diagonal less its scaled row's off-diagonal sum over S (Ns = 2: the exact value)
    const double at = fabs(t.x) + fabs(t.y);
    double rs = i >= Ns && j >= Ns ? at : 0.0;
    double lo = 0.0;
    if (Ns > 2 && i < Ns && j < Ns && i != j) {
        // rows scaled by the diagonal's roots: a row far below the first's keeps its bound
        const double wi = rsqrt64(fmax(di, 1e-200)), wj = rsqrt64(fmax(dj, 1e-200));
        lo = at * (di * wi * wj);
    }
    double sm = di, sd = i < Ns ? di : 1e300;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
        rs += __shfl_xor(rs, o);
        lo += __shfl_xor(lo, o);
    }
    lo = i < Ns ? di - lo : 1e300;
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) {
        rs = fmax(rs, __shfl_xor(rs, o));
        lo = fmin(lo, __shfl_xor(lo, o));
        sm = fmin(sm, __shfl_xor(sm, o));
        sd = fmin(sd, __shfl_xor(sd, o));
    }
    const double t0 = readlane64(t.x, 0);
    if (Ns == 2) {
        const double t1 = readlane64(t.x, 9), gx = readlane64(t.x, 1), gy = readlane64(t.y, 1);
        const double h = 0.5 * fabs(t0 - t1), g2 = fma(gx, gx, gy * gy);
        lo = fmin(t0, t1) - (g2 > 0.0 ? g2 / (h + sqrt(fma(h, h, g2))) : 0.0);
    }
    const bool any_big = __any(big);
    // residuals count against their own Ritz value where those of S do not mix, |T_ij| <= min(T_ii, T_jj)
    const bool mixed = __any(i < Ns && j < Ns && i != j && at > fmin(di, dj));
    if (i == j) {
        const double u = j < Ns && dj > 0.0 ? rcp64(dj) : 0.0;
        sh.unit[j] = u;
        sh.weight[j] = j < Ns ? (mixed ? rcp64(fmax(sd, 1e-300)) : u) : 0.0;
    }
    if (lane == 0) {
        sh.th1 = t0;
        sh.thS = lo;
        sh.thR = rs;
        sh.thC = sm;
        sh.thD = sd;
        sh.coupled = any_big ? 1 : 0;
    }
}

// One bin.  Kf: K^{-1} of the bin ([M][M] FP64) or null (SEVD-MUSIC: A = R); Rf, Af: [M][M] complex64,
// Af written only where the Jacobi solve will read it (never with Kf null: A is R there).  stf: the status
// that the Jacobi solve looks at; outf: the caller's copy of a final one, or null.  False where the Jacobi solve
// has to follow.
template <int NW, int KQ>
__device__ __forceinline__ bool subspace_bin(const double2 *__restrict__ Kf, int kst,
                                             const float2 *__restrict__ Rf, float2 *__restrict__ Af,
                                             int M, int Ns, bool keep_a, int32_t *__restrict__ stf,
                                             int32_t *__restrict__ outf,
                                             float2 *__restrict__ Esf, double2 *__restrict__ Lf)
{
    typedef SubShared<NW> Sh;
    constexpr int MP = 16 * NW, NT = 64 * NW, kAs = Sh::kAs;
    __shared__ Sh sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int kl = lane >> 4, cl = lane & 15;
    const int row = 16 * wave + cl;                    // A-operand row of this lane
    const double sgn = cl < 8 ? -1.0 : 1.0;

    if (kst != SSL_BIN_OK) {                           // uniform: the noise set failed in this bin
        if (tid == 0) gstore(stf, (int32_t)kst);
        if (tid == 0 && outf) gstore(outf, (int32_t)kst);
        return true;
    }
    {
        double2 kw[KQ];                                // this wave's rows of K^{-1}
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const int k = 4 * q + kl;
            kw[q] = Kf && row < M && k < M ? gload(Kf + (size_t)row * M + k)
                                           : make_double2(0.0, 0.0);
        }
        float2 v[MP * MP / NT];
#pragma unroll
        for (int u = 0; u < MP * MP / NT; ++u) {
            const int k = (tid + NT * u) / MP, j = tid % MP;
            v[u] = k < M && j < M ? gload(Rf + (size_t)k * M + j) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < MP * MP / NT; ++u) sh.A[(tid + NT * u) / MP * kAs + tid % MP] = v[u];
        __syncthreads();
        if (Kf) {
            // A = K^{-1} R in FP64, rounded to complex64: the whitening product (noise.hip)
            float2 at[NW][4];
#pragma unroll
            for (int ct = 0; ct < NW; ++ct) {
                __builtin_amdgcn_sched_barrier(0);     // one tile's operands at a time
                const float2 *rc = sh.A + kl * kAs + 16 * ct + cl;
                doublex4 p1 = {0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
#pragma unroll
                for (int q = 0; q < KQ; ++q) {
                    const float2 r = rc[4 * q * kAs];
                    const double br = (double)r.x, bi = (double)r.y;
                    asm volatile("" : "+v"(kw[q].x));  // keeps re + im from being held for all q
                    p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(kw[q].x, br, p1, 0, 0, 0);
                    p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(kw[q].y, bi, p2, 0, 0, 0);
                    p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(kw[q].x + kw[q].y, br + bi, p3, 0, 0, 0);
                }
                const doublex4 ar = p1 - p2, ai = p3 - p1 - p2;
#pragma unroll
                for (int e = 0; e < 4; ++e) at[ct][e] = make_float2((float)ar[e], (float)ai[e]);
            }
            __syncthreads();                           // every wave has read R
#pragma unroll
            for (int ct = 0; ct < NW; ++ct)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sh.A[(16 * wave + kl + 4 * e) * kAs + 16 * ct + cl] = at[ct][e];
            __syncthreads();
        }
    }
    // operand strips: this wave's rows of A and of A^H, scaled by a power of two to max |re|, |im| in
    // [0.5, 1) (sigma^2 stays in FP32 range)
    float2 aw[KQ], hw[KQ];
    float amax = 0.0f;
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        aw[q] = sh.A[row * kAs + 4 * q + kl];
        hw[q] = sh.A[(4 * q + kl) * kAs + row];
        amax = fmaxf(amax, fmaxf(fabsf(aw[q].x), fabsf(aw[q].y)));
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
    if (lane == 0) sh.amax[wave] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) amax = fmaxf(amax, sh.amax[w]);
    const int ex = amax > 0.0f ? __builtin_amdgcn_frexp_expf(amax) : 0;
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        aw[q] = make_float2(ldexpf(aw[q].x, -ex), ldexpf(aw[q].y, -ex));
        hw[q] = make_float2(ldexpf(hw[q].x, -ex), ldexpf(hw[q].y, -ex));
    }
    // (the widening stays in the loop: hoisted, the strips would take twice the registers)
    auto opa = [&](int q) {
        asm volatile("" : "+v"(aw[q].x), "+v"(aw[q].y));
        return make_double2((double)aw[q].x, (double)aw[q].y);
    };
    auto oph = [&](int q) {
        asm volatile("" : "+v"(hw[q].x), "+v"(hw[q].y));
        return make_double2((double)hw[q].x, -(double)hw[q].y);
    };
    const int rd = kl * kLd + cl;                      // block element (row kl, column cl)
    const int wr = (16 * wave + kl) * kLd + cl;        // this wave's result rows kl + 4 e
    auto from = [&](const double *b) { return [=](int q) { return b[rd + 4 * q * kLd]; }; };
    auto store = [&](double *b, const double (&y)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) b[wr + 4 * e * kLd] = y[e];
    };
    const int wr32 = (16 * wave + 4 * kl) * kLd + cl;  // the FP32 products' rows 4 kl + e
    auto store32 = [&](double *b, const double (&y)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) b[wr32 + e * kLd] = y[e];
    };
    auto opa32 = [&](int q) { return aw[q]; };
    auto oph32 = [&](int q) { return make_float2(hw[q].x, -hw[q].y); };

    double y[4];
    double v[4] = {0.0, 0.0, 0.0, 0.0};                // V on this wave's rows
    // M <= 8: the block starts as A itself (its whole range) and only has to be turned to the Ritz vectors
    constexpr bool whole = 4 * KQ <= kBlk;
    if constexpr (whole) {
        strip_product<KQ>(opa, [&](int q) { return 4 * q + kl == cl ? 1.0 : 0.0; }, sgn, y);       // A
    } else {
        strip_product32<KQ>(opa32, [&](int q) { return omega(4 * q + kl, cl); }, sgn, y);
    }
    // a wave's rows' share of a Gram matrix a^H b, combined to the complex 8 x 8 form
    auto gram = [&](const double (&a)[4], const double (&b)[4], double *out) {
        doublex4 s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], s, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 2; ++e)
            out[(cl >> 3) * 64 + 8 * (kl + 4 * e) + (cl & 7)] = fma(-sgn, ror8(s[e + 2]), s[e]);
    };
    auto sum_parts = [&](int m) {
        double2 g = make_double2(0.0, 0.0);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            g.x += sh.part[w][m][lane];
            g.y += sh.part[w][m][64 + lane];
        }
        return g;
    };
    bool plain = true;                                 // y = A A^H V (not a filtered block)
    bool fresh = true;                                 // V is not from a filtered block
    // the test: r = Y q_S - V q_S M on this wave's rows
    auto residual = [&] {
        doublex4 zz = {0.0, 0.0, 0.0, 0.0}, x = zz;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * q + kl, o = 16 * k + cl;
            zz = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.Y[row * kLd + k], sh.BY[o], zz, 0, 0, 0);
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.V[row * kLd + k], sh.BV[o], x, 0, 0, 0);
        }
        const double un = sh.weight[cl & 7];
        double n2 = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d = (zz[e] - x[e]) * un;
            n2 = fma(d, d, n2);
        }
        n2 = row_sum(n2);
        n2 += __shfl_xor(n2, 16);
        n2 += __shfl_xor(n2, 32);
        if (lane == 0) sh.rpart[wave] = n2;
    };
    // What a test says: solved, given up, or the degree of the filter that follows (0, 1: none).  The same in
    // every thread, and known to be, so that the branches on it are uniform.
    auto verdict = [&](int step, bool fresh) {
        const double th1 = sh.th1, thS = sh.thS, thR = sh.thR, thC = sh.thC;
        double off = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) off += sh.rpart[w];
        const double err2 = off * (thR * thR), tol2 = (kTol * thS) * (kTol * thS);
        const bool apart = sh.coupled == 0 && thR < thS;
        int next = 0;
        if (apart && thS >= kRange * th1 && err2 <= tol2) {
            next = kSolved;
        } else if (step >= kMaxSteps || !(th1 > 0.0) || sh.thD < 0.0625 * kRange * th1) {
            next = kLeft;
        } else if ((step > kFirstTest || whole) && sh.thD < kRange * th1) {
            next = kLeft;
        } else if ((step > kFirstTest || whole) && thS > 0.0) {    // the block has been turned to its Ritz vectors
            // bits that the error has to lose, and loses in an application: thC / thS in a plain one, the
            // growth of the Chebyshev polynomials at 2 thS / thC - 1 in a filter
            const float need = 0.5f * __log2f((float)(err2 / tol2));
            const float c = (float)(thS / thC), x = 2.0f * c - 1.0f;
            const int wide = (int)((fresh ? kWideFresh : kWide) / __log2f((float)(4.0 * th1 / thC)));
            const float gain = wide > 1 ? __log2f(x + sqrtf(fmaxf(fmaf(x, x, -1.0f), 0.0f))) : __log2f(c);
            if ((thC > 0.0 && !((kBudget<NW> - (float)step) * gain >= 1.3f * need)) ||
                (!apart && need <= 0.0f && step > kFirstTest + 3))             // no gap
                next = kLeft;
            else if (apart && wide > 1 && step >= kAccel && thC > kRange * thS)
                next = min(max((int)ceilf((need + 1.0f) / gain), 2), min(wide, step));
        }
        return __builtin_amdgcn_readfirstlane(next);
    };
    int next = kLeft;
    constexpr int kStart = whole ? kFirstTest - 1 : 0;
    for (int step = kStart; __builtin_amdgcn_readfirstlane(amax > 0.0f);) {
        const bool test = step >= kFirstTest && plain;
        // what depends on the lane is made where it is used, not held in registers from before the loop
        int ln = lane;
        asm volatile("" : "+v"(ln), "+v"(kl), "+v"(cl));
        gram(y, y, sh.part[wave][0]);
        if (test) gram(v, y, sh.part[wave][1]);
        if (step < kFirstTest && !whole) store32(sh.Y, y);
        else store(sh.Y, y);                           // own rows only: the operand of Y B, Y BY
        __syncthreads();
        if (NW == 1 && test) {                         // nobody to orthonormalise beside the test
            prepare_test(sum_parts(1), Ns, ln, sh);
            __syncthreads();
            residual();
            __syncthreads();
            next = verdict(step, fresh);
            if (next < 0) break;
        }
        if (wave == (NW > 1 ? 1 : 0)) {
            double2 G = sum_parts(0);
            const int i = ln >> 3, j = ln & 7;
            if (i == j) G.y = 0.0;
            double2 Q = make_double2(i == j ? 1.0 : 0.0, 0.0);
            if (step >= kFirstTest || whole)
                ritz(G, Q, Ns, whole ? kCoupleAll : step == kFirstTest ? 1e-2 : kCouple, whole ? kCoupleAll : kCouple,
                     step < kFirstTest ? 2e-28 : 0.0, plain && !whole ? 1e-23 : 0.0, ln);
            const double2 a = orth_factor(G, Q, ln);
            if (step == kStart) {
                const bool gone = whole ? G.x < kRange * readlane64(G.x, 0) : a.x == 0.0 && a.y == 0.0;
                const bool lost = __any(i == j && i < Ns && gone);
                if (ln == 0) sh.lost = lost ? 1 : 0;
            }
            put_real(sh.B, j, i, conjd(a));
        }
        if (NW > 1 && wave == 0 && test) prepare_test(sum_parts(1), Ns, ln, sh);
        __syncthreads();
        // V' = Y B and, for the test, r, on this wave's rows
        doublex4 vn = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * q + kl;
            vn = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.Y[row * kLd + k], sh.B[16 * k + cl], vn, 0, 0, 0);
        }
        if (NW > 1 && test) residual();
        {
            const double vs[4] = {vn[0], vn[1], vn[2], vn[3]};
            store(sh.V, vs);
        }
        __syncthreads();
        if (step == kStart && __builtin_amdgcn_readfirstlane(sh.lost)) break;
        if (NW > 1 && test) {
            next = verdict(step, fresh);
            if (next < 0) break;
        }
        if (test && next > 0) {
            // slow bin: the block filtered by the Chebyshev polynomial of A A^H on [0, thC], thC the smallest
            // Ritz value: W_0 = V, W_1 = (a A A^H - 1) V, W_{k+1} = 2 (a A A^H - 1) W_k - W_{k-1}, from the V
            // and Y at hand
            const double a2 = 2.0 / sh.thC;
            double w1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w1[e] = fma(a2, y[e], -v[e]);
#pragma unroll 1
            for (int d = 1; d < next; ++d) {
                __syncthreads();                       // V and thC have been read
                store(sh.V, w1);
                __syncthreads();
                strip_product<KQ>(oph, from(sh.V), sgn, y);
                store(sh.W, y);
                __syncthreads();
                strip_product<KQ>(opa, from(sh.W), sgn, y);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double w0 = v[e];
                    v[e] = w1[e];
                    w1[e] = fma(2.0, fma(a2, y[e], -w1[e]), -w0);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = w1[e];
            plain = false;
            step += next - 1;
            continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = sh.V[wr + 4 * e * kLd];
        fresh = plain;
        plain = true;
        ++step;
        if (step < kFirstTest) {
            strip_product32<KQ>(oph32, from(sh.V), sgn, y);
            store32(sh.W, y);                          // B, BY, BV were read before the barrier above
            __syncthreads();
            strip_product32<KQ>(opa32, from(sh.W), sgn, y);
        } else {
            strip_product<KQ>(oph, from(sh.V), sgn, y);
            store(sh.W, y);
            __syncthreads();
            strip_product<KQ>(opa, from(sh.W), sgn, y);
        }
    }

    const bool solved = next == kSolved;
    if (solved) {
        // the vectors Y q_s (about unit length), rounded to complex64, and their FP64 Gram matrix
        const double un = sh.unit[cl & 7];
        doublex4 zz = {0.0, 0.0, 0.0, 0.0};            // Y and BY as the test read them
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 4 * q + kl;
            zz = __builtin_amdgcn_mfma_f64_16x16x4f64(sh.Y[row * kLd + k], sh.BY[16 * k + cl], zz, 0, 0, 0);
        }
        double ef[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float own = (float)(zz[e] * un);
            ef[e] = (double)own;
            const float im = (float)ror8(ef[e]);
            const int r = 16 * wave + kl + 4 * e;
            if (cl < Ns && r < M) gstore(Esf + (size_t)cl * M + r, make_float2(own, im));
        }
        gram(ef, ef, sh.part[wave][0]);
        if (tid == 0) gstore(stf, (int32_t)SSL_BIN_OK);
        if (tid == 0 && outf) gstore(outf, (int32_t)SSL_BIN_OK);
        __syncthreads();
        if (wave == 0) {
            const double2 g = sum_parts(0);            // e_i^H e_j
            double gr[6], gi[6];
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int s2 = 0; s2 <= t; ++s2) {
                    gr[t * (t + 1) / 2 + s2] = readlane64(g.x, 8 * s2 + t);
                    gi[t * (t + 1) / 2 + s2] = s2 == t ? 0.0 : readlane64(g.y, 8 * s2 + t);
                }
            if (lane == 0) write_inverse_factor(gr, gi, true, Ns, Lf);
        }
    } else if (tid == 0) {
        gstore(stf, (int32_t)SSL_BIN_PENDING);
    }
    if (Kf && (!solved || keep_a)) {                   // A for the Jacobi solve, from the row strips
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const int k = 4 * q + kl;
            if (row < M && k < M)
                gstore(Af + (size_t)row * M + k,
                       make_float2(ldexpf(aw[q].x, ex), ldexpf(aw[q].y, ex)));
        }
    }
    return solved;
}

template <int NW, int KQ>
__global__ __launch_bounds__((SubCfg<NW, KQ>::THREADS))
__attribute__((amdgpu_waves_per_eu(2))) void subspace_single(
    const double2 *__restrict__ Kinv, const int32_t *__restrict__ kstatus,
    const float2 *__restrict__ R, float2 *__restrict__ A, int M, int Ns,
    int32_t *__restrict__ status, int32_t *__restrict__ status_out, float2 *__restrict__ Es,
    double2 *__restrict__ Esl)
{
    const int f = blockIdx.x;
    const size_t o = (size_t)f * M * M;
    subspace_bin<NW, KQ>(Kinv ? Kinv + o : nullptr, kstatus ? kstatus[f] : SSL_BIN_OK, R + o, A + o,
                         M, Ns, false, status + f, status_out ? status_out + f : nullptr,
                         Es + (size_t)f * Ns * M, Esl + 6 * (size_t)f);
}

// Item = (block, bin).  Lists the items that the Jacobi launch takes: those not solved here, and those of blocks
// that ask for the Jacobi statistics.
template <int NW, int KQ>
__global__ __launch_bounds__((SubCfg<NW, KQ>::THREADS))
__attribute__((amdgpu_waves_per_eu(3))) void subspace_batch(
    const BlockDev *__restrict__ blk, const int2 *__restrict__ items, LeftBins left, int first)
{
    const int2 it = items[blockIdx.x];
    const BlockDev &B = blk[it.x];
    const int f = it.y, M = B.M, Ns = B.Ns;
    const size_t o = (size_t)f * M * M;
    const bool whiten = B.Kinv && !B.Kisq;             // GEVD: A = C = W R W is there already
    const bool stats = B.conv != nullptr;
    const bool solved = subspace_bin<NW, KQ>(whiten ? B.Kinv + o : nullptr, B.kstatus ? B.kstatus[f] : SSL_BIN_OK,
                                             (B.Kisq ? B.A : B.R) + o, B.A + o, M, Ns, stats, B.status + f,
                                             B.status_out ? B.status_out + f : nullptr,
                                             B.Es + (size_t)f * Ns * M, B.Esl + 6 * (size_t)f);
    if (threadIdx.x == 0 && (!solved || stats)) {
        const int l = (first + (int)blockIdx.x) % kLeftLists;
        left.list(l)[atomicAdd(left.queue + kLeftStride * l, 1u)] = it;
    }
}

// Calls fn.template operator()<NW, KQ>() for a subspace class.
template <class Fn>
hipError_t with_class(int cls, Fn &&fn)
{
    switch (cls) {
    case 8: return fn.template operator()<1, 2>();
    case 16: return fn.template operator()<1, 4>();
    case 32: return fn.template operator()<2, 8>();
    case 48: return fn.template operator()<3, 12>();
    case 60: return fn.template operator()<4, 15>();
    case 64: return fn.template operator()<4, 16>();
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_subspace(const ssl_c128 *Kinv, const int32_t *kstatus, const ssl_c64 *R,
                           ssl_c64 *A, int F, int M, int Ns, int32_t *bin_status,
                           int32_t *status_out, ssl_c64 *Es, ssl_c128 *Esl, hipStream_t st)
{
    return with_class(subspace_class(M), [&]<int NW, int KQ>() {
        hipLaunchKernelGGL((subspace_single<NW, KQ>), dim3(F), dim3(SubCfg<NW, KQ>::THREADS), 0, st,
                           reinterpret_cast<const double2 *>(Kinv), kstatus,
                           reinterpret_cast<const float2 *>(R), reinterpret_cast<float2 *>(A), M,
                           Ns, bin_status, status_out, reinterpret_cast<float2 *>(Es),
                           reinterpret_cast<double2 *>(Esl));
        return hipGetLastError();
    });
}

hipError_t launch_subspace_batch(const BlockDev *blk, const int2 *items, int n_items, int cls,
                                 const LeftBins &left, int first, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    return with_class(cls, [&]<int NW, int KQ>() {
        hipLaunchKernelGGL((subspace_batch<NW, KQ>), dim3(n_items), dim3(SubCfg<NW, KQ>::THREADS), 0,
                           st, blk, items, left, first);
        return hipGetLastError();
    });
}
