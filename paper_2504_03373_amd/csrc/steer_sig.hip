// MUSIC pseudo-spectrum, eq.5 of arXiv 2504.03373 with p = 2, through the signal subspace.
//
// With U = [E_s E_n] unitary, sum over the noise vectors of |h^H e|^2 = |h|^2 - |E_s^H h|^2, so the
// denominator needs the Ns signal vectors instead of the M - Ns noise vectors (2 instead of 58 on
// the 60-channel workload).  The difference cancels where h lies close to the signal subspace --
// at the peaks -- so it is formed in FP64 from FP64 products of the stored complex64 inputs, and
// with the exact projector onto span E_s, E_s (E_s^H E_s)^{-1} E_s^H (the Jacobi solve supplies
// L^{-1}, L the Cholesky factor of the Gram matrix in FP64), so that the O(2^-24) departure of the
// stored vectors from orthonormality does not enter:
//   g = E_s^H h (FP64),   den = |h|^2 - |L^{-1} g|^2,   P = |h|^2 / max(den, FLT_MIN).
// What remains of the stored vectors' rounding is a rotation of their span, whose effect on den is
// first order in sqrt(den), as for the noise-vector form (the solver's own subspace error enters
// both forms the same way).
//
// Workgroup = 4 waves x 16 directions of one bin; a wave keeps its 16 rows of H in registers
// (complex64) and computes g for a tile of up to 16 signal vectors, those of the next blocks sharing the
// steering table (listed by Ns, their columns packed without gaps), staged in LDS, with
//   Re g = sum a c + b d,   Im g = sum b c - a d     (h = a + ib, e = c + id, FP64 operands:
// g_s = e_s^H h, the conjugate of h^H e_s, so that y = L^{-1} g with L from E_s^H E_s = L L^H),
// on three real products instead of four (Gauss's trick): P1 = sum a c, P2 = sum b (-d),
// P3 = sum (a + b)(c - d), Re g = P1 - P2, Im g = P3 - P1 - P2.  a + b and c - d are sums of two
// FP32-representable values, exact in FP64 unless their exponents differ by more than 29.
//   A tile takes v_mfma_f64_16x16x4f64 (64 cycles per k-step and product whatever it holds); a single
// block, 1 to 3 columns, v_mfma_f64_4x4x4f64 (22 cycles for 4 columns).  Both give a column the same
// bits (same k order and rounding, checked bit for bit), so a block's result does not depend on
// the tile it shares.  A k-step holds elements 8 p + 2
// (l / 16) + h, h = 0 or 1, so that a lane loads the two of k-steps 2 p and 2 p + 1 at once (16
// bytes) where rows are 16-byte aligned.
//   FP64 vector instructions do not run beside FP64 MFMAs (measured: each adds its own 4.5 cycles), so
// the epilogue is kept short: reciprocal by Newton steps instead of a division, one lane per
// (block, direction) with consecutive lanes on consecutive directions.
//   Measured (60 channels, 257 bins, 1368 directions): one block 47 us (68 us with 16-column tiles and
// 8-byte loads; the 169 MB table alone takes 34 us at copy rate), 128 blocks 0.78 ms (as before; the
// FP64 MFMAs alone take 0.43 ms).  Blocks of 8, 16, 32 and 60 channels, 257 and 513 bins, one to three
// sources, 96 in all: 0.95 ms against 1.25 ms with column tiles spaced for the largest Ns and as
// many k-steps as 64 channels need.
#include "ssl_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kRows = 16 * kWaves;          // directions per workgroup
constexpr int kEs = SSL_MAX_M + 2;          // complex64 stride of a staged signal vector
constexpr int kChunk = kThreads;            // blocks whose descriptors are held in LDS at once

// Steering-table readers: one complex element per word, complex64 (FP32 tables) or a pair of
// 16-bit values (re at the lower address) for bf16 / fp16 tables, widened exactly to FP32.
struct TabF32 {
    typedef float2 W;
    static __device__ __forceinline__ float2 get(const W *p) { return gload(p); }
    static __device__ __forceinline__ void get2(const W *p, float2 &x, float2 &y)
    {
        const float4 v = gload(reinterpret_cast<const float4 *>(p));
        x = make_float2(v.x, v.y);
        y = make_float2(v.z, v.w);
    }
};
struct TabBF16 {
    typedef unsigned int W;
    static __device__ __forceinline__ float2 get(const W *p)
    {
        return wide(gload(p));
    }
    static __device__ __forceinline__ float2 wide(unsigned int w)
    {
        return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    }
    static __device__ __forceinline__ void get2(const W *p, float2 &x, float2 &y)
    {
        const uint2 v = gload(reinterpret_cast<const uint2 *>(p));
        x = wide(v.x);
        y = wide(v.y);
    }
};
struct TabF16 {
    typedef unsigned int W;
    static __device__ __forceinline__ float2 get(const W *p)
    {
        return wide(gload(p));
    }
    static __device__ __forceinline__ float2 wide(unsigned int w)
    {
        return make_float2((float)__builtin_bit_cast(_Float16, (unsigned short)(w & 0xffffu)),
                           (float)__builtin_bit_cast(_Float16, (unsigned short)(w >> 16)));
    }
    static __device__ __forceinline__ void get2(const W *p, float2 &x, float2 &y)
    {
        const uint2 v = gload(reinterpret_cast<const uint2 *>(p));
        x = wide(v.x);
        y = wide(v.y);
    }
};

// Orders a wave's LDS accesses: the hardware completes one wave's in issue order, so only the compiler
// has to be kept from moving them across.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 1/x for normal x > 0: hardware estimate and two Newton steps
__device__ __forceinline__ double rcp_refined(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// The blocks of a column tile: t1 with one signal vector, then t2 with two, then t3 with three.
struct Tile {
    int t1, t2, t3;
    __device__ __forceinline__ int blocks() const { return t1 + t2 + t3; }
    __device__ __forceinline__ int ns(int b) const { return b < t1 ? 1 : b < t1 + t2 ? 2 : 3; }
    __device__ __forceinline__ int column(int b) const      // first column of block b
    {
        return b < t1 ? b : b < t1 + t2 ? 2 * b - t1 : 3 * b - 2 * t1 - t2;
    }
    __device__ __forceinline__ int block(int j) const       // block of column j (>= blocks() beyond)
    {
        const int r = j - t1, q = r - 2 * t2;
        return r < 0 ? j : q < 0 ? t1 + (r >> 1) : t1 + t2 + q / 3;
    }
};

// A lane's elements of a table row: k-steps in pairs (2 p, 2 p + 1) over elements 8 p .. 8 p + 7; a
// remainder of up to 4 elements takes one k-step (element 8 p + l / 16).
template <class Tab, int KQ> struct Rows {
    const typename Tab::W *Hf;
    int D, M, P8, rem, kl;
    bool lone, pair;                                         // the last k-step is a single one; 16-byte loads
    __device__ __forceinline__ Rows(const typename Tab::W *Hf_, int D_, int M_, int kl_)
        : Hf(Hf_), D(D_), M(M_), P8(M_ >> 3), rem(M_ & 7), kl(kl_), lone((M_ & 7) != 0 && (M_ & 7) <= 4),
          pair((M_ & 1) == 0 && (reinterpret_cast<size_t>(Hf_) & (2 * sizeof(*Hf_) - 1)) == 0)
    {
    }
    __device__ __forceinline__ int slot(int m) const         // position of element m: 4 q + l / 16
    {
        const int p = m >> 3, w = m & 7;
        return lone && p == P8 ? m : 8 * p + ((w & 1) << 2) + (w >> 1);
    }
    __device__ __forceinline__ int element(int s) const      // its inverse
    {
        const int p = s >> 3, w = s & 7;
        return lone && p == P8 ? s : 8 * p + ((w & 3) << 1) + (w >> 2);
    }
    __device__ __forceinline__ void load(int row, float2 (&h)[KQ + (KQ & 1)]) const
    {
        const typename Tab::W *hrow = Hf + (size_t)(row < D ? row : 0) * M;
#pragma unroll
        for (int p = 0; p < (KQ + 1) / 2; ++p) {
            const int m = 8 * p + 2 * kl;
            float2 x = make_float2(0.f, 0.f), y = x;
            if (p < P8 || (p == P8 && rem > 4)) {            // uniform
                if (pair) {
                    if (m < M && row < D) Tab::get2(hrow + m, x, y);
                } else if (row < D) {
                    if (m < M) x = Tab::get(hrow + m);
                    if (m + 1 < M) y = Tab::get(hrow + m + 1);
                }
            } else if (p == P8 && lone) {
                if (8 * p + kl < M && row < D) x = Tab::get(hrow + 8 * p + kl);
            }
            h[2 * p] = x;
            h[2 * p + 1] = y;
        }
    }
};

// The next blocks, from block c of n on, that fill COLS columns: blocks [0, e1) have Ns = 1, [e1, e2)
// Ns = 2, the rest Ns = 3.
template <int COLS>
__device__ __forceinline__ Tile tile_from(int c, int e1, int e2, int n)
{
    Tile t;
    t.t1 = min(COLS, max(e1 - c, 0));
    t.t2 = c + t.t1 < e1 ? 0 : min((COLS - t.t1) / 2, max(e2 - c - t.t1, 0));
    t.t3 = c + t.t1 + t.t2 < e2 ? 0 : min((COLS - t.t1 - 2 * t.t2) / 3, max(n - c - t.t1 - t.t2, 0));
    return t;
}

// P of one (block, direction): g = E_s^H x (ns values), L = L^{-1}, lower triangular by rows (00, 10, 11,
// 20, 21, 22), xx = |x|^2: hh / (xx - |L g|^2), x = h or K^{-1/2} h
__device__ __forceinline__ float spectrum(const double2 *g, const double2 *L, int ns, double hh, double xx)
{
    const double2 g0 = g[0];
    const double2 y0 = make_double2(L[0].x * g0.x, L[0].x * g0.y);
    double q2 = y0.x * y0.x + y0.y * y0.y;
    if (ns >= 2) {
        const double2 g1 = g[1];
        const double2 y1 = make_double2(L[1].x * g0.x - L[1].y * g0.y + L[2].x * g1.x,
                                        L[1].x * g0.y + L[1].y * g0.x + L[2].x * g1.y);
        q2 += y1.x * y1.x + y1.y * y1.y;
        if (ns >= 3) {
            const double2 g2 = g[2];
            const double2 y2 = make_double2(
                L[3].x * g0.x - L[3].y * g0.y + L[4].x * g1.x - L[4].y * g1.y + L[5].x * g2.x,
                L[3].x * g0.y + L[3].y * g0.x + L[4].x * g1.y + L[4].y * g1.x + L[5].x * g2.y);
            q2 += y2.x * y2.x + y2.y * y2.y;
        }
    }
    const double den = fmax(xx - q2, 1.17549435e-38);
    return (float)(hh * rcp_refined(den));
}

// One workgroup: nd tiles of 64 directions of bin f from tile0 on, for nb blocks sharing the table Hf
// (the bin's [D][M] rows), in ascending order of Ns.  blk(i, Es, L, ns, ok, P) gives block i's signal
// vectors and L^{-1} of the bin, its Ns, whether the bin is valid, and its P row of the bin.  COLS:
// columns of a tile (16, or 4 for a single block); KQ: k-steps (at least those of M; the ones beyond
// hold zeros).  LOOP: nd tiles, else one.  Column tiles pass through two LDS stages; with LOOP, where two
// column tiles hold all blocks, they stay there for every direction tile, whose rows are loaded under
// the previous one's products, and the waves run without barriers.
template <class Tab, int COLS, int KQ, bool LOOP, class BlockAt>
__device__ __forceinline__ void sig_tile(const typename Tab::W *__restrict__ Hf, int D, int M,
                                         int tile0, int nd, int nb, BlockAt &&blk)
{
    constexpr int CHUNK = COLS < 16 ? 4 : kChunk;
    constexpr int GS = COLS + 1;                             // complex128 stride of a direction
    __shared__ float2 Es[2][COLS * kEs];                     // signal vectors, by tile parity
    __shared__ double2 Ls[2][COLS][6];
    __shared__ double2 Gs[kWaves][16 * GS];
    __shared__ float *Pp[CHUNK];                             // per block of the chunk
    __shared__ const float2 *Ep[CHUNK];
    __shared__ const double2 *Lp[CHUNK];
    __shared__ int Nsb[CHUNK];                               // Ns, 0 for a failed bin
    __shared__ double nrm_s[kRows];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kl = lane >> 4;
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    const Rows<Tab, KQ> rows(Hf, D, M, kl);
    // this lane's A operands: row (lane & 15) of the wave's 16 directions
    auto load_h = [&](int tile, float2 (&h)[KQ + (KQ & 1)]) {
        rows.load(tile * kRows + 16 * wave + (lane & 15), h);
    };

    // One column tile's operands into registers: a wave holds every kWaves-th column, one element per
    // lane (zero if absent); threads below COLS * 6 hold one L^{-1} entry.  Loaded
    // one tile ahead, so that the loads are in flight under the current tile's products and
    // epilogue; stored to the other parity's buffers.
    static_assert(SSL_MAX_M == 64, "a lane per element of a column");
    constexpr int kPer = COLS / kWaves;
    float2 ev[kPer];
    double2 lv;
    auto load_tile = [&](int c0, const Tile &t) {            // c0: first block, chunk-relative
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int j = uwave + kWaves * i, m = lane;
            const int bi = t.block(j), s = j - t.column(bi);
            ev[i] = (bi < t.blocks() && m < M && Nsb[c0 + bi] > 0)
                        ? gload(Ep[c0 + bi] + (size_t)s * M + m)
                        : make_float2(0.f, 0.f);
        }
        const int bi = tid / 6, k = tid - bi * 6;
        lv = (tid < COLS * 6 && bi < t.blocks() && Nsb[c0 + bi] > 0) ? gload(Lp[c0 + bi] + k)
                                                                     : make_double2(0.0, 0.0);
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int j = uwave + kWaves * i;
            Es[buf][j * kEs + rows.slot(lane)] = ev[i];
        }
        if (tid < COLS * 6) Ls[buf][tid / 6][tid % 6] = lv;
    };

    float2 ha[KQ + (KQ & 1)], hb[KQ + (KQ & 1)];
    load_h(tile0, hb);
    bool resident = false;                                   // both column tiles are in LDS
    int nc = 0, e1 = 0, e2 = 0;
    auto tile_at = [&](int c) { return tile_from<COLS>(c, e1, e2, nc); };
    for (int dt = 0; dt < nd; ++dt) {
        const int d0 = (tile0 + dt) * kRows;
#pragma unroll
        for (int q = 0; q < KQ; ++q) ha[q] = hb[q];
        if constexpr (LOOP)
            if (dt + 1 < nd) load_h(tile0 + dt + 1, hb);
        double hn = 0.0;
#pragma unroll
        for (int q = 0; q < KQ; ++q)
            hn = fma((double)ha[q].x, (double)ha[q].x, fma((double)ha[q].y, (double)ha[q].y, hn));
        hn += __shfl_xor(hn, 16);
        hn += __shfl_xor(hn, 32);
        if (lane < 16) nrm_s[16 * wave + lane] = hn;

        for (int h0 = 0; h0 < nb; h0 += CHUNK) {            // chunks of the blocks' descriptors
            Tile t = tile_at(0);
            if (!resident) {
                nc = min(CHUNK, nb - h0);
                __syncthreads();                             // the previous chunk is finished
                int myns = 4;
                if (tid < nc) {
                    const float2 *e;
                    const double2 *L;
                    float *P;
                    int ns = 0;
                    bool ok = false;
                    blk(h0 + tid, e, L, ns, ok, P);
                    myns = ns;
                    Nsb[tid] = ok ? ns : 0;
                    Pp[tid] = P;
                    Ep[tid] = e;
                    Lp[tid] = L;
                }
                e1 = __builtin_amdgcn_readfirstlane(__syncthreads_count(myns <= 1));
                e2 = __builtin_amdgcn_readfirstlane(__syncthreads_count(myns <= 2));
                t = tile_at(0);
                load_tile(0, t);
                store_tile(0);
                if (LOOP && nb == nc) {                      // uniform
                    const int c1 = t.blocks();
                    const Tile tn = tile_at(c1);
                    resident = c1 + tn.blocks() == nc;
                    if (resident && c1 < nc) {
                        load_tile(c1, tn);
                        store_tile(1);
                    }
                }
                __syncthreads();
            }
            int c0 = 0;
            for (int buf = 0; c0 < nc; buf ^= 1) {
                const int nt = t.blocks(), c1 = c0 + nt;
                Tile tn = t;
                if (c1 < nc) {
                    tn = tile_at(c1);
                    if (!resident) load_tile(c1, tn);
                }
                if constexpr (COLS == 16) {
                    doublex4 p1 = {0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
                    const float2 *ecol = Es[buf] + (lane & 15) * kEs + kl;
#pragma unroll
                    for (int q = 0; q < KQ; ++q) {
                        const float2 e = ecol[4 * q];
                        // used a few times: not held in FP64 (twice the registers)
                        if constexpr (LOOP) asm volatile("" : "+v"(ha[q].x), "+v"(ha[q].y));
                        const double a = ha[q].x, b = ha[q].y, c = e.x, d = e.y;
                        p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, c, p1, 0, 0, 0);
                        p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(b, -d, p2, 0, 0, 0);
                        p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(a + b, c - d, p3, 0, 0, 0);
                    }
                    const doublex4 gre = p1 - p2, gim = p3 - p1 - p2;
                    // FP64 result layout: element e of lane l is row l / 16 + 4 e, column l % 16
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        Gs[wave][(kl + 4 * e) * GS + (lane & 15)] = make_double2(gre[e], gim[e]);
                } else {
                    double p1 = 0.0, p2 = 0.0, p3 = 0.0;
                    const float2 *ecol = Es[buf] + (lane & 3) * kEs + kl;
#pragma unroll
                    for (int q = 0; q < KQ; ++q) {
                        const float2 e = ecol[4 * q];
                        const double a = ha[q].x, b = ha[q].y, c = e.x, d = e.y;
                        p1 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, c, p1, 0, 0, 0);
                        p2 = __builtin_amdgcn_mfma_f64_4x4x4f64(b, -d, p2, 0, 0, 0);
                        p3 = __builtin_amdgcn_mfma_f64_4x4x4f64(a + b, c - d, p3, 0, 0, 0);
                    }
                    // lane l: row 4 (l / 4 mod 4) + l / 16, column l % 4
                    Gs[wave][(4 * ((lane >> 2) & 3) + kl) * GS + (lane & 3)] =
                        make_double2(p1 - p2, p3 - p1 - p2);
                }
                wave_lds_sync();                             // Gs and nrm_s are this wave's own
                // items (block bi, direction row i of this wave): den = |h|^2 - |L^{-1} g|^2
                for (int it = lane; it < 16 * nt; it += 64) {
                    const int bi = it >> 4, i = it & 15;
                    const int d = d0 + 16 * wave + i;
                    float *P = Pp[c0 + bi];
                    if (d >= D || P == nullptr) continue;
                    const double hh = nrm_s[16 * wave + i];
                    float out = 0.0f;
                    if (Nsb[c0 + bi] > 0)
                        out = spectrum(&Gs[wave][i * GS + t.column(bi)], Ls[buf][bi], t.ns(bi), hh, hh);
                    gstore(P + d, out);
                }
                wave_lds_sync();
                // the other parity was last read in the previous tile, before its barrier
                if (!resident) {
                    if (c1 < nc) store_tile(buf ^ 1);
                    __syncthreads();
                }
                c0 = c1;
                t = tn;
            }
        }
    }
}

// GEVD-MUSIC: the noise vectors are W y, W = K^{-1/2} and y the noise eigenvectors of C = W R W, so that
//   den = sum |h^H W y|^2 = |W h|^2 - |L^{-1} E_s^H W h|^2,
// E_s the signal vectors of C: the same form on u = W h.  One workgroup: nd tiles of 64 directions of bin f
// from tile0 on, for nb blocks sharing the table Hf and the noise set Wf (both of the bin), in ascending
// order of Ns.  W waits in LDS; a wave forms u for its 16 directions, u = W H^T with the directions as
// columns, whose FP64 result layout (element e of lane l: row l / 16 + 4 e, column l % 16) is the B operand
// of E_s^H u as it stands: u never leaves the registers, and serves every block.  A wave's tile costs 180
// MFMAs for u at 60 channels, 45 per 16 signal vectors, and 45 of the short ones for up to 4.
//   Measured (60 channels, 257 bins, 1368 directions): 8 blocks of one noise set 0.28 ms, where the FP32
// noise-vector form took 0.80 ms and 0.10 ms to form its vectors W y.  The matrix cores are busy half of
// that time: two waves per SIMD (W fills the LDS) leave the latency of a workgroup's start and of each tile's
// stores partly uncovered.
template <class Tab, int NT, int KQ, class BlockAt>
__device__ __forceinline__ void gevd_tile(const double2 *__restrict__ Wf,
                                          const typename Tab::W *__restrict__ Hf, int D, int M,
                                          int tile0, int nd, int nb, BlockAt &&blk)
{
    constexpr int MP = 16 * NT, WS = 4 * KQ + 1, GS = 17;
    __shared__ double2 Ws[MP * WS];                          // row m, element position s
    __shared__ double2 Gs[kWaves][16 * GS];
    __shared__ double2 Ls[16 * 6];                           // of the column tile's blocks: L^{-1},
    __shared__ float *Pp[16];                                // P row,
    __shared__ int Ds[16];                                   // first column + 256 Ns (0: failed bin)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kl = lane >> 4, cl = lane & 15;
    const Rows<Tab, KQ> rows(Hf, D, M, kl);
    float2 h[KQ + (KQ & 1)], ev[KQ];
    rows.load(tile0 * kRows + 16 * wave + cl, h);
    constexpr int kW = MP * 4 * KQ / kThreads;               // whole: MP is a multiple of 16, 4 * 16 = 64
    double2 wv[kW];                                          // all in flight at once
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        const int x = tid + kThreads * i, r = x / (4 * KQ), m = rows.element(x - r * (4 * KQ));
        wv[i] = r < M && m < M ? gload(Wf + (size_t)r * M + m) : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        const int x = tid + kThreads * i, r = x / (4 * KQ);
        Ws[r * WS + x - r * (4 * KQ)] = wv[i];
    }
    const float2 *E;
    const double2 *L;
    float *P;
    int ns;
    bool ok;
    int e1 = 0, e2 = 0;                                      // blocks with Ns <= 1, <= 2
    for (int b = 0; b < nb; b += 64) {
        int n = 4;
        if (b + lane < nb) blk(b + lane, E, L, n, ok, P);
        e1 += __popcll(__ballot(n <= 1));
        e2 += __popcll(__ballot(n <= 2));
    }
    auto small = [](const Tile &t) { return t.t1 + 2 * t.t2 + 3 * t.t3 <= 4; };
    auto load_e = [&](int c0, const Tile &t) {               // operands: column l % 16 (l % 4) of the tile
        const int j = small(t) ? cl & 3 : cl;
        const int bi = t.block(j);
        const bool in = bi < t.blocks();
        if (in) blk(c0 + bi, E, L, ns, ok, P);
        const float2 *col = in && ok ? E + (size_t)(j - t.column(bi)) * M : nullptr;
#pragma unroll
        for (int q = 0; q < KQ; ++q)
            ev[q] = col != nullptr && 4 * q + kl < M ? gload(col + 4 * q + kl) : make_float2(0.f, 0.f);
    };
    auto stage = [&](int c0, const Tile &t) {
        const int bi = tid / 6, k = tid - 6 * bi;
        if (bi < t.blocks()) {                               // at most 16
            blk(c0 + bi, E, L, ns, ok, P);
            Ls[tid] = ok ? gload(L + k) : make_double2(0.0, 0.0);
            if (k == 0) {
                Pp[bi] = P;
                Ds[bi] = ok ? t.column(bi) + 256 * ns : 0;
            }
        }
    };
    Tile t = tile_from<16>(0, e1, e2, nb);
    const bool single = t.blocks() == nb;                    // one column tile: staged once
    load_e(0, t);
    if (single) stage(0, t);
    __syncthreads();
    for (int dt = 0; dt < nd; ++dt) {
        const int d = (tile0 + dt) * kRows + 16 * wave + cl; // this lane's direction
        double hh = 0.0;
#pragma unroll
        for (int q = 0; q < KQ; ++q)
            hh = fma((double)h[q].x, (double)h[q].x, fma((double)h[q].y, (double)h[q].y, hh));
        hh += __shfl_xor(hh, 16);
        hh += __shfl_xor(hh, 32);
        doublex4 ur[NT], ui[NT];
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) {
            doublex4 p1 = {0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
            const double2 *wr = Ws + (16 * rt + cl) * WS + kl;
#pragma unroll
            for (int q = 0; q < KQ; ++q) {
                const double2 w = wr[4 * q];
                asm volatile("" : "+v"(h[q].x), "+v"(h[q].y));      // not held in FP64
                const double a = h[q].x, b = h[q].y;
                p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, a, p1, 0, 0, 0);
                p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, b, p2, 0, 0, 0);
                p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x + w.y, a + b, p3, 0, 0, 0);
            }
            ur[rt] = p1 - p2;
            ui[rt] = p3 - p1 - p2;
        }
        if (dt + 1 < nd) rows.load(d + kRows, h);
        double uu = 0.0;
#pragma unroll
        for (int rt = 0; rt < NT; ++rt)
#pragma unroll
            for (int e = 0; e < 4; ++e) uu = fma(ur[rt][e], ur[rt][e], fma(ui[rt][e], ui[rt][e], uu));
        uu += __shfl_xor(uu, 16);
        uu += __shfl_xor(uu, 32);
        for (int c0 = 0; c0 < nb;) {
            const int nt = t.blocks(), c1 = c0 + nt;
            if (small(t)) {                                  // uniform: 22 cycles a product instead of 64
                double p1 = 0.0, p2 = 0.0, p3 = 0.0;
#pragma unroll
                for (int q = 0; q < KQ; ++q) {
                    asm volatile("" : "+v"(ev[q].x), "+v"(ev[q].y));
                    const double c = ev[q].x, s = ev[q].y, a = ur[q >> 2][q & 3], b = ui[q >> 2][q & 3];
                    p1 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, c, p1, 0, 0, 0);
                    p2 = __builtin_amdgcn_mfma_f64_4x4x4f64(b, s, p2, 0, 0, 0);
                    p3 = __builtin_amdgcn_mfma_f64_4x4x4f64(a + b, c - s, p3, 0, 0, 0);
                }
                // lane l: direction 4 (l / 4 mod 4) + l / 16, column l % 4
                Gs[wave][(4 * ((lane >> 2) & 3) + kl) * GS + (lane & 3)] = make_double2(p1 + p2, p3 - p1 + p2);
            } else {
                doublex4 p1 = {0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
#pragma unroll
                for (int q = 0; q < KQ; ++q) {
                    asm volatile("" : "+v"(ev[q].x), "+v"(ev[q].y));
                    const double c = ev[q].x, s = ev[q].y, a = ur[q >> 2][q & 3], b = ui[q >> 2][q & 3];
                    p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(c, a, p1, 0, 0, 0);
                    p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(s, b, p2, 0, 0, 0);
                    p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(c - s, a + b, p3, 0, 0, 0);
                }
                const doublex4 gr = p1 + p2, gi = p3 - p1 + p2;
#pragma unroll
                for (int e = 0; e < 4; ++e) Gs[wave][cl * GS + kl + 4 * e] = make_double2(gr[e], gi[e]);
            }
            if (!single) {                                   // uniform
                __syncthreads();                             // the last tile's items are done
                stage(c0, t);
                __syncthreads();
                t = tile_from<16>(c1 < nb ? c1 : 0, e1, e2, nb);
                if (c1 < nb || dt + 1 < nd) load_e(c1 < nb ? c1 : 0, t);
            }
            wave_lds_sync();
            for (int it = lane; it < 16 * nt; it += 64) {    // (block, this lane's direction)
                const int bi = it >> 4, ds = Ds[bi];
                if (d < D && Pp[bi] != nullptr)
                    gstore(Pp[bi] + d, ds ? spectrum(&Gs[wave][cl * GS + (ds & 255)], Ls + 6 * bi, ds >> 8,
                                                     hh, uu)
                                          : 0.0f);
            }
            wave_lds_sync();
            c0 = c1;
        }
    }
}

// Workgroup -> (item, direction tile), dealt XCD by XCD as in the noise-vector projection.
constexpr int kXcds = 8;
__host__ __device__ inline int sig_grid(int n_items, int n_tiles)
{
    return kXcds * ((n_items + kXcds - 1) / kXcds) * n_tiles;
}
__device__ __forceinline__ bool sig_item(int n_items, int n_tiles, int &item, int &tile)
{
    const int w = blockIdx.x;
    const int slot = w / kXcds;
    item = (slot / n_tiles) * kXcds + w % kXcds;
    tile = slot % n_tiles;
    return item < n_items;
}

template <class Tab, int KQ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void steer_sig_single(
    const typename Tab::W *__restrict__ H, const float2 *__restrict__ Es,
    const double2 *__restrict__ Esl,
    const int32_t *__restrict__ bin_status, int F, int D, int M, int Ns, float *__restrict__ P,
    int n_tiles)
{
    int f, tile;
    if (!sig_item(F, n_tiles, f, tile)) return;
    sig_tile<Tab, 4, KQ, false>(H + (size_t)f * D * M, D, M, tile, 1, 1,
             [&](int, const float2 *&e, const double2 *&L, int &ns, bool &ok, float *&Pf) {
                 e = Es + (size_t)f * Ns * M;
                 L = Esl + 6 * (size_t)f;
                 ns = Ns;
                 ok = bin_status == nullptr || bin_status[f] == SSL_BIN_OK;
                 Pf = P + (size_t)f * D;
             });
}

// Batched: item = (group, bin), groups[g] = (first, count) into gblocks, the blocks of one
// steering table in ascending order of Ns.
// (3 waves per SIMD: the next tile's operands in registers would otherwise cost one)
template <class Tab, int KQ, bool LOOP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(3))) void steer_sig_batch(
    const BlockDev *__restrict__ blk, const int2 *__restrict__ items, int n_items, int n_tiles,
    const int2 *__restrict__ groups, const int *__restrict__ gblocks, int per_wg)
{
    int ii, tile;
    if (!sig_item(n_items, n_tiles, ii, tile)) return;
    const int2 it = items[ii];
    const int2 gr = groups[it.x];
    const BlockDev &B0 = blk[gblocks[gr.x]];
    const int f = it.y, M = B0.M, D = B0.D;
    const int t0 = tile * per_wg, nd = min(per_wg, (D + kRows - 1) / kRows - t0);
    if (nd <= 0) return;
    sig_tile<Tab, 16, KQ, LOOP>(static_cast<const typename Tab::W *>(B0.H) + (size_t)f * D * M, D, M, t0, nd, gr.y,
             [&](int i, const float2 *&e, const double2 *&L, int &ns, bool &ok, float *&Pf) {
                 const BlockDev &B = blk[gblocks[gr.x + i]];
                 e = B.Es + (size_t)f * B.Ns * M;
                 L = B.Esl + 6 * (size_t)f;
                 ns = B.Ns;
                 ok = gload(B.status + f) == SSL_BIN_OK;
                 Pf = B.P + (size_t)f * D;
             });
}

template <class Tab, int NT, int KQ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void steer_gevd_single(
    const double2 *__restrict__ W, const typename Tab::W *__restrict__ H, const float2 *__restrict__ Es,
    const double2 *__restrict__ Esl, const int32_t *__restrict__ bin_status, int F, int D, int M, int Ns,
    float *__restrict__ P, int n_tiles, int per_wg)
{
    int f, tile;
    if (!sig_item(F, n_tiles, f, tile)) return;
    const int t0 = tile * per_wg, nd = min(per_wg, (D + kRows - 1) / kRows - t0);
    if (nd <= 0) return;
    gevd_tile<Tab, NT, KQ>(W + (size_t)f * M * M, H + (size_t)f * D * M, D, M, t0, nd, 1,
             [&](int, const float2 *&e, const double2 *&L, int &ns, bool &ok, float *&Pf) {
                 e = Es + (size_t)f * Ns * M;
                 L = Esl + 6 * (size_t)f;
                 ns = Ns;
                 ok = bin_status[f] == SSL_BIN_OK;
                 Pf = P + (size_t)f * D;
             });
}

// Batched: items and groups as above, the blocks of a group sharing the noise set as well.
template <class Tab, int NT, int KQ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void steer_gevd_batch(
    const BlockDev *__restrict__ blk, const int2 *__restrict__ items, int n_items, int n_tiles,
    const int2 *__restrict__ groups, const int *__restrict__ gblocks, int per_wg)
{
    int ii, tile;
    if (!sig_item(n_items, n_tiles, ii, tile)) return;
    const int2 it = items[ii];
    const int2 gr = groups[it.x];
    const BlockDev &B0 = blk[gblocks[gr.x]];
    const int f = it.y, M = B0.M, D = B0.D;
    const int t0 = tile * per_wg, nd = min(per_wg, (D + kRows - 1) / kRows - t0);
    if (nd <= 0) return;
    gevd_tile<Tab, NT, KQ>(B0.Kisq + (size_t)f * M * M,
                           static_cast<const typename Tab::W *>(B0.H) + (size_t)f * D * M, D, M, t0, nd, gr.y,
             [&](int i, const float2 *&e, const double2 *&L, int &ns, bool &ok, float *&Pf) {
                 const BlockDev &B = blk[gblocks[gr.x + i]];
                 e = B.Es + (size_t)f * B.Ns * M;
                 L = B.Esl + 6 * (size_t)f;
                 ns = B.Ns;
                 ok = gload(B.status + f) == SSL_BIN_OK;
                 Pf = B.P + (size_t)f * D;
             });
}

// Calls fn with the table reader of prec and kq.
template <class KQ, class Fn>
hipError_t with_table(ssl_prec prec, KQ kq, Fn &&fn)
{
    if (prec == SSL_BF16) return fn(TabBF16(), kq);
    if (prec == SSL_FP16) return fn(TabF16(), kq);
    return fn(TabF32(), kq);
}
// Calls fn with the table reader of prec and the k-steps of a class.
template <class Fn>
hipError_t with_variant(ssl_prec prec, int cls, Fn &&fn)
{
    auto table = [&](auto kq) { return with_table(prec, kq, fn); };
    switch (cls) {
    case 16: return table(std::integral_constant<int, 4>());
    case 32: return table(std::integral_constant<int, 8>());
    case 48: return table(std::integral_constant<int, 12>());
    case 60: return table(std::integral_constant<int, 15>());
    default: return table(std::integral_constant<int, 16>());
    }
}

// The same for the classes that take the GEVD form (use_sig, abi.hip).
template <class Fn>
hipError_t with_gevd_variant(ssl_prec prec, int cls, Fn &&fn)
{
    switch (cls) {
    case 32: return with_table(prec, std::integral_constant<int, 8>(), fn);
    case 48: return with_table(prec, std::integral_constant<int, 12>(), fn);
    case 60: return with_table(prec, std::integral_constant<int, 15>(), fn);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Direction tiles of a workgroup, 0 for the kernel without the direction loop.  Where a table's blocks
// fill two column tiles (32 signal vectors) or fewer on average, a workgroup's setup (a chain of
// descriptor loads, then the signal vectors) costs more than one direction tile, so it is paid once for
// several: as few as leave 8 workgroups per CU (two or three launch rounds), eight at most.  Measured
// with 0 / 1 / 2 / 4 / 8 tiles: 8 and 16 channels, 257 bins, 11 blocks 87 / 91 / 72 / 66 / 62 us; 60
// channels, 5 blocks 100 / 105 / 99 / 108 / 120 us (too few workgroups from 3 tiles on).  With more
// blocks the setup is hidden and the rows of one direction tile are kept in FP64 instead (128 blocks:
// 0.78 ms without the loop, 0.86 ms with it).
int steer_sig_per_wg(int64_t n_items, int n_tiles, double columns, int cus)
{
    if (columns > 32.0) return 0;
    return (int)std::max<int64_t>(1, std::min<int64_t>(8, n_items * n_tiles / (8 * (int64_t)cus)));
}

int steer_sig_tiles(int D) { return (D + kRows - 1) / kRows; }

hipError_t launch_steer_sig(const void *H, ssl_prec hprec, const ssl_c64 *Es,
                            const ssl_c128 *Esl, int F, int D, int M, int Ns,
                            const int32_t *bin_status, float *P, hipStream_t st)
{
    const int nt = steer_sig_tiles(D);
    return with_variant(hprec, steer_sig_class(M), [&](auto tab, auto kq) {
        typedef decltype(tab) Tab;
        hipLaunchKernelGGL((steer_sig_single<Tab, kq>), dim3(sig_grid(F, nt)), dim3(kThreads), 0,
                           st, static_cast<const typename Tab::W *>(H),
                           reinterpret_cast<const float2 *>(Es),
                           reinterpret_cast<const double2 *>(Esl), bin_status, F, D, M, Ns, P, nt);
        return hipGetLastError();
    });
}

hipError_t launch_steer_sig_batch(const BlockDev *blk, const int2 *items, int n_items,
                                  const int2 *groups, const int *gblocks, int cls, int max_dtiles,
                                  int per_wg, ssl_prec hprec, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    const int per = per_wg > 0 ? per_wg : 1, nt = (max_dtiles + per - 1) / per;
    return with_variant(hprec, cls, [&](auto tab, auto kq) {
        typedef decltype(tab) Tab;
        const dim3 grid(sig_grid(n_items, nt)), block(kThreads);
        if (per_wg > 0)
            hipLaunchKernelGGL((steer_sig_batch<Tab, kq, true>), grid, block, 0, st, blk, items,
                               n_items, nt, groups, gblocks, per);
        else
            hipLaunchKernelGGL((steer_sig_batch<Tab, kq, false>), grid, block, 0, st, blk, items,
                               n_items, nt, groups, gblocks, per);
        return hipGetLastError();
    });
}

// Direction tiles of a workgroup: W (58 KB at 60 channels) is staged once for them, and 8 workgroups per CU
// are left where there are that many; at most 8 tiles.  8 blocks with noise sets of their own, at most 2 / 4
// / 8 / 12 tiles: 60 channels 1883 / 1955 / 1781 / 1922 us, 32 channels 679 / 659 / 599 / 634 us.
int steer_gevd_per_wg(int64_t n_items, int n_tiles, int cus)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(8, n_items * n_tiles / (8 * (int64_t)cus)));
}

hipError_t launch_steer_gevd(const ssl_c128 *W, const void *H, ssl_prec hprec, const ssl_c64 *Es,
                             const ssl_c128 *Esl, int F, int D, int M, int Ns, const int32_t *bin_status,
                             float *P, int per_wg, hipStream_t st)
{
    const int nt = (steer_sig_tiles(D) + per_wg - 1) / per_wg;
    return with_gevd_variant(hprec, steer_sig_class(M), [&](auto tab, auto kq) {
        typedef decltype(tab) Tab;
        hipLaunchKernelGGL((steer_gevd_single<Tab, (kq + 3) / 4, kq>), dim3(sig_grid(F, nt)), dim3(kThreads),
                           0, st, reinterpret_cast<const double2 *>(W),
                           static_cast<const typename Tab::W *>(H), reinterpret_cast<const float2 *>(Es),
                           reinterpret_cast<const double2 *>(Esl), bin_status, F, D, M, Ns, P, nt, per_wg);
        return hipGetLastError();
    });
}

hipError_t launch_steer_gevd_batch(const BlockDev *blk, const int2 *items, int n_items,
                                   const int2 *groups, const int *gblocks, int cls, int max_dtiles,
                                   int per_wg, ssl_prec hprec, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    const int nt = (max_dtiles + per_wg - 1) / per_wg;
    return with_gevd_variant(hprec, cls, [&](auto tab, auto kq) {
        typedef decltype(tab) Tab;
        hipLaunchKernelGGL((steer_gevd_batch<Tab, (kq + 3) / 4, kq>), dim3(sig_grid(n_items, nt)),
                           dim3(kThreads), 0, st, blk, items, n_items, nt, groups, gblocks, per_wg);
        return hipGetLastError();
    });
}
