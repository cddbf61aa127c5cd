// The Gram factor of a bin's signal vectors, shared by the solvers that produce them.
#pragma once

#include "ssl_internal.h"

// Lf[0..5] = the inverse L^{-1} of the Cholesky factor of the Gram matrix Gamma = E_s^H E_s of Ns <= 3
// signal vectors, lower triangle by rows (00, 10, 11, 20, 21, 22); zero if !ok or if Gamma is not
// positive definite.  gr, gi: Gamma_st = e_s^H e_t, s <= t, at index t (t + 1) / 2 + s.  One lane.
__device__ __forceinline__ void write_inverse_factor(const double (&gr)[6], const double (&gi)[6],
                                                     bool ok, int Ns, double2 *__restrict__ Lf)
{
    double2 out[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) out[i] = make_double2(0.0, 0.0);
    // Gamma = L L^H: L_t0 = conj(Gamma_0t) / L00, ... (lower rows t, columns s)
    const double l00 = sqrt(gr[0]);
    bool pd = ok && gr[0] > 0.0;
    double2 l10 = make_double2(0.0, 0.0), l20 = l10, l21 = l10;
    double l11 = 1.0, l22 = 1.0;
    if (Ns >= 2 && pd) {
        l10 = make_double2(gr[1] / l00, -gi[1] / l00);
        const double d = gr[2] - (l10.x * l10.x + l10.y * l10.y);
        pd = d > 0.0;
        l11 = sqrt(fmax(d, 0.0));
    }
    if (Ns >= 3 && pd) {
        l20 = make_double2(gr[3] / l00, -gi[3] / l00);
        // Gamma_21 = conj(Gamma_12) minus L20 conj(L10), over L11
        const double2 g21 = make_double2(gr[4], -gi[4]);
        const double2 t21 = make_double2(g21.x - (l20.x * l10.x + l20.y * l10.y),
                                         g21.y - (l20.y * l10.x - l20.x * l10.y));
        l21 = make_double2(t21.x / l11, t21.y / l11);
        const double d = gr[5] - (l20.x * l20.x + l20.y * l20.y) -
                         (l21.x * l21.x + l21.y * l21.y);
        pd = d > 0.0;
        l22 = sqrt(fmax(d, 0.0));
    }
    if (pd) {
        const double i00 = 1.0 / l00, i11 = 1.0 / l11, i22 = 1.0 / l22;
        // inverse of the lower triangular L, column by column
        const double2 i10 = make_double2(-l10.x * i00 * i11, -l10.y * i00 * i11);
        const double2 i21 = make_double2(-l21.x * i11 * i22, -l21.y * i11 * i22);
        const double2 s20 = make_double2(l20.x * i00 + (l21.x * i10.x - l21.y * i10.y),
                                         l20.y * i00 + (l21.x * i10.y + l21.y * i10.x));
        const double2 i20 = make_double2(-s20.x * i22, -s20.y * i22);
        out[0] = make_double2(i00, 0.0);
        out[1] = i10;
        out[2] = make_double2(i11, 0.0);
        out[3] = i20;
        out[4] = i21;
        out[5] = make_double2(i22, 0.0);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) Lf[i] = out[i];
}

// The same from the vectors themselves: the FP64 Gram matrix of the stored complex64 values, by the
// 64 lanes r of one wave; vec(k, r) gives element r (< M) of vector k.
template <class Vec>
__device__ __forceinline__ void write_signal_factor(Vec &&vec, bool ok, int Ns, int M, int r,
                                                    double2 *__restrict__ Lf)
{
    double2 e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float2 v = (ok && k < Ns && r < M) ? vec(k, r) : make_float2(0.f, 0.f);
        e[k] = make_double2(v.x, v.y);
    }
    double gr[6], gi[6];                       // Gamma_st = e_s^H e_t, index t (t + 1) / 2 + s
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int s2 = 0; s2 <= t; ++s2) {
            const int i = t * (t + 1) / 2 + s2;
            gr[i] = gi[i] = 0.0;
            if (t >= Ns) continue;             // uniform: absent vectors
            double a = fma(e[s2].x, e[t].x, e[s2].y * e[t].y);
            double b = fma(e[s2].x, e[t].y, -e[s2].y * e[t].x);
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                a += __shfl_xor(a, o);
                b += __shfl_xor(b, o);
            }
            gr[i] = a;
            gi[i] = b;
        }
    if (r == 0) write_inverse_factor(gr, gi, ok, Ns, Lf);
}
