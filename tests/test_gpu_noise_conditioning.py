"""K^{-1} of badly conditioned noise sets: one to three directional noises or a diffuse (sinc-coherent)
one over a white floor, cond(K) up to 1e11, at the edges of the inverse's pivot blocks of 16, set from K and
updated from frames.  R holds K's own noise beside a source, as in use, so that K^{-1} R cancels its large
directions.  MI355X only.

Bar: sigma of A = K^{-1} R against an inverse in 80-bit arithmetic.  Scalar Gauss-Jordan in FP64 has
|K^{-1} K - I| = e, about 2^-53 cond(K), computed here for every K by that elimination in numpy; a backward
stable elimination in another order of operations is given 8 max(e, M 2^-53 cond(K)), which moves sigma by
that times |A| at most, besides the SVD's own 8 M 2^-24 |A|_F."""
import numpy as np
import pytest

from gpu_util import S, ctx, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
U64 = 2.0 ** -53


def eliminate(K, dtype):
    """K^{-1} by in-place Gauss-Jordan elimination, scalar pivots, in the given complex type."""
    W = K.astype(dtype)
    for k in range(len(W)):
        ip = 1 / W[k, k].real
        r, c = W[k] * ip, W[:, k].copy()
        W = W - np.outer(c, r)
        W[k], W[:, k] = r, -c * ip
        W[k, k] = ip
    return W


def noise_set(rng, M, kind, c):
    if kind == "diffuse":
        x = rng.uniform(0, 1, (M, 3))
        return np.eye(M) + c / M * np.sinc(0.5 * np.linalg.norm(x[:, None] - x[None], axis=2)).astype(complex)
    d = np.exp(2j * np.pi * rng.uniform(size=(M, int(kind[0]))))
    return np.eye(M) + c / M * (d @ d.conj().T)


def check(S, ctx, n, K, R):  # noqa: F811
    import torch
    F, M, _ = K.shape
    sg = torch.zeros((F, M), dtype=torch.float32, device="cuda:0")
    st = torch.full((F,), -7, dtype=torch.int32, device="cuda:0")
    S.ssl_gsvd(ctx, to_dev(R), n, 1, torch.zeros((F, M - 1, M), dtype=torch.complex64, device="cuda:0"), sg, st)
    sg, st = to_host(sg), to_host(st)
    assert np.all(st == 0), st
    for f in range(F):
        W = eliminate(K[f], np.clongdouble)
        A = (W @ R[f].astype(np.clongdouble)).astype(complex)
        ref = np.linalg.svd(A, compute_uv=False)
        cond = np.linalg.cond(K[f])
        e = np.linalg.norm((eliminate(K[f], complex) @ K[f].astype(np.clongdouble) - np.eye(M)).astype(complex), 2)
        bar = 8 * max(e, M * U64 * cond) * ref[0] + 8 * M * 2.0 ** -24 * np.linalg.norm(A)
        err = np.max(np.abs(sg[f] - ref))
        print(f"  bin {f} cond {cond:.1e}: |sigma - ref| {err:.2e} (bar {bar:.2e}, |A| {ref[0]:.1f})", flush=True)
        assert err <= bar, (f, err, bar)


@pytest.mark.parametrize("kind", ["1 noise", "2 noises", "3 noises", "diffuse"])
@pytest.mark.parametrize("M", [17, 24, 33, 60, 64])
def test_inverse_of_a_set(S, ctx, M, kind):  # noqa: F811
    rng = np.random.default_rng(100 * M + len(kind))
    K = np.stack([noise_set(rng, M, kind, c) for c in (1e8, 1e9, 1e10, 1e11)])
    s = np.exp(2j * np.pi * rng.uniform(size=(4, M, 1)))
    R = (K + 10 * (s @ s.conj().transpose(0, 2, 1))).astype(np.complex64)
    n = S.ssl_noise_create(ctx, 4, M)
    S.ssl_noise_set(n, to_dev(K), S.SSL_FP64)
    check(S, ctx, n, K, R)
    S.ssl_noise_destroy(n)


@pytest.mark.parametrize("M", [24, 60])
def test_inverse_of_a_batched_update(S, ctx, M):  # noqa: F811
    """K <- (K + K^) / 2, K^ from frames of two strong noises, two handles in one call."""
    import torch
    rng = np.random.default_rng(M)
    F, T = 2, 2 * M
    ns, fr = [], []
    for _ in range(2):
        n = S.ssl_noise_create(ctx, F, M)
        S.ssl_noise_set(n, to_dev(np.tile(np.eye(M, dtype=complex), (F, 1, 1))), S.SSL_FP64)
        d = np.exp(2j * np.pi * rng.uniform(size=(F, 2, M)))
        X = 3e4 * (rng.standard_normal((F, T, 2)) @ d) + rng.standard_normal((F, T, M))
        ns.append(n)
        fr.append(to_dev(X.astype(np.complex64)))
    S.ssl_noise_update_frames(ctx, ns, fr, 0.5)
    for n in ns:
        Kd = torch.zeros((F, M, M), dtype=torch.complex128, device="cuda:0")
        S.ssl_noise_get(n, Kd)
        K = to_host(Kd)
        s = np.exp(2j * np.pi * rng.uniform(size=(F, M, 1)))
        check(S, ctx, n, K, (K + 10 * (s @ s.conj().transpose(0, 2, 1))).astype(np.complex64))
        S.ssl_noise_destroy(n)
