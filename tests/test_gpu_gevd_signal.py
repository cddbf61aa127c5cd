"""GEVD-MUSIC through the signal subspace (|W h|^2 - |L^{-1} E_s^H W h|^2, W = K^{-1/2}) at the sizes that
take it and beside those that do not: rows of a tile exactly filled and not, one and several column
tiles, all table precisions, blocks sharing a noise set or not, ill-conditioned noise, failed bins.
Against the FP64 oracle (P-bar within 1e-4, the FP32 path's bar) and a batch against each block alone,
bit for bit.  MI355X only."""
import numpy as np
import pytest

import oracle
from conftest import crandn
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2504_03373_amd as S
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    S.lib()
    return S


@pytest.fixture()
def ctx(S):
    c = S.ssl_ctx_create(0, 0)
    S.ssl_ctx_set_subspace(c, S.SSL_SUBSPACE_GEVD)
    yield c
    S.ssl_ctx_destroy(c)


def handle(S, ctx, K):
    n = S.ssl_noise_create(ctx, K.shape[0], K.shape[1])
    S.ssl_noise_set(n, to_dev(np.ascontiguousarray(K)), S.SSL_FP64)
    S.ssl_noise_enable_gevd(n)
    return n


def outs(F, D, Ns):
    import torch
    return (torch.full((Ns,), -7, dtype=torch.int32, device="cuda:0"),
            torch.zeros(Ns, device="cuda:0"), torch.zeros(D, device="cuda:0"),
            torch.full((F,), -7, dtype=torch.int32, device="cuda:0"))


def noise(rng, F, M, cond):
    """Hermitian positive definite K with eigenvalues spread evenly (in log) over cond."""
    K = np.empty((F, M, M), np.complex128)
    for f in range(F):
        U = np.linalg.qr(crandn(rng, M, M))[0]
        K[f] = (U * np.logspace(0, -np.log10(cond), M)) @ U.conj().T
        K[f] = 0.5 * (K[f] + K[f].conj().T)
    return K


@pytest.mark.parametrize("M,Nss,own,cond,prec", [
    (30, [2, 3, 2], False, 10.0, "fp32"),          # the first size of two tiles that takes the form
    (29, [2, 3, 2], False, 10.0, "fp32"),          # the last that does not
    (32, [2, 2, 2, 2, 1, 4], True, 1e3, "fp32"),   # full tiles; Ns = 1 and 4 keep the noise form
    (45, [3] * 6, False, 10.0, "bf16"),            # 18 columns: two column tiles
    (47, [2, 3], True, 10.0, "fp16"),
    (48, [2] * 9, False, 1e6, "fp32"),             # 18 columns, mixed order kept
    (60, [2, 3] * 8, False, 1e3, "fp32"),          # 40 columns
    (60, [2, 2], True, 1e4, "fp32"),
    (61, [2, 2], False, 10.0, "fp32"),             # beyond: noise form
])
def test_sizes(S, ctx, M, Nss, own, cond, prec):
    import torch
    F, D, T = 20, 150, 50
    p = {"fp32": S.SSL_FP32, "bf16": S.SSL_BF16, "fp16": S.SSL_FP16}[prec]
    rng = np.random.default_rng(M * 7 + len(Nss))
    H = np.exp(2j * np.pi * rng.random((F, D, M))).astype(np.complex64)
    Ks = [noise(rng, F, M, cond) for _ in range(len(Nss) if own else 1)]
    ns_h = [handle(S, ctx, K) for K in Ks]
    Xs = []
    for b in range(len(Nss)):
        C = np.linalg.cholesky(Ks[b % len(Ks)])
        X = np.einsum("fij,ftj->fti", C, crandn(rng, F, T, M))
        for k, d in enumerate(rng.choice(D, Nss[b], replace=False)):
            X += (4.0 - k / 2) * crandn(rng, F, T)[:, :, None] * H[:, None, d]
        X = X.astype(np.complex64)
        Xs.append(X if prec == "fp32" else (X / np.abs(X.view(np.float32)).max()).astype(np.complex64))
    Hd = to_dev(H)
    if prec != "fp32":
        Hd = torch.view_as_real(Hd).to(torch.bfloat16 if prec == "bf16" else torch.float16)
        Hd = Hd.reshape(F, D, 2 * M).contiguous()
    Xd = [to_dev(X) for X in Xs]
    alone = []
    for b, Ns in enumerate(Nss):
        o = outs(F, D, Ns)
        S.ssl_localize(ctx, Xd[b], ns_h[b % len(Ks)], Hd, p, D, 1, Ns, 2, *o)
        alone.append([to_host(v) for v in o])
        assert np.all(alone[b][3] == 0)
        if prec == "fp32" and b < 4:
            r = oracle.localize(Xs[b], Ks[b % len(Ks)], H, D, 1, Ns, nthreads=8, gevd=True)
            rel = float(np.max(np.abs(alone[b][2] - r["Pbar"]) / r["Pbar"]))
            print(f"  M={M} Ns={Ns} cond {cond:g}: P-bar {rel:.2e}", flush=True)
            assert rel <= 1e-4
    for _ in range(2):                              # the second call replays the captured batch
        bo = [outs(F, D, Ns) for Ns in Nss]
        S.ssl_localize_batch(ctx, [S.block_desc(Xd[b], ns_h[b % len(Ks)], Hd, D, 1, Ns, *bo[b])
                                   for b, Ns in enumerate(Nss)], p, 2)
        for b in range(len(Nss)):
            for got, ref in zip(bo[b], alone[b]):
                assert np.array_equal(to_host(got).view(np.int32), ref.view(np.int32)), b
    for n in ns_h:
        S.ssl_noise_destroy(n)


def test_failed_and_zero_bins(S, ctx):
    """A noise set that is not positive definite in one bin and a bin of zeros: statuses as with the
    noise-vector form, the failed bin adds nothing."""
    M, Ns, F, D, T = 48, 2, 6, 70, 50
    rng = np.random.default_rng(3)
    K = noise(rng, F, M, 10.0)
    K[2] = np.diag(np.r_[1.0, -1.0, np.ones(M - 2)])
    H = np.exp(2j * np.pi * rng.random((F, D, M))).astype(np.complex64)
    X = crandn(rng, F, T, M) + 5 * crandn(rng, F, T)[:, :, None] * H[:, None, 7] \
        + 4 * crandn(rng, F, T)[:, :, None] * H[:, None, 50]
    X = X.astype(np.complex64)
    X[4] = 0
    n = handle(S, ctx, K)
    got = {}
    for form in (S.SSL_PROJ_SIGNAL, S.SSL_PROJ_NOISE):
        S.ssl_ctx_set_projection(ctx, form)
        o = outs(F, D, Ns)
        S.ssl_localize(ctx, to_dev(X), n, to_dev(H), S.SSL_FP32, D, 1, Ns, 2, *o)
        got[form] = [to_host(v) for v in o]
    assert np.array_equal(got[S.SSL_PROJ_SIGNAL][3], got[S.SSL_PROJ_NOISE][3])
    assert got[S.SSL_PROJ_SIGNAL][3][2] != 0
    S.ssl_noise_destroy(n)
