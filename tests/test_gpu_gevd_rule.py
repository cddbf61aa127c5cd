"""Which GEVD-MUSIC blocks go through the signal subspace (use_sig, csrc/abi.hip): the sizes on both sides of
the rule's edges, by the rounding of P-bar, which tells the two forms of eq.5 apart; the sizes that take the form
against the oracle and in batches; and what a failed bin adds.  MI355X only."""
import numpy as np
import pytest

import test_gpu_gevd_signal as sig
from conftest import crandn
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
S, ctx = sig.S, sig.ctx


def localize(S, ctx, X, n, H, Ns, form):
    S.ssl_ctx_set_projection(ctx, form)
    o = sig.outs(H.shape[0], H.shape[1], Ns)
    S.ssl_localize(ctx, to_dev(X), n, to_dev(H), S.SSL_FP32, H.shape[1], 1, Ns, 2, *o)
    S.ssl_ctx_set_projection(ctx, S.SSL_PROJ_SIGNAL)
    return [to_host(v) for v in o]


def scene(M, F, D, rng, K):
    H = np.exp(2j * np.pi * rng.random((F, D, M))).astype(np.complex64)
    X = np.einsum("fij,ftj->fti", np.linalg.cholesky(K), crandn(rng, F, 50, M))
    for a, d in ((5, 7), (4, 50)):
        X += a * crandn(rng, F, 50)[:, :, None] * H[:, None, d]
    return X.astype(np.complex64), H


@pytest.mark.parametrize("M,Ns,signal", [(16, 2, False), (29, 2, False), (30, 2, True), (32, 1, False), (33, 2, False),
                                         (35, 2, False), (36, 2, True), (40, 3, True), (48, 2, True),
                                         (49, 2, False), (56, 2, False), (57, 2, True), (58, 3, True),
                                         (59, 2, True), (60, 2, True), (60, 1, False), (61, 2, False)])
def test_rule(S, ctx, M, Ns, signal):
    F, D = 9, 70
    rng = np.random.default_rng(M)
    K = sig.noise(rng, F, M, 10.0)
    X, H = scene(M, F, D, rng, K)
    n = sig.handle(S, ctx, K)
    a, b = (localize(S, ctx, X, n, H, Ns, f)[2] for f in (S.SSL_PROJ_SIGNAL, S.SSL_PROJ_NOISE))
    assert np.max(np.abs(a - b) / b) <= 1e-4
    assert np.array_equal(a, b) != signal
    S.ssl_noise_destroy(n)


@pytest.mark.parametrize("M,Nss,own,cond,prec", [(36, [2, 3, 2], False, 1e3, "fp32"), (37, [2, 3], True, 10.0, "fp16"),
                                                 (41, [3] * 6, False, 1e4, "fp32"), (44, [2] * 3, True, 10.0, "fp32"),
                                                 (57, [2, 3, 3], True, 1e3, "fp32"), (58, [2] * 9, False, 10.0, "bf16"),
                                                 (59, [2, 3], False, 1e4, "fp32")])
def test_sizes(S, ctx, M, Nss, own, cond, prec):
    sig.test_sizes(S, ctx, M, Nss, own, cond, prec)


@pytest.mark.parametrize("M", [36, 48, 60])
def test_failed_bin_adds_nothing(S, ctx, M):
    """P-bar with a bin whose noise set is not positive definite equals P-bar without the bin, bit for bit."""
    F, D = 6, 70
    rng = np.random.default_rng(M + 1)
    K = sig.noise(rng, F, M, 10.0)
    X, H = scene(M, F, D, rng, K)
    K[2] = np.diag(np.r_[1.0, -1.0, np.ones(M - 2)])
    keep = np.r_[0, 1, 3, 4, 5]
    got = []
    for f in (np.arange(F), keep):
        n = sig.handle(S, ctx, K[f])
        got.append(localize(S, ctx, np.ascontiguousarray(X[f]), n, np.ascontiguousarray(H[f]), 2, S.SSL_PROJ_SIGNAL))
        S.ssl_noise_destroy(n)
    assert got[0][3].tolist() == [0, 0, 1, 0, 0, 0] and np.all(got[1][3] == 0)
    for i in (0, 1, 2):
        assert np.array_equal(got[0][i], got[1][i])
