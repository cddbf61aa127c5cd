"""K^{-1} by Gauss-Jordan elimination in blocks of 16 pivots (csrc/noise.hip) at the edges of its blocks
and size classes.  The inverse is read through ssl_gsvd: sigma of A = K^{-1} R against numpy's FP64
values within the SVD's bar 8 M 2^-24 |A|_F (the FP64 inverse's own error, 2^-53 cond(K), is far below
it), also for a K of condition 1e8, whose pivot blocks are as badly conditioned as K.  A pivot that is not
positive marks the bin NOT_PD wherever it stands.  MI355X only."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2504_03373_amd as S
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    S.lib()
    return S


@pytest.fixture(scope="module")
def ctx(S):
    c = S.ssl_ctx_create(0, 0)
    yield c
    S.ssl_ctx_destroy(c)


def sigma_of(S, ctx, K, R):
    import torch
    F, M, _ = K.shape
    dev = "cuda:0"
    n = S.ssl_noise_create(ctx, F, M)
    kst = torch.full((F,), -7, dtype=torch.int32, device=dev)
    S.ssl_noise_set(n, to_dev(np.ascontiguousarray(K)), S.SSL_FP64, kst)
    En = torch.zeros((F, M - 1, M), dtype=torch.complex64, device=dev)
    sg = torch.zeros((F, M), dtype=torch.float32, device=dev)
    st = torch.full((F,), -7, dtype=torch.int32, device=dev)
    S.ssl_gsvd(ctx, to_dev(R), n, 1, En, sg, st)
    out = to_host(sg), to_host(st), to_host(kst)
    S.ssl_noise_destroy(n)
    return out


@pytest.mark.parametrize("M", [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 60, 63, 64])
@pytest.mark.parametrize("cond", [1e1, 1e8])
def test_sigma_through_the_inverse(S, ctx, M, cond):
    F = 5
    rng = np.random.default_rng(int(M + cond))
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    d = cn(F, M, 1)
    d /= np.abs(d)                                        # I + rho d d^H: condition 1 + M rho
    K = np.eye(M)[None] + (cond - 1) / M * (d @ d.conj().transpose(0, 2, 1))
    X = cn(F, M, max(2, M // 2))
    R = (X @ X.conj().transpose(0, 2, 1)).astype(np.complex64)
    sg, st, kst = sigma_of(S, ctx, K, R)
    assert np.all(kst == 0) and np.all(st == 0)
    A = np.linalg.solve(K, R.astype(np.complex128))
    ref = np.linalg.svd(A, compute_uv=False)
    bar = 8 * M * 2.0 ** -24 * np.linalg.norm(A, axis=(1, 2))
    assert np.all(np.abs(sg - ref) <= bar[:, None]), np.max(np.abs(sg - ref) / bar[:, None])


@pytest.mark.parametrize("M,at", [(4, 3), (16, 0), (17, 16), (40, 15), (40, 31), (60, 59), (64, 48)])
def test_bad_pivot_marks_the_bin(S, ctx, M, at):
    """Bins: good, negative pivot, pivot at 2^-41 of the largest diagonal entry, NaN, Inf, good."""
    F = 6
    K = np.tile(np.eye(M, dtype=np.complex128), (F, 1, 1))
    for f, v in ((1, -1.0), (2, 2.0 ** -41), (3, np.nan), (4, np.inf)):
        K[f, at, at] = v
    R = np.tile(np.eye(M, dtype=np.complex64), (F, 1, 1))
    sg, st, kst = sigma_of(S, ctx, K, R)
    assert kst.tolist() == [0, 1, 1, 1, 1, 0]
    assert st.tolist() == [0, 1, 1, 1, 1, 0]
    assert np.allclose(sg[[0, 5]], 1.0, atol=1e-5) and np.all(sg[1:5] == 0)
