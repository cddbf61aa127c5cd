"""ssl_sliding_localize without conv: windows through the signal subspace.  Against the FP64 oracle on
each window, cold and warm, between calls that ask for conv (whose kept singular vectors have to
stay usable), at 8, 16 and 60 channels, and with the modes that keep the whole solve.  MI355X only."""
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


@pytest.mark.parametrize("M,Ns,mode", [(8, 1, "default"), (16, 3, "default"), (60, 2, "default"),
                                       (60, 2, "stop_never"), (60, 2, "noise_form"), (9, 4, "default")])
def test_windows_without_conv(S, M, Ns, mode):
    import torch
    ctx = S.ssl_ctx_create(0, 0)
    if mode == "stop_never":
        S.ssl_ctx_set_stop(ctx, S.SSL_STOP_NEVER)
    if mode == "noise_form":
        S.ssl_ctx_set_projection(ctx, S.SSL_PROJ_NOISE)
    F, T, az, hop = 20, 50, 90, 10
    rng = np.random.default_rng(17 * M + Ns)
    H = np.exp(2j * np.pi * rng.random((F, az, M))).astype(np.complex64)
    X = crandn(rng, F, T + 6 * hop, M)
    for k, d in enumerate(rng.choice(az, Ns, replace=False)):
        X += (6.0 - k) * crandn(rng, F, X.shape[1])[:, :, None] * H[:, None, d]
    X = X.astype(np.complex64)
    Xn = crandn(rng, F, 4 * M, M).astype(np.complex64)
    K = oracle.noise_corr(Xn)
    n = S.ssl_noise_create(ctx, F, M)
    S.ssl_noise_set(n, to_dev(K), S.SSL_FP64)
    Hd, Xd = to_dev(H), to_dev(X)
    s = S.ssl_sliding_create(ctx, F, M, T)
    S.ssl_sliding_push(s, Xd[:, :T])
    pk = torch.zeros(Ns, dtype=torch.int32, device="cuda:0")
    pv = torch.zeros(Ns, device="cuda:0")
    Pbar = torch.zeros(az, device="cuda:0")
    st = torch.full((F,), -7, dtype=torch.int32, device="cuda:0")
    conv = torch.zeros((F, 3), dtype=torch.int32, device="cuda:0")
    plan = [(0, None), (1, None), (1, conv), (0, None), (1, conv), (1, None)]   # (warm, conv)
    for i, (warm, cv) in enumerate(plan):
        f = T + i * hop - 1
        S.ssl_sliding_localize(s, n, Hd, S.SSL_FP32, az, 1, Ns, 2, warm, pk, pv, Pbar, st, cv)
        r = oracle.localize_frame(X, T, f, K, H, az, 1, Ns, nthreads=8)
        rel = float(np.max(np.abs(to_host(Pbar) - r["Pbar"]) / r["Pbar"]))
        print(f"  M={M} {mode} window {i} warm {warm} conv {cv is not None}: P-bar {rel:.2e}", flush=True)
        assert np.all(to_host(st) == 0) and rel <= 1e-4
        assert np.array_equal(to_host(pk), r["peaks"])
        if cv is not None and i == 4:
            assert np.all(to_host(cv)[:, 2] == M)              # from the vectors kept at window 2
        S.ssl_sliding_push(s, Xd[:, f + 1:f + 1 + hop])
    S.ssl_sliding_destroy(s)
    S.ssl_noise_destroy(n)
    S.ssl_ctx_destroy(ctx)
