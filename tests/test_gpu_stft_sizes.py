"""ssl_stft at the sizes whose transforms have an even number of stages (one radix-2 pass fewer) and at
channel counts around a workgroup's, with channels 10^6 apart in level: each frame and channel against
numpy's FP64 transform within (8 log2 N + 4) u sqrt(N) |w x| of its own norm.  MI355X only."""
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


@pytest.mark.parametrize("nfft,hop,T,M", [(32, 8, 9, 16), (128, 128, 5, 15), (256, 64, 6, 33), (512, 1, 3, 2),
                                          (2048, 512, 4, 5), (1024, 512, 2, 64)])
def test_sizes(S, nfft, hop, T, M):
    import torch
    ctx = S.ssl_ctx_create(0, 0)
    rng = np.random.default_rng(nfft + M)
    x = rng.standard_normal(((T - 1) * hop + nfft, M)).astype(np.float32)
    x[:, 1::2] *= np.float32(1e-6)
    X = torch.zeros(nfft // 2 + 1, T, M, dtype=torch.complex64, device="cuda:0")
    S.ssl_stft(ctx, to_dev(x), nfft, hop, T, X)
    got = to_host(X).astype(np.complex128)
    w = np.sin(np.pi * np.arange(nfft) / nfft) ** 2
    for t in range(T):
        y = x[t * hop:t * hop + nfft].astype(np.float64) * w[:, None]
        err = np.linalg.norm(got[:, t] - np.fft.rfft(y, axis=0), axis=0)
        bound = (8 * np.log2(nfft) + 4) * 2.0 ** -24 * np.sqrt(nfft) * np.linalg.norm(y, axis=0)
        assert np.all(err <= bound), (t, (err / bound).max())
    S.ssl_ctx_destroy(ctx)
