"""ssl_corr_accum in FP64 at the edges of its chunks of 64 frames and of its 16 x 16 tiles, stored and
accumulated: against numpy in complex128 within the rounding of 2 T products and sums per part
(2 (T + 2) 2^-53 sum |x_i| |x_j|), Hermitian to the bit.  MI355X only."""
import numpy as np
import pytest

from conftest import crandn
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 47, 60, 64])
@pytest.mark.parametrize("T", [1, 3, 64, 65, 130])
def test_corr_f64(M, T):
    import torch
    import paper_2504_03373_amd as S
    ctx = S.ssl_ctx_create(0, 0)
    rng = np.random.default_rng(M * 1000 + T)
    F = 5
    X = (crandn(rng, F, T, M) * np.logspace(-3, 3, M)).astype(np.complex64)
    R0 = crandn(rng, F, M, M)
    R0 = R0 + R0.conj().transpose(0, 2, 1)
    x = X.astype(np.complex128)
    ref = np.einsum("fti,ftj->fij", x, x.conj())
    mag = 2 * (T + 2) * 2.0 ** -53 * np.einsum("fti,ftj->fij", abs(x), abs(x)) / T
    for acc in (0, 1):
        R = to_dev(R0)
        S.ssl_corr_accum(ctx, to_dev(X), 1.0 / T, acc, S.SSL_FP64, R)
        got = to_host(R)
        want = ref / T + (R0 if acc else 0)
        bound = np.sqrt(2) * mag + 2.0 ** -52 * abs(want)
        assert np.all(abs(got - want) <= bound), (acc, (abs(got - want) / bound).max())
        assert np.array_equal(got, got.conj().transpose(0, 2, 1))
    S.ssl_ctx_destroy(ctx)
