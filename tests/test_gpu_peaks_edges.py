"""The bin sum's last launch and the peak search at their edges: more directions than a pass of the
workgroup takes and than its LDS copy holds, grids one and two azimuths wide, equal values (the lower
index wins), signed zeros, non-finite values, fewer maxima than asked for, and chunk counts around the
number summed at once (P-bar against the same FP32 sum in numpy, exactly).  MI355X only."""
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


def rule(pb, n_az, n_el, Ns):
    """Sec. III-A's local maxima, by value, then by lower index."""
    found = []
    for d in range(n_az * n_el):
        if not np.isfinite(pb[d]):
            continue
        el, az = divmod(d, n_az)
        nbs = {e * n_az + a % n_az for e in range(max(el - 1, 0), min(el + 1, n_el - 1) + 1)
               for a in (az - 1, az, az + 1)} - {d}
        if all(not np.isfinite(pb[b]) or pb[d] > pb[b] or (pb[d] == pb[b] and d < b) for b in nbs):
            found.append(d)
    found.sort(key=lambda d: (-pb[d], d))
    idx = (found + [-1] * Ns)[:Ns]
    return np.array(idx, np.int32), np.array([pb[d] if d >= 0 else 0.0 for d in idx], np.float32)


@pytest.mark.parametrize("n_az,n_el", [(1, 1), (1, 7), (2, 5), (3, 1), (72, 19), (64, 16), (65, 32),
                                       (64, 128), (91, 91)])
@pytest.mark.parametrize("values", ["plain", "ties", "odd"])
def test_peaks(S, ctx, n_az, n_el, values):
    import torch
    rng = np.random.default_rng(n_az * 100 + n_el)
    D, Ns = n_az * n_el, 5
    pb = rng.standard_normal(D).astype(np.float32)
    if values == "ties":
        pb = np.sign(pb).astype(np.float32) * np.float32(0.5) * rng.integers(0, 2, D).astype(np.float32)
    if values == "odd":
        for v in (np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-40, -3.4028235e38):
            pb[rng.integers(0, D, max(D // 9, 1))] = v
    pk = torch.full((Ns,), -7, dtype=torch.int32, device="cuda:0")
    pv = torch.full((Ns,), -7.0, device="cuda:0")
    S.ssl_peaks(ctx, to_dev(pb), n_az, n_el, Ns, pk, pv)
    i, v = rule(pb, n_az, n_el, Ns)
    assert np.array_equal(to_host(pk), i), (to_host(pk), i)
    assert np.array_equal(to_host(pv), v)


@pytest.mark.parametrize("F,n_az,n_el", [(1, 72, 1), (16, 33, 31), (255, 64, 32), (257, 64, 33),
                                         (513, 72, 19), (40, 128, 65)])
def test_bin_sum(S, ctx, F, n_az, n_el):
    """P-bar from ssl_music_spectrum's own P: chunks of 16 bins in order, then the chunks in order."""
    import torch
    rng = np.random.default_rng(F + n_az)
    D, M, Ns = n_az * n_el, 4, 2
    H = (rng.standard_normal((F, D, M)) + 1j * rng.standard_normal((F, D, M))).astype(np.complex64)
    E = (rng.standard_normal((F, M - Ns, M)) + 1j * rng.standard_normal((F, M - Ns, M))).astype(np.complex64)
    P = torch.zeros(F, D, device="cuda:0")
    Pbar = torch.zeros(D, device="cuda:0")
    S.ssl_music_spectrum(ctx, to_dev(H), S.SSL_FP32, to_dev(E), Ns, 2, P, Pbar, None)
    p = to_host(P)
    parts = []
    for f in range(0, F, 16):
        s = np.zeros(D, np.float32)
        for b in range(f, min(f + 16, F)):
            s += p[b]
        parts.append(s)
    ref = np.zeros(D, np.float32)
    for s in parts:
        ref += s
    assert np.array_equal(to_host(Pbar), ref)
