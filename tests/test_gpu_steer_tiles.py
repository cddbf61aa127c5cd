"""Tiles of the signal-subspace projection (csrc/steer_sig.hip): channel counts around its k-steps (a
remainder of 0, 1..4 and 5..7 of 8 channels, an odd count, a table that is not 16-byte aligned),
column tiles of mixed Ns filled exactly, over and under, one or several direction tiles per
workgroup, and every table precision.  A block alone against the FP64 oracle (P-bar within 1e-4,
the FP32 path's bar), the blocks of a batch against each alone, bit for bit.  MI355X only."""
import numpy as np
import pytest

import oracle
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


def scene(M, F, D, T, nb):
    """Unit-modulus table, frames of two of its directions (three where M allows) in white noise."""
    rng = np.random.default_rng(1000 * M + D + nb)
    H = np.exp(2j * np.pi * rng.random((F, D, M))).astype(np.complex64)
    Xs = []
    for _ in range(nb):
        X = rng.standard_normal((F, T, M)) + 1j * rng.standard_normal((F, T, M))
        for k, d in enumerate(rng.choice(D, 3, replace=False)):
            s = rng.standard_normal((F, T)) + 1j * rng.standard_normal((F, T))
            X += (5.0 - k) * s[:, :, None] * H[:, None, d].astype(np.complex128)
        Xs.append(X.astype(np.complex64))
    return H, Xs


def table(S, H, prec, shift):
    """The table on the device, its start moved by one element where shift."""
    import torch
    t = to_dev(H)
    if prec != S.SSL_FP32:
        t = torch.view_as_real(t).to(torch.bfloat16 if prec == S.SSL_BF16 else torch.float16)
        rounded = torch.view_as_complex(t.float().contiguous()).cpu().numpy()
        t = t.reshape(H.shape[0], H.shape[1], 2 * H.shape[2])
    else:
        rounded = H
    if shift:
        step = 1 if prec == S.SSL_FP32 else 2
        buf = torch.zeros(t.numel() + step, dtype=t.dtype, device="cuda:0")
        buf[step:] = t.reshape(-1)
        t = buf[step:].view(t.shape)
    return t.contiguous(), rounded


def outs(F, D, Ns):
    import torch
    return (torch.full((Ns,), -7, dtype=torch.int32, device="cuda:0"),
            torch.zeros(Ns, device="cuda:0"), torch.zeros(D, device="cuda:0"),
            torch.full((F,), -7, dtype=torch.int32, device="cuda:0"))


@pytest.mark.parametrize("M,az,Nss,shift,prec", [
    (5, 65, [1, 2, 3], False, "fp32"),             # lone k-step of 5..8
    (8, 64, [1] * 16, False, "fp32"),              # one tile, exactly full
    (16, 63, [1, 2, 3] * 6, False, "bf16"),        # 36 columns: streamed
    (17, 130, [3] * 5 + [1], False, "fp32"),       # odd, exactly 16 columns
    (22, 200, [3] * 10, True, "fp32"),             # 30 columns in two resident tiles, unaligned
    (33, 65, [2] * 16, False, "fp16"),             # 32 columns
    (47, 129, [1, 1, 2, 3, 3, 2], True, "bf16"),
    (60, 193, [3] * 6 + [2] * 8, True, "fp32"),    # 34 columns, mixed
    (61, 64, [2], False, "fp32"),
    (64, 65, [1, 3, 2, 3], False, "fp16"),
])
def test_tiles(S, ctx, M, az, Nss, shift, prec):
    F, T, nb = 70, 40 if M > 32 else 30, len(Nss)
    p = {"fp32": S.SSL_FP32, "bf16": S.SSL_BF16, "fp16": S.SSL_FP16}[prec]
    H, Xs = scene(M, F, az, T, nb)
    if prec != "fp32":
        s = max(np.abs(X.view(np.float32)).max() for X in Xs)
        Xs = [(X / s).astype(np.complex64) for X in Xs]
    Hd, Hr = table(S, H, p, shift)
    Xd = [to_dev(X) for X in Xs]
    alone = []
    for X, ns in zip(Xd, Nss):
        o = outs(F, az, ns)
        S.ssl_localize(ctx, X, None, Hd, p, az, 1, ns, 2, *o)
        alone.append([to_host(v) for v in o])
    if prec == "fp32":
        for b in (0, nb - 1):
            I = np.broadcast_to(np.eye(M, dtype=np.complex128), (F, M, M))
            r = oracle.localize(Xs[b], I, Hr, az, 1, Nss[b], nthreads=8)
            rel = np.max(np.abs(alone[b][2] - r["Pbar"]) / r["Pbar"])
            print(f"  M={M} block {b}: P-bar {rel:.2e}", flush=True)
            assert np.all(alone[b][3] == 0) and rel <= 1e-4
    for _ in range(2):                              # the second call replays the captured batch
        bo = [outs(F, az, ns) for ns in Nss]
        S.ssl_localize_batch(ctx, [S.block_desc(X, None, Hd, az, 1, ns, *o)
                                   for X, ns, o in zip(Xd, Nss, bo)], p, 2)
        for b in range(nb):
            for got, ref in zip(bo[b], alone[b]):
                assert np.array_equal(to_host(got).view(np.int32), ref.view(np.int32)), b
