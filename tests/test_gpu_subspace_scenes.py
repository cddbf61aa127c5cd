"""Scenes that do not hold as many resolved sources as are asked for: one source over floors 20 to 60 dB below,
none at all (short and long averages), silence, fewer frames than sources.  The signal subspace is then ill
conditioned or not defined, and the subspace iteration (csrc/subspace.hip) has to decide such bins or to leave
them to the Jacobi solve soon.  MI355X only.

Accuracy: P-bar against the FP64 oracle, no further from it than 1e-4 or four times what the Jacobi solve of the
whole SVD (SSL_STOP_NEVER) is on the same input: with close singular values both are limited by A's rounding
to complex64.  Time: at most three times that solve's, and 60 us."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import S, ctx, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
GRID = synth.DirectionGrid(24, 2)


def frames(kind, M, F, rng):
    T = {"one frame": 1, "long average": 500}.get(kind, 50)
    H = synth.steering_table(synth.circle_array(M), GRID, synth.bin_freqs(257)[60:60 + F]).astype(complex)
    X = np.zeros((F, T, M), complex)
    if "dB" in kind or kind == "noise free":
        X += synth.cn(rng, (F, T, 1), 1.0) * H[:, 9][:, None, :]
        if kind != "noise free":
            X += 10 ** (-float(kind.split()[0]) / 20) * synth.cn(rng, (F, T, M), 1.0)
    elif kind != "silence":
        X += synth.cn(rng, (F, T, M), 1.0)
    return X.astype(np.complex64), H.astype(np.complex64)


def caller(S, ctx, X, H, Ns):  # noqa: F811
    import torch
    dev = "cuda:0"
    Xd, Hd = to_dev(X), to_dev(H)
    o = dict(pk=torch.full((Ns,), -7, dtype=torch.int32, device=dev),
             pv=torch.zeros(Ns, dtype=torch.float32, device=dev),
             Pbar=torch.zeros(H.shape[1], dtype=torch.float32, device=dev),
             st=torch.full((X.shape[0],), -7, dtype=torch.int32, device=dev))
    return o, lambda: S.ssl_localize(ctx, Xd, None, Hd, S.SSL_FP32, GRID.n_az, GRID.n_el, Ns, 2, o["pk"], o["pv"],
                                     o["Pbar"], o["st"])


@pytest.fixture
def full(S, ctx):  # noqa: F811
    def run(fn):
        S.ssl_ctx_set_stop(ctx, S.SSL_STOP_NEVER)
        try:
            return fn()
        finally:
            S.ssl_ctx_set_stop(ctx, S.SSL_STOP_LOCALIZE)
    return run


@pytest.mark.parametrize("kind", ["20 dB", "30 dB", "40 dB", "60 dB", "noise", "long average"])
@pytest.mark.parametrize("M,Ns", [(8, 2), (16, 3), (24, 2), (48, 2), (60, 3)])
def test_accuracy(S, ctx, full, M, Ns, kind):  # noqa: F811
    F = 19
    X, H = frames(kind, M, F, np.random.default_rng(M + len(kind)))
    o, call = caller(S, ctx, X, H, Ns)
    call()
    got, st = to_host(o["Pbar"]), to_host(o["st"])
    full(call)
    ref_gpu = to_host(o["Pbar"])
    K = np.broadcast_to(np.eye(M, dtype=complex), (F, M, M)).copy()
    ref = oracle.localize(X, K, H, GRID.n_az, GRID.n_el, Ns, nthreads=8)["Pbar"]
    err, err_full = (float(np.max(np.abs(p.astype(np.float64) - ref) / ref)) for p in (got, ref_gpu))
    print(f"  M={M} Ns={Ns} {kind}: P-bar {err:.1e}, whole SVD {err_full:.1e}", flush=True)
    assert np.all(st == 0)
    assert err <= max(1e-4, 4 * err_full)


@pytest.mark.parametrize("kind", ["silence", "one frame", "noise free", "40 dB", "noise"])
@pytest.mark.parametrize("M", [8, 16, 24, 60])
def test_time(S, ctx, full, M, kind):  # noqa: F811
    import torch
    X, H = frames(kind, M, 129, np.random.default_rng(M))
    _, call = caller(S, ctx, X, H, 2)

    def once():
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            call()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / 5 * 1e3

    call()
    full(call)
    now, whole = min(once() for _ in range(5)), min(full(once) for _ in range(5))
    print(f"  M={M} {kind}: {now:.0f} us, whole SVD {whole:.0f} us", flush=True)
    assert now <= 3 * whole + 60
