"""Signal vectors by block subspace iteration (csrc/subspace.hip): the p = 2 localization with
Ns <= 3 and more than 16 channels.  Against the FP64 oracle at the edges of its size classes (rows
and k-steps of its tiles: 17, 32, 33, 48, 49, 60, 61, 64 channels), over frames, sources and modes,
with the bins it leaves to the Jacobi solve (no second signal, extreme scales, non-finite input)
against the same call with the solve run to the end (SSL_STOP_NEVER, which never iterates).
MI355X only.

Bar: P-bar within 1e-4 of the oracle (the FP32 path's bar; R is FP32 and the iteration ends at the
FP32 roundoff of the weakest signal value), equal peaks where the oracle's decision is not a
near-tie."""
import sys

import numpy as np
import pytest

import oracle
import synth
from gpu_util import peak_ambiguity, to_dev, to_host

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


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


def run(S, ctx, X, n, H, grid, Ns):
    import torch
    F, D = H.shape[0], H.shape[1]
    dev = "cuda:0"
    o = dict(pk=torch.full((Ns,), -7, dtype=torch.int32, device=dev),
             pv=torch.zeros(Ns, dtype=torch.float32, device=dev),
             Pbar=torch.zeros(D, dtype=torch.float32, device=dev),
             st=torch.full((F,), -7, dtype=torch.int32, device=dev))
    S.ssl_localize(ctx, to_dev(X), n, to_dev(H), S.SSL_FP32, grid.n_az, grid.n_el, Ns, 2, o["pk"],
                   o["pv"], o["Pbar"], o["st"])
    return {k: to_host(v) for k, v in o.items()}


def full_solve(S, ctx, *a):
    """The same call without the iteration: the Jacobi solve of the whole SVD."""
    S.ssl_ctx_set_stop(ctx, S.SSL_STOP_NEVER)
    try:
        return run(S, ctx, *a)
    finally:
        S.ssl_ctx_set_stop(ctx, S.SSL_STOP_LOCALIZE)


def handle(S, ctx, K):
    F, M, _ = K.shape
    n = S.ssl_noise_create(ctx, F, M)
    S.ssl_noise_set(n, to_dev(np.ascontiguousarray(K)), S.SSL_FP64)
    return n


@pytest.mark.parametrize("mode", ["gsvd", "sevd"])
@pytest.mark.parametrize("M,Ns,F,T", [(17, 1, 33, 50), (32, 3, 40, 50), (33, 2, 17, 50),
                                      (48, 1, 29, 20), (49, 3, 21, 50), (60, 2, 73, 50),
                                      (60, 3, 31, 7), (61, 2, 19, 100), (64, 1, 16, 64),
                                      (64, 3, 23, 50)])
def test_matches_oracle(S, ctx, mode, M, Ns, F, T):
    w = synth.workload_paper(n_blocks=1, seed=4000 + M * 10 + Ns, M=M, F=F, Ns=Ns)
    w.T = T
    X, _, _ = w.block(0)
    H = w.steering_table()
    if mode == "gsvd":
        K = oracle.noise_corr(w.noise_frames())
        n = handle(S, ctx, K)
    else:
        n, K = None, np.broadcast_to(np.eye(M, dtype=np.complex128), (F, M, M)).copy()
    g = run(S, ctx, X, n, H, w.grid, Ns)
    r = oracle.localize(X, K, H, w.grid.n_az, w.grid.n_el, Ns, nthreads=8)
    rel = float(np.max(np.abs(g["Pbar"].astype(np.float64) - r["Pbar"]) / r["Pbar"]))
    amb = peak_ambiguity(r["Pbar"], w.grid.n_el, w.grid.n_az, Ns, max(rel, 1e-7))
    say(f"  {mode} M={M} Ns={Ns} F={F} T={T}: rel {rel:.2e} peaks {g['pk']} ref {r['peaks']}")
    assert np.all(g["st"] == 0)
    assert rel <= 1e-4
    if not amb:
        assert np.array_equal(g["pk"], r["peaks"])
    if n is not None:
        S.ssl_noise_destroy(n)


@pytest.mark.parametrize("kind", ["unit channels", "equal sources", "rank equals sources"])
def test_structured_bins(S, ctx, kind):
    """Input without the randomness of a scene: signals confined to single channels (A diagonal in
    the signal directions, the start block must still see them), two exactly equal signal values,
    and rank(A) = Ns."""
    M, F, T, Ns = 40, 9, 50, 2
    rng = np.random.default_rng(11)
    X = np.zeros((F, T, M), np.complex128)
    if kind == "unit channels":
        X += 1e-3 * synth.cn(rng, (F, T, M), 1.0)
        X[:, :, 3] += 3 * synth.cn(rng, (F, T), 1.0)
        X[:, :, 11] += synth.cn(rng, (F, T), 1.0)
    elif kind == "equal sources":
        X[:, ::2, 5] = 2.0                       # R = diag: two equal entries, the rest far below
        X[:, 1::2, 21] = 2.0
        X[:, :, 7] = 2.0 ** -12
    else:
        X[:, :, 2] = synth.cn(rng, (F, T), 1.0)
        X[:, :, 30] = 0.3 * synth.cn(rng, (F, T), 1.0)
    X = X.astype(np.complex64)
    grid = synth.DirectionGrid(24, 2)
    H = synth.steering_table(synth.circle_array(M), grid, synth.bin_freqs(F))
    K = np.broadcast_to(np.eye(M, dtype=np.complex128), (F, M, M)).copy()
    g = run(S, ctx, X, None, H, grid, Ns)
    r = oracle.localize(X, K, H, grid.n_az, grid.n_el, Ns, nthreads=8)
    rel = float(np.max(np.abs(g["Pbar"].astype(np.float64) - r["Pbar"]) / r["Pbar"]))
    say(f"  {kind}: rel {rel:.2e}")
    assert np.all(g["st"] == 0)
    assert rel <= 1e-4


@pytest.mark.parametrize("kind", ["small", "large", "zero bins", "one frame", "non-finite",
                                  "not positive definite"])
def test_bins_left_to_the_jacobi_solve(S, ctx, kind):
    """What the iteration cannot decide gives what the full solve gives: scales (P-bar within the bar:
    MUSIC is scale invariant), zero bins, a missing second signal, NaN and a failed noise set (the
    same status per bin; P-bar where every bin is defined)."""
    w = synth.workload_paper(n_blocks=1, seed=77, M=24, F=33, Ns=2)
    X, _, _ = w.block(0)
    H = w.steering_table()
    K = oracle.noise_corr(w.noise_frames())
    defined = True
    if kind == "small":
        X = (X * 1e-16).astype(np.complex64)      # R about 1e-31: A about 1e-31
    elif kind == "large":
        X = (X * 1e14).astype(np.complex64)
    elif kind == "zero bins":
        X[4:9] = 0
        defined = False
    elif kind == "one frame":
        X = np.ascontiguousarray(X[:, :1])
        defined = False
    elif kind == "non-finite":
        X[3, 2, 1] = np.nan
        X[5, 0, 0] = np.inf
    else:
        K[6] = np.diag(np.r_[1.0, -1.0, np.ones(w.M - 2)]).astype(complex)
    n = handle(S, ctx, K)
    g = run(S, ctx, X, n, H, w.grid, w.Ns)
    f = full_solve(S, ctx, X, n, H, w.grid, w.Ns)
    say(f"  {kind}: statuses {np.unique(g['st'])}")
    assert np.array_equal(g["st"], f["st"])
    if kind in ("non-finite", "not positive definite"):
        assert np.any(g["st"] != 0)
    if defined:
        assert np.all(np.abs(g["Pbar"] - f["Pbar"]) <= 1e-4 * f["Pbar"])
    S.ssl_noise_destroy(n)


def test_batch_equals_single_with_and_without_statistics(S, ctx):
    """Blocks of every size class in one batch, some asking for the Jacobi statistics (conv, which run
    the Jacobi solve besides) and one with bins that the iteration leaves: every block equals its
    single-block call bit for bit, on the first call and on replay."""
    import torch
    cases = []
    for i, (M, Ns) in enumerate([(17, 1), (32, 2), (40, 3), (60, 2), (64, 3), (60, 1), (16, 2)]):
        w = synth.workload_paper(n_blocks=1, seed=900 + i, M=M, F=21, Ns=Ns)
        X, _, _ = w.block(0)
        if i == 3:
            X[2] = 0
        n = handle(S, ctx, oracle.noise_corr(w.noise_frames()))
        cases.append((w, to_dev(X), n, to_dev(w.steering_table()), Ns, i % 2 == 0))

    def outs(w, Ns):
        dev = "cuda:0"
        return dict(pk=torch.full((Ns,), -7, dtype=torch.int32, device=dev),
                    pv=torch.zeros(Ns, dtype=torch.float32, device=dev),
                    Pbar=torch.zeros(w.D, dtype=torch.float32, device=dev),
                    st=torch.full((w.F,), -7, dtype=torch.int32, device=dev))

    for rep in range(2):
        bo = [outs(w, Ns) for w, _, _, _, Ns, _ in cases]
        cv = [torch.full((w.F, 3), -7, dtype=torch.int32, device="cuda:0") for w, *_ in cases]
        S.ssl_localize_batch(ctx, [
            S.block_desc(Xd, n, Hd, w.grid.n_az, w.grid.n_el, Ns, o["pk"], o["pv"], o["Pbar"],
                         o["st"], c if stats else None)
            for (w, Xd, n, Hd, Ns, stats), o, c in zip(cases, bo, cv)], S.SSL_FP32, 2)
        for (w, Xd, n, Hd, Ns, stats), o, c in zip(cases, bo, cv):
            s = outs(w, Ns)
            S.ssl_localize(ctx, Xd, n, Hd, S.SSL_FP32, w.grid.n_az, w.grid.n_el, Ns, 2, s["pk"],
                           s["pv"], s["Pbar"], s["st"])
            for k in s:
                assert np.array_equal(to_host(s[k]), to_host(o[k])), (rep, w.M, Ns, k)
            conv = to_host(c)
            assert np.all(conv[:, 2] >= 0) if stats else np.all(conv == -7)
    for _, _, n, _, _, _ in cases:
        S.ssl_noise_destroy(n)
