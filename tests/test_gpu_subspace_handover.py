"""What the subspace iteration (csrc/subspace.hip) hands over to the Jacobi solve behind it, and what the
caller's bin_status sees of it.  MI355X only."""
import numpy as np
import pytest

import synth
from gpu_util import S, ctx, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu


def scene(F, M, T, grid, weak, seed, floor=1e-4):
    """Two sources over a white floor, the second with `weak` of the first's amplitude; X and the steering
    table.  No noise set: A is R."""
    rng = np.random.default_rng(seed)
    H = synth.steering_table(synth.circle_array(M), grid, synth.bin_freqs(257)[100:100 + F])
    s = synth.cn(rng, (F, T, 2), 1.0) * np.array([1.0, weak])
    X = s @ H[:, [grid.n_az // 3, 2 * grid.n_az // 3], :].astype(complex)
    return (X + floor * synth.cn(rng, (F, T, M), 1.0)).astype(np.complex64), H


def sigma(X):
    """Singular values of R per bin."""
    return np.linalg.svd(X.astype(complex), compute_uv=False) ** 2 / X.shape[1]


def single(S, ctx, X, H, grid):  # noqa: F811
    o = outs(X.shape[0], grid.n_az * grid.n_el)
    S.ssl_localize(ctx, to_dev(X), None, to_dev(H), S.SSL_FP32, grid.n_az, grid.n_el, 2, 2, o["pk"], o["pv"],
                   o["Pbar"], o["st"])
    return {k: to_host(v) for k, v in o.items()}


def outs(F, D, Ns=2):
    import torch
    dev = "cuda:0"
    return dict(pk=torch.full((Ns,), -7, dtype=torch.int32, device=dev),
                pv=torch.zeros(Ns, dtype=torch.float32, device=dev),
                Pbar=torch.zeros(D, dtype=torch.float32, device=dev),
                st=torch.full((F,), -7, dtype=torch.int32, device=dev))


@pytest.mark.parametrize("M", [8, 24, 60])
def test_blocks_sharing_a_status_array(S, ctx, M):  # noqa: F811
    """Two blocks of a batch write one bin_status: every bin of the first is left to the Jacobi solve, none
    of the second, so that a hand-over in the caller's array would cross.  As with arrays of their own."""
    import torch
    F, T, grid = 37, 40, synth.DirectionGrid(24, 2)
    hard, H = scene(F, M, T, grid, 0.02, M)
    easy, _ = scene(F, M, T, grid, 0.7, M + 1)
    th = sigma(hard) ** 2
    assert np.all(th[:, 1] < 1e-6 * th[:, 0])          # below the ratio that the iteration decides
    th = sigma(easy) ** 2
    assert np.all(th[:, 1] > 1e-4 * th[:, 0]) and np.all(th[:, 2] < 1e-6 * th[:, 1])
    Hd, Xd = to_dev(H), [to_dev(hard), to_dev(easy)]

    def batch(share):
        o = [outs(F, grid.n_az * grid.n_el) for _ in Xd]
        if share:
            o[1]["st"] = o[0]["st"]
        S.ssl_localize_batch(ctx, [S.block_desc(x, None, Hd, grid.n_az, grid.n_el, 2, q["pk"], q["pv"], q["Pbar"],
                                                q["st"]) for x, q in zip(Xd, o)], S.SSL_FP32, 2)
        return [{k: to_host(v) for k, v in q.items()} for q in o]

    own, shared = batch(False), batch(True)
    for b in range(2):
        assert np.all(own[b]["st"] == 0)
        for k in own[b]:
            assert np.array_equal(own[b][k], shared[b][k]), (b, k)
    torch.cuda.synchronize()


@pytest.mark.parametrize("M", [8, 24, 60])
def test_any_magnitude(S, ctx, M):  # noqa: F811
    """Frames scaled by a power of two (R from 2^-95 to 2^115): every step of the iteration is the same, so the
    results are, bit for bit, also in bins that take many steps (sources close to the floor)."""
    F, T, grid = 37, 40, synth.DirectionGrid(24, 2)
    X, H = scene(F, M, T, grid, 0.4, M + 2, floor=0.4)
    ref = single(S, ctx, X, H, grid)
    assert np.all(ref["st"] == 0)
    for k in (-47, -30, 30, 55):
        g = single(S, ctx, (X * np.float32(2.0 ** k)).astype(np.complex64), H, grid)
        for name in ref:
            assert np.array_equal(g[name], ref[name]), (k, name)


def test_lists_of_bins_left(S, ctx):  # noqa: F811
    """Blocks of every Jacobi class in one batch, replayed on other data: all bins left to the Jacobi solve,
    none, every other one, in blocks with and without the Jacobi statistics.  Every call equals its blocks'
    single-block calls bit for bit and has the statistics of the first."""
    import torch
    F, T, grid = 41, 30, synth.DirectionGrid(24, 2)
    cases = []
    for M, stats in ((8, False), (16, True), (24, False), (60, True), (60, False), (12, False)):
        hard, H = scene(F, M, T, grid, 0.0, M, floor=0.0)          # rank 1: no second direction
        easy, _ = scene(F, M, T, grid, 0.7, M + 1)
        mixed = easy.copy()
        mixed[::2] = hard[::2]
        cases.append(dict(data=[to_dev(x) for x in (hard, easy, mixed)], X=to_dev(easy), H=to_dev(H), o=outs(F, 48),
                          cv=torch.zeros((F, 3), dtype=torch.int32, device="cuda:0") if stats else None))

    def call():
        S.ssl_localize_batch(ctx, [S.block_desc(c["X"], None, c["H"], grid.n_az, grid.n_el, 2, c["o"]["pk"],
                                                c["o"]["pv"], c["o"]["Pbar"], c["o"]["st"], c["cv"]) for c in cases],
                             S.SSL_FP32, 2)

    seen = {}
    for kind in (0, 1, 2, 1, 0, 2):
        for c in cases:
            c["X"].copy_(c["data"][kind])
            if c["cv"] is not None:
                c["cv"].fill_(-7)
        call()
        for n, c in enumerate(cases):
            s = outs(F, 48)
            S.ssl_localize(ctx, c["X"], None, c["H"], S.SSL_FP32, grid.n_az, grid.n_el, 2, 2, s["pk"], s["pv"],
                           s["Pbar"], s["st"])
            for k in s:
                assert np.array_equal(to_host(s[k]), to_host(c["o"][k])), (kind, n, k)
            if c["cv"] is not None:
                cv = to_host(c["cv"])
                assert np.all(cv >= 0)
                assert np.array_equal(seen.setdefault((kind, n), cv), cv)


@pytest.mark.parametrize("kind", ["zero bins", "rank one"])
@pytest.mark.parametrize("M", [8, 16, 33, 60])
def test_left_bins_among_others(S, ctx, M, kind):  # noqa: F811
    """P-bar of a block with undefined bins (zero, or without a second signal) is that of its defined bins
    plus that of the others: what is left to the Jacobi solve changes nothing in the bins beside it."""
    F, T, grid = 29, 40, synth.DirectionGrid(24, 2)
    X, H = scene(F, M, T, grid, 0.7, M)
    out = np.arange(F) % 5 == 2
    X[out] = 0 if kind == "zero bins" else scene(F, M, T, grid, 0.0, M + 3, floor=0.0)[0][out]
    th = sigma(X) ** 2
    assert np.all(th[out, 1] <= 1e-12 * th[out, 0]) and np.all(th[~out, 1] > 1e-4 * th[~out, 0])
    full = single(S, ctx, X, H, grid)
    parts = [single(S, ctx, np.ascontiguousarray(X[m]), np.ascontiguousarray(H[m]), grid) for m in (~out, out)]
    assert np.all(full["st"] == 0) and np.all(parts[0]["st"] == 0)
    want = parts[0]["Pbar"].astype(np.float64) + parts[1]["Pbar"]
    # a sum of F terms in another order: F 2^-24
    assert np.all(np.abs(full["Pbar"] - want) <= F * 2.0 ** -24 * want)
