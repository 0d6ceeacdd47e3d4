"""A batched step's two parts: clouds that meet tol at the first correction beside
clouds whose refinement goes on (plain steps, GMRES), for fixed scales and for both
search methods, against the single solves; and the one-launch check of all clouds."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


# factors of the cutoff scale: none, some and all of the clouds go on after the first correction
@pytest.mark.parametrize("factors", [(1.0, 0.8, 1.5, 2.0), (1.0, 0.02, 1.5, 0.03), (0.02, 0.03, 0.025, 0.02)])
def test_fixed_scales(mag, factors):
    sizes = (300, 129, 1, 512)
    clouds = [W.gaussian(n, 3, seed=n) for n in sizes]
    ts = [f * W.gaussian_cutoff_estimate(max(n, 2), 3) for f, n in zip(factors, sizes)]
    Xp, offs = W.pack_clouds(clouds)
    w, M, info = mag.weighting_batch(dev(Xp), offs, ts)
    w = w.cpu().numpy()
    rounds = [i["outer_iters"] for i in info]
    print(rounds)
    for b, (X, t) in enumerate(zip(clouds, ts)):
        wb = w[offs[b]:offs[b + 1]]
        assert info[b]["resid_inf"] <= 1e-12
        assert np.abs(oracle.residual(X, t, wb)).max() <= 1.1e-12
        assert M[b] == pytest.approx(wb.sum(), rel=1e-14)
        assert rounds[b] > 2 or factors[b] >= 0.5 or sizes[b] == 1


@pytest.mark.parametrize("method", ["bisection", "ridders"])
def test_searches_match_single(mag, method):
    clouds = [W.gaussian_mixture(n, 3, seed=n) for n in (200, 90, 333)] + [W.gaussian(150, 3, seed=9)]
    Xp, offs = W.pack_clouds(clouds)
    tp, w, info = mag.tplus_batch(dev(Xp), offs, want_w=True, rtol=1e-10, method=method)
    for b, X in enumerate(clouds):
        one = mag.tplus(dev(X), rtol=1e-10, method=method)
        # both brackets hold the root to rtol
        assert tp[b] == pytest.approx(one.t_plus, rel=3e-10)
        assert np.abs(oracle.residual(X, tp[b], w.cpu().numpy()[offs[b]:offs[b + 1]])).max() <= 1.1e-12


@pytest.mark.parametrize("n", [1, 2, 64, 128, 129, 700])
def test_validation(mag, n):
    # the last coordinate of the last cloud, its only coincident pair, and the smallest distance
    clouds = [W.gaussian(65, 3, seed=1), W.gaussian(n, 3, seed=2)]
    Xp, offs = W.pack_clouds(clouds)
    mag.weighting_batch(dev(Xp), offs, [2.0, 2.0])
    for v in (np.nan, np.inf, -np.inf):
        Y = Xp.copy()
        Y[-1, -1] = v
        with pytest.raises(mag.MagError) as e:
            mag.weighting_batch(dev(Y), offs, [2.0, 2.0])
        assert e.value.code == -1
    if n > 1:
        Y = Xp.copy()
        Y[-1] = Y[-n]
        with pytest.raises(mag.MagError) as e:
            mag.weighting_batch(dev(Y), offs, [2.0, 2.0])
        assert e.value.code == -2
        info = mag.tplus_batch(dev(Xp), offs)[2]
        assert info[1]["d_min"] == mag.dmin(dev(clouds[1]))


@pytest.mark.parametrize("sizes", [(1, 256, 257, 511), (512, 513, 100, 769), (1300, 1025, 640)])
def test_panels_and_the_path_without_room_for_them(mag, sizes):
    clouds = [W.gaussian(n, 3, seed=n) for n in sizes]
    Xp, offs = W.pack_clouds(clouds)
    ts = [W.gaussian_cutoff_estimate(max(n, 2), 3) for n in sizes]
    out = []
    free, capped = mag.Context(0), mag.Context(0)
    for _ in range(2):  # the second call finds the exchanges as the first left them
        out.append(mag.weighting_batch(dev(Xp), offs, ts, ctx=free)[0].cpu().numpy())
    capped.set_workspace_limit(free.workspace_bytes() - 1)  # the panels' exchanges come last
    out.append(mag.weighting_batch(dev(Xp), offs, ts, ctx=capped)[0].cpu().numpy())
    assert capped.workspace_bytes() < free.workspace_bytes()
    assert np.array_equal(out[0], out[1])
    for w in out:
        for b, (X, t) in enumerate(zip(clouds, ts)):
            assert np.abs(oracle.residual(X, t, w[offs[b]:offs[b + 1]])).max() <= 1.1e-12
    free.close()
    capped.close()
