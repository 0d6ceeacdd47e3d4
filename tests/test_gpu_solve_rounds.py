"""The speculated first rounds of a solve (x0, one plain step and both residuals
enqueued at once): answers taken at x0, at x1 and later, the limits that leave no
room for the step, bad points and FP32 breakdowns found after the step was
enqueued; and the matrix-free product at the edges of its two tile sizes."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 257, 3072, 3073])
def test_product_at_tile_edges(mag, n):
    X = W.gaussian(n, 3, seed=n)
    v = np.random.default_rng(n).standard_normal(n)
    y = mag.zmatvec(dev(X), 1.7, dev(v)).cpu().numpy()
    scale = oracle.zmatvec(X, 1.7, np.abs(v))
    assert np.all(np.abs(y - oracle.zmatvec(X, 1.7, v)) <= 64 * U64 * scale)
    r, rinf = mag.residual(dev(X), 1.7, dev(v))
    assert rinf == float(r.abs().max())


# tol met by x0 (an FP32-accurate solution), by x1, by later corrections (a quarter of
# the cutoff scale), and by none
@pytest.mark.parametrize("scale,tol,outer", [(1.0, 1e-3, 1), (1.0, 1e-12, 2), (0.12, 1e-14, 3), (1.0, 1e-19, None)])
def test_rounds(mag, scale, tol, outer):
    n = 900
    X = W.gaussian(n, 3, seed=3)
    t = scale * W.gaussian_cutoff_estimate(n, 3)
    out = torch.full((n,), 7.0, dtype=torch.float64, device="cuda:0")
    res = mag.weighting(dev(X), t, tol=tol, out=out, raise_on_noconv=False)
    w = res.w.cpu().numpy()
    info = res.info
    if outer is None:
        assert info["status"] == -3
    else:
        assert info["status"] == 0 and info["outer_iters"] >= outer and info["resid_inf"] <= tol
        if outer < 3:
            assert info["outer_iters"] == outer
    # whichever iterate was taken: the reported numbers are those of the returned w
    r, rinf = mag.residual(dev(X), t, res.w)
    assert rinf == info["resid_inf"]
    assert abs(info["magnitude"] - w.sum()) <= 4 * U64 * np.abs(w).sum() * np.log2(n)
    assert info["min_w"] == w.min() and info["argmin_w"] == int(w.argmin())


def test_no_room_for_a_correction(mag):
    X = W.gaussian(500, 3, seed=4)
    t = W.gaussian_cutoff_estimate(500, 3)
    res = mag.weighting(dev(X), t, max_outer=1, raise_on_noconv=False)
    # one residual (of x0) and the step after it, whose result is not looked at
    assert res.info["status"] == -3 and res.info["outer_iters"] == 1 and res.info["gmres_iters"] == 1
    assert 1e-12 < res.info["resid_inf"] < 1e-3
    assert mag.residual(dev(X), t, res.w)[1] == res.info["resid_inf"]


def test_bad_points_leave_the_output_alone(mag):
    X = W.gaussian(700, 3, seed=5)
    for what, code in (("nan", -1), ("inf", -1), ("pair", -2)):
        Y = X.copy()
        if what == "pair":
            Y[600] = Y[3]
        else:
            Y[650, 2] = float(what)
        out = torch.full((700,), 7.0, dtype=torch.float64, device="cuda:0")
        with pytest.raises(mag.MagError) as e:
            mag.weighting(dev(Y), 2.0, out=out)
        assert e.value.code == code
        assert bool((out == 7.0).all())
        # the context solves the good cloud after it
        assert mag.weighting(dev(X), 2.0).info["resid_inf"] <= 1e-12
        with pytest.raises(mag.MagError) as e:
            mag.weighting_and_magnitude(dev(Y), 2.0)
        assert e.value.code == code


def test_breakdown_retried_with_a_shift(mag):
    # Z ~ 1 1^T - t d: the FP32 factor meets a pivot that is not positive
    X = W.gaussian(400, 3, seed=8)
    res = mag.weighting(dev(X), 1e-5, raise_on_noconv=False, max_gmres=400)
    assert res.info["shifted"] == 1 and res.info["shift"] > 0
    w = res.w.cpu().numpy()
    r = np.abs(oracle.residual(X, 1e-5, w)).max()
    assert abs(r - res.info["resid_inf"]) <= 64 * U64 * oracle.zmatvec(X, 1e-5, np.abs(w)).max()


def test_cap_without_room_for_small_tiles(mag):
    n = 1500
    X = W.gaussian(n, 3, seed=6)
    v = np.random.default_rng(6).standard_normal(n)
    npad = mag.padded_size(n)
    ctx = mag.Context(0)
    try:
        base = ctx.workspace_bytes()
        y = mag.zmatvec(dev(X), 1.7, dev(v), ctx=ctx)
        held = ctx.workspace_bytes()
        ctx.close()
        ctx = mag.Context(0)
        # the 64-edged tiles' partial sums take twice those of the 128-edged ones
        T = npad // 128
        least = base + 8 * (T * (T + 1) // 2 * 256 + T + 8 + 64) + 8 * (npad + 256)
        assert least < held
        ctx.set_workspace_limit(least)
        y2 = mag.zmatvec(dev(X), 1.7, dev(v), ctx=ctx)
        assert ctx.workspace_bytes() <= least
        scale = oracle.zmatvec(X, 1.7, np.abs(v))
        assert np.all(np.abs((y - y2).cpu().numpy()) <= 64 * U64 * scale)
    finally:
        ctx.close()
