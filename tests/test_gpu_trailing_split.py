"""The FP32 factor's trailing update on three-component BF16 splits: the factor
against FP64 at the edges of its tiles, and a context whose cap leaves no room
for the split image (the update then runs on the FP32 matrix instruction)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def backward_error(mag, X, t, ctx):
    n = len(X)
    L, _, bd = mag.factor32(dev(X), t, ctx=ctx)
    assert bd == 0
    Lf = torch.tril(L.T).double()
    Z = torch.eye(Lf.shape[0], dtype=torch.float64, device="cuda:0")
    Z[:n, :n] = dev(oracle.zmatrix(X, t))
    E = Lf @ Lf.T - Z
    return float(E.norm() / Z.norm()), float(E.abs().max())


# trailing rows 256, 512, 768 (one and two super-tiles, the odd
# half), 4864, 5120 and 5632 (ten and eleven); panels of
# 512 (K = 1024) and 256 columns (K = 512)
@pytest.mark.parametrize("n,nb", [(1280, 512), (1281, 512), (1790, 512), (5888, 512), (6144, 512), (6500, 512),
                                  (700, 256), (2049, 256)])
def test_factor_with_split_update(mag, n, nb):
    X = W.gaussian(n, 3, seed=n)
    t = W.gaussian_cutoff_estimate(n, 3) / 2
    ctx = mag.Context(0)
    try:
        mag.tune_panel(n, nb, ctx=ctx)
        rel, worst = backward_error(mag, X, t, ctx)
    finally:
        ctx.close()
    npad = mag.padded_size(n)
    print(f"n={n} nb={nb}: backward error {rel:.3e}, largest entry {worst:.3e}")
    # |E| <= gamma_{npad + 1} |L| |L^T| entrywise, (|L| |L^T|)_ij <= 1 (Z has a unit diagonal)
    assert rel <= 4 * npad * U32 and worst <= (npad + 1) * U32


def test_cap_without_room_for_the_image(mag):
    n = 3000
    X = W.gaussian(n, 3, seed=5)
    Xd, t = dev(X), W.gaussian_cutoff_estimate(n, 3)
    npad = mag.padded_size(n)
    image = (npad - 1024) * 6 * 1024  # three 2-byte components of 1024 columns
    ctx = mag.Context(0)
    try:
        w = mag.weighting(Xd, t, ctx=ctx).w.cpu().numpy()
        held = ctx.workspace_bytes()
        ctx.close()
        ctx = mag.Context(0)
        ctx.set_workspace_limit(held - image)  # everything but the image
        res = mag.weighting(Xd, t, ctx=ctx)
        assert ctx.workspace_bytes() <= held - image
        wc = res.w.cpu().numpy()
        assert res.info["resid_inf"] <= 1e-12 and np.abs(wc - w).max() <= 1e-10 * np.abs(w).max()
        # an image that is held makes way for a buffer a call cannot do without
        ctx.set_workspace_limit(held)
        mag.weighting(Xd, t, ctx=ctx)
        assert ctx.workspace_bytes() <= held
        need = 8 * npad * 4
        ctx.set_workspace_limit(held - image + need + 4096)
        _, d = mag.dwdt(Xd, t, ctx=ctx)
        assert ctx.workspace_bytes() <= held - image + need + 4096
        assert torch.isfinite(d).all()
    finally:
        ctx.close()


# clouds whose trailing updates fall on the 128-row tiles (few) and on the 256-row
# ones (many), in both groupings, beside clouds with no trailing update at all
@pytest.mark.parametrize("group", [1, 2])
@pytest.mark.parametrize("sizes", [(200, 300, 513, 1025), (3000,) * 6 + (257, 767, 2049)])
def test_batched_split_update(mag, sizes, group):
    clouds = [W.gaussian(n, 3, seed=n + b) for b, n in enumerate(sizes)]
    X, offs = W.pack_clouds(clouds)
    ts = [W.gaussian_cutoff_estimate(n, 3) for n in sizes]
    ctx = mag.Context(0)
    try:
        mag.tune_batch_group(max(sizes), group, ctx=ctx)
        w, _, infos = mag.weighting_batch(dev(X), offs, ts, ctx=ctx)
        w = w.cpu().numpy()
        held = ctx.workspace_bytes()
        for b, (Xb, t) in enumerate(zip(clouds, ts)):
            assert infos[b]["status"] == 0
            assert np.abs(oracle.residual(Xb, t, w[offs[b]:offs[b + 1]])).max() <= 1e-12
        # the same without room for the images: the FP32 updates
        ctx.close()
        ctx = mag.Context(0)
        mag.tune_batch_group(max(sizes), group, ctx=ctx)
        ctx.set_workspace_limit(held - 1)
        wc, _, infos = mag.weighting_batch(dev(X), offs, ts, ctx=ctx)
        assert ctx.workspace_bytes() < held and all(i["status"] == 0 for i in infos)
        assert np.abs(wc.cpu().numpy() - w).max() <= 1e-10 * np.abs(w).max()
    finally:
        ctx.close()
