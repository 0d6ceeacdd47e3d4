"""Batched factors with each part of the optional scratch: the split image (BF16 updates)
and the panel launches' exchanges, one without the other, and neither (FP32 updates,
128 columns at a time), in both groupings.  The cap is set so that only the rest fits, and
what is held afterwards says which path ran."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

# no trailing update, one of a tile, several; odd and even panel counts
SIZES = (257, 512, 767, 1100, 1537, 2049, 3000, 3000, 3000)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def image_bytes(npad):
    def img(rows, K):
        return -(-max(rows, 0) // 256) * 256 * (K // 8) * 3 * 16
    return max(img(npad - 512, 512), img(npad - 256, 256))


def exchange_bytes(npad):
    def bank(cols):
        return (cols // 16) * (cols // 16 + 1) // 2 * 1536
    return 256 + bank(min(npad, 512)) + bank(min(max(npad - 512, 0), 512))


def test_without_optional_scratch(mag):
    clouds = [W.gaussian(n, 3, seed=n + b) for b, n in enumerate(SIZES)]
    Xp, offs = W.pack_clouds(clouds)
    ts = [W.gaussian_cutoff_estimate(n, 3) for n in SIZES]
    img, exch = (sum(f(mag.padded_size(n)) for n in SIZES) for f in (image_bytes, exchange_bytes))
    assert exch < img
    Xd = dev(Xp)

    def run(group, limit):
        ctx = mag.Context(0)
        try:
            mag.tune_batch_group(max(SIZES), group, ctx=ctx)
            ctx.set_workspace_limit(limit)
            w, _, infos = mag.weighting_batch(Xd, offs, ts, ctx=ctx)
            w = w.cpu().numpy()
            for b, (X, t) in enumerate(zip(clouds, ts)):
                assert infos[b]["status"] == 0
                assert np.abs(oracle.residual(X, t, w[offs[b]:offs[b + 1]])).max() <= 1.1e-12
            tp = mag.tplus_batch(Xd, offs, ctx=ctx)[0]
            return ctx.workspace_bytes(), w, [i["outer_iters"] for i in infos], tp
        finally:
            ctx.close()

    for group in (1, 2):
        held, w, iters, tp = run(group, 0)
        rest = held - img - (exch if group == 2 else 0)
        # (cap, what is then held): the image does not fit, the exchanges do; neither does;
        # the image does, the exchanges, which come last, do not
        caps = [(held - 1, rest)] if group == 1 else [(rest + img - 1, rest + exch), (rest + exch - 1, rest),
                                                      (held - 1, rest + img)]
        for cap, left in caps:
            print(f"group {group}: cap {cap}, expected {left}", flush=True)
            got, wc, itc, tpc = run(group, cap)
            assert got == left
            # a factor as good as with them: as many corrections, the same answer
            assert itc == iters
            assert np.abs(wc - w).max() <= 1e-10 * np.abs(w).max()
            assert np.allclose(tpc, tp, rtol=3e-6, atol=0)
