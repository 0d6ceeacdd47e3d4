"""The FP32 factor's panel kernel (one launch per 256 or 512 columns, steps handed
between workgroups) at the edges of its sub-panels, panels and padding, in both
widths, and two contexts' factors at once on their own streams."""
import threading

import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def check(mag, X, t, ctx):
    n = len(X)
    L, dinv, bd = mag.factor32(dev(X), t, ctx=ctx)
    assert bd == 0
    Lc = L.cpu().numpy().T
    npad = Lc.shape[0]
    Lf = np.tril(Lc).astype(np.float64)
    assert np.array_equal(np.triu(Lc, 1), np.tril(Lc, -1).T)
    Z = np.eye(npad)
    Z[:n, :n] = oracle.zmatrix(X, t)
    # |E| <= gamma_{npad + 1} |L| |L^T| with (|L| |L^T|)_ij <= 1, doubled for the products
    # with the inverses of 16-column blocks
    assert np.abs(Lf @ Lf.T - Z).max() <= 2 * (npad + 1) * U32
    assert np.array_equal(Lf[n:, n:], np.eye(npad - n)) and not Lf[n:, :n].any()
    D = dinv.cpu().numpy()
    for b in range(npad // 128):
        blk = Lf[128 * b:128 * (b + 1), 128 * b:128 * (b + 1)]
        Db = D[b].T.astype(np.float64)
        assert np.all(np.abs(Db @ blk - np.eye(128)) <= 2 * 129 * U32 * (np.abs(Db) @ np.abs(blk)) + 1e-30)
    return Lc


@pytest.mark.parametrize("nb", [256, 512])
@pytest.mark.parametrize("n", [256, 511, 512, 513, 640, 769, 1025, 1281])
def test_panels(mag, n, nb):
    ctx = mag.Context(0)
    mag.tune_panel(n, nb, ctx=ctx)
    X = W.gaussian(n, 3, seed=n)
    first = check(mag, X, 1.5, ctx)
    assert np.array_equal(first, check(mag, X, 1.5, ctx))  # the exchange is left ready for the next factor
    ctx.close()


def test_two_contexts_at_once(mag):
    X = W.gaussian(3000, 3, seed=5)
    ctxs = [mag.Context(0) for _ in range(2)]
    w = [None, None]

    def solve(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                w[i] = mag.weighting(dev(X), 3.0, ctx=ctxs[i]).w.cpu().numpy()

    threads = [threading.Thread(target=solve, args=(i,)) for i in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert np.array_equal(w[0], w[1])
    assert np.abs(oracle.residual(X, 3.0, w[0])).max() <= 1e-12
    for c in ctxs:
        c.close()
