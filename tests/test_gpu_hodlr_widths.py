"""HODLR bases of every width class (one slab of 64 columns, the three-launch node
corrections from two on, the 512-column sampling), at ragged sizes: the solve and the
rate of its inner iteration."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rank", [(1500, 40), (1500, 64), (2001, 100), (3001, 180), (4099, 256), (4099, 500), (9001, 512)])
def test_widths(mag, n, rank):
    X = W.gaussian(n, 3, seed=n)
    t = W.gaussian_cutoff_estimate(n, 3)
    Xd = torch.from_numpy(X).to("cuda:0")
    res = mag.weighting(Xd, t, solver="hodlr", max_rank=rank, power_iters=1)
    w = res.w.cpu().numpy()
    print(f"n={n} rank={rank}: {res.info['outer_iters']} outer, {res.info['gmres_iters']} inner")
    assert np.abs(oracle.residual(X, t, w)).max() <= 1.1e-12
    again = mag.weighting(Xd, t, solver="hodlr", max_rank=rank, power_iters=1)
    assert np.array_equal(w, again.w.cpu().numpy())
    # a wider basis is a preconditioner at least about as good
    wide = mag.weighting(Xd, t, solver="hodlr", max_rank=min(512, 2 * rank), power_iters=1)
    assert wide.info["gmres_iters"] <= res.info["gmres_iters"] + 2
