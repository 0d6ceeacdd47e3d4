"""The gradients in the points and the scale from one pass over the pairs, at the edges
of its row blocks and in every compiled dimension, against the passes of their own."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n,m", [(1, 3), (2, 1), (255, 2), (256, 3), (257, 4), (700, 8), (513, 5), (300, 16), (300, 17)])
def test_both_gradients_match_their_own_passes(mag, n, m):
    X = W.gaussian(n, m, seed=n)
    t = 0.8 * W.gaussian_cutoff_estimate(max(n, 2), m)
    gw = dev(np.random.default_rng(n).standard_normal(n))
    out = []
    for need_t in (True, False):
        Xd = dev(X).requires_grad_(True)
        td = torch.tensor(t, dtype=torch.float64, device="cuda:0", requires_grad=need_t)
        w, M = mag.weighting_and_magnitude(Xd, td)
        g = torch.autograd.grad((w, M), (Xd, td) if need_t else (Xd,), (gw, torch.ones_like(M)))
        out.append((w.detach().cpu().numpy(), [x.cpu().numpy() for x in g]))
    assert np.array_equal(out[0][1][0], out[1][1][0])
    dt_ref, dX_ref, sol = oracle.grad(X, t, gM=1.0, gw=gw.cpu().numpy())
    # as for the other gradients: 1e-10, or what kappa_M leaves of two FP64 evaluations
    tol = 1e-10 + 8 * 2.0 ** -53 * oracle.kappa_M(sol)
    assert abs(out[0][1][1] - dt_ref) <= tol * max(abs(dt_ref), np.abs(dX_ref).max())
    assert np.abs(out[0][1][0] - dX_ref).max() <= tol * max(np.abs(dX_ref).max(), 1e-300)
