"""A solve whose first iterate meets tol pays for one application and one product, not
for the step enqueued after it: the refinement's time at the default limits against that
with max_outer = 1, which leaves no room for the step (it is twice that if the step runs)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


# the product on its symmetric tiles and, above 16 dimensions, by rows; x0 of an FP32
# factor meets 1e-4, that of a compressed one half of the right-hand side
@pytest.mark.parametrize("solver,n,m,tol", [("fp32_ir", 16384, 3, 1e-4), ("fp32_ir", 8192, 20, 1e-4),
                                            ("hodlr", 16384, 3, 0.5), ("hss", 16384, 3, 0.5)])
def test_refinement_time(mag, solver, n, m, tol):
    Xd, t = dev(W.gaussian(n, m, seed=1)), W.gaussian_cutoff_estimate(n, m)
    ctx = mag.Context(0)
    try:
        def solve(**kw):
            res = mag.weighting(Xd, t, solver=solver, tol=tol, profile=True, ctx=ctx, **kw)
            assert res.info["outer_iters"] == 1 and res.info["resid_inf"] <= tol
            return res
        ms, w = {}, {}
        for k in (1, 10):
            solve(max_outer=k)
            runs = [solve(max_outer=k) for _ in range(5)]
            ms[k], w[k] = min(r.info["ms_refine"] for r in runs), runs[0].w
        print(f"{solver} n={n} m={m}: {ms[10]:.3f} ms, {ms[1]:.3f} ms without room for a step")
        assert ms[10] <= 1.4 * ms[1]
        assert torch.equal(w[1], w[10])
    finally:
        ctx.close()


# both sides of the gate on one context: the step's vectors and tickets are left as they were
def test_gate_leaves_the_context_ready(mag):
    for n in (100, 129, 900, 3000):
        Xd, t = dev(W.gaussian(n, 3, seed=n)), W.gaussian_cutoff_estimate(n, 3)
        ctx = mag.Context(0)
        try:
            ref = mag.weighting(Xd, t, ctx=ctx).w
            for _ in range(2):
                loose = mag.weighting(Xd, t, tol=1e-3, ctx=ctx)
                assert loose.info["outer_iters"] == 1
                r, rinf = mag.residual(Xd, t, loose.w)
                assert rinf == loose.info["resid_inf"]
                assert loose.info["min_w"] == float(loose.w.min())
                assert torch.equal(mag.weighting(Xd, t, ctx=ctx).w, ref)
        finally:
            ctx.close()
