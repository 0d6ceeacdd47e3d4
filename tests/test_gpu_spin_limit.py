"""A wait that gives up is MAG_EINTERNAL in every call that factors or solves, not a
breakdown of Z: a limit of one poll, set from the host, makes the factor's panels and the
substitutions give up (every kernel still finishes), and the context works again after it."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

EINTERNAL = -6


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def forward(mag, ctx, Xd, t):
    w, h, opts = torch.empty(len(Xd), dtype=torch.float64, device=Xd.device), ctypes.c_void_p(), mag.make_opts()
    rc = ctx.lib.mag_weighting_fwd(ctx.handle, ctypes.c_void_p(Xd.data_ptr()), len(Xd), Xd.shape[1], float(t),
                                   ctypes.c_void_p(w.data_ptr()), ctypes.byref(h), ctypes.byref(opts), None)
    if rc != 0:
        raise mag.MagError(rc, "mag_weighting_fwd")
    ctx.lib.mag_factor_free(h)
    return w


def gives_up(mag, ctx, call):
    """call's result at the default limit; MAG_EINTERNAL at one poll; the same result after."""
    ref = call()
    ctx.set_spin_limit(1)
    with pytest.raises(mag.MagError) as e:
        call()
    assert e.value.code == EINTERNAL
    ctx.set_spin_limit(0)
    return ref, call()


# one, one and a half, and six panels
@pytest.mark.parametrize("n", [129, 700, 3000])
def test_single(mag, n):
    Xd, t = dev(W.gaussian(n, 3, seed=n)), W.gaussian_cutoff_estimate(n, 3)
    ctx = mag.Context(0)
    try:
        calls = {
            "factor32": lambda: mag.factor32(Xd, t, ctx=ctx)[0],
            "weighting": lambda: mag.weighting(Xd, t, ctx=ctx).w,
            "forward": lambda: forward(mag, ctx, Xd, t),
            "dwdt": lambda: mag.dwdt(Xd, t, ctx=ctx)[1],
            "zero": lambda: mag.weighting_zero(Xd, ctx=ctx).w,
            "tplus": lambda: mag.tplus(Xd, ctx=ctx).w,
        }
        for name, call in calls.items():
            print(name, flush=True)
            a, b = gives_up(mag, ctx, call)
            assert torch.equal(a, b)
        for call in (lambda: mag.eig_extremes(Xd, t, ctx=ctx, max_iter=4), lambda: mag.autotune(Xd, t, ctx=ctx)):
            gives_up(mag, ctx, call)
    finally:
        ctx.close()


# both groupings: 512-column panels with their exchange, and 128 columns at a time, where only
# the substitutions wait
@pytest.mark.parametrize("group", [1, 2])
def test_batched(mag, group):
    sizes = (129, 300, 1100)
    Xp, offs = W.pack_clouds([W.gaussian(n, 3, seed=n) for n in sizes])
    Xd, ts = dev(Xp), [W.gaussian_cutoff_estimate(n, 3) for n in sizes]
    ctx = mag.Context(0)
    try:
        mag.tune_batch_group(max(sizes), group, ctx=ctx)
        a, b = gives_up(mag, ctx, lambda: mag.weighting_batch(Xd, offs, ts, ctx=ctx)[0])
        assert torch.equal(a, b)
        a, b = gives_up(mag, ctx, lambda: mag.tplus_batch(Xd, offs, want_w=True, ctx=ctx)[1])
        assert torch.equal(a, b)
        gives_up(mag, ctx, lambda: mag.autotune_batch(Xd, offs, ts, ctx=ctx))
    finally:
        ctx.close()
