"""What a batch holds for the panel launches' exchanges: no more than the factors they
serve, nothing where the grouping has no such launch; and clouds of every panel count in
one batch, whose exchanges differ in size."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def held_and_weights(mag, sizes, group):
    Xp, offs = W.pack_clouds([W.gaussian(n, 3, seed=n + b) for b, n in enumerate(sizes)])
    ts = [W.gaussian_cutoff_estimate(max(n, 2), 3) for n in sizes]
    ctx = mag.Context(0)
    try:
        mag.tune_batch_group(max(sizes), group, ctx=ctx)
        w = [mag.weighting_batch(dev(Xp), offs, ts, ctx=ctx)[0].cpu().numpy() for _ in range(2)]
        assert np.array_equal(w[0], w[1])
        for b, t in enumerate(ts):
            X = Xp[offs[b]:offs[b + 1]]
            assert np.abs(oracle.residual(X, t, w[0][offs[b]:offs[b + 1]])).max() <= 1.1e-12
        return ctx.workspace_bytes()
    finally:
        ctx.close()


@pytest.mark.parametrize("sizes", [(200,) * 40, (256, 257, 512, 513, 768, 769, 1024, 1025, 1100, 1537) * 2, (1,)])
def test_exchanges(mag, sizes):
    single, pairs = held_and_weights(mag, sizes, 1), held_and_weights(mag, sizes, 2)
    factors = sum(4 * mag.padded_size(n) ** 2 for n in sizes)
    print(f"{len(sizes)} clouds: {pairs / 1e6:.2f} MB, {single / 1e6:.2f} MB without exchanges, factors {factors / 1e6:.2f} MB")
    assert single < pairs <= single + factors
