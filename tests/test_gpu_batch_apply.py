"""The batched preconditioner apply multiplies by nothing but the FP32 factor and its
diagonal blocks' inverses, in FP64: the first iterate L^{-T} L^{-1} 1 of a batch (all that a
loose tolerance asks for) against the same substitutions in numpy, to FP64 rounding."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def apply(L, D, r):
    """L^{-T} L^{-1} r by blocks of 128, x_b = D_b (r_b - sum T(b, j) x_j), and the largest
    magnitude that its sums run through."""
    nb, big = len(D), 0.0
    y, z = np.zeros_like(r), np.zeros_like(r)
    for b in range(nb):
        s = slice(128 * b, 128 * b + 128)
        y[s] = D[b] @ (r[s] - L[s, :128 * b] @ y[:128 * b])
        big = max(big, (np.abs(D[b]) @ (np.abs(r[s]) + np.abs(L[s, :128 * b]) @ np.abs(y[:128 * b]))).max())
    for b in reversed(range(nb)):
        s = slice(128 * b, 128 * b + 128)
        e = 128 * b + 128
        z[s] = D[b].T @ (y[s] - L[e:, s].T @ z[e:])
        big = max(big, (np.abs(D[b].T) @ (np.abs(y[s]) + np.abs(L[e:, s].T) @ np.abs(z[e:]))).max())
    return z, big


# up to one panel of 512 columns, whose factor in a batch is that of a single solve
def test_first_iterate(mag):
    sizes = (1, 128, 129, 256, 257, 384, 385, 500, 512)
    clouds = [W.gaussian_mixture(n, 3, seed=n) for n in sizes]
    Xp, offs = W.pack_clouds(clouds)
    ts = [W.gaussian_cutoff_estimate(max(2, n / 5), 3) / 0.1 for n in sizes]
    w, _, info = mag.weighting_batch(dev(Xp), offs, ts, tol=1e-2)
    w = w.cpu().numpy()
    for b, (X, t) in enumerate(zip(clouds, ts)):
        assert info[b]["outer_iters"] == 1
        L, dinv, bd = mag.factor32(dev(X), t)
        assert bd == 0
        n, npad = len(X), L.shape[0]
        r = np.zeros(npad)
        r[:n] = 1.0
        D = [d.T.astype(np.float64) for d in dinv.cpu().numpy()]
        z, big = apply(np.tril(L.cpu().numpy().T).astype(np.float64), D, r)
        # each of the npad / 128 blocks a direction adds two sums of at most npad + 1 roundings, carried
        # on by the later ones no further than the sums' own magnitudes
        err, bound = np.abs(w[offs[b]:offs[b + 1]] - z[:n]).max(), 4 * (npad // 128) * (npad + 1) * U64 * big
        print(f"n={n}: error {err:.2e}, bound {bound:.2e}")
        assert err <= bound
