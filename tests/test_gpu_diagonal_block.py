"""The 128 x 128 diagonal block of the FP32 factor (16-column steps, blocks in
registers): L, its transpose and the inverse at the edges of the 16-column
blocks and of the identity padding, and the pivot index of a breakdown."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 127, 128, 129, 144, 255, 257, 385])
def test_diagonal_blocks(mag, n):
    X = W.gaussian(n, 3, seed=n)
    t = 2.0
    L, dinv, bd = mag.factor32(dev(X), t)
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
        assert not np.triu(Db, 1).any()
        # forward error of the computed inverse: |D L - I| <= gamma_128 |D| |L| and as much
        # again from the 16-column steps
        assert np.all(np.abs(Db @ blk - np.eye(128)) <= 2 * 129 * U32 * (np.abs(Db) @ np.abs(blk)) + 1e-30)


@pytest.mark.parametrize("k", [1, 5, 16, 100, 130, 300])
def test_breakdown_reports_the_first_pivot(mag, k):
    # points k - 1 and k coincide: Z is exactly singular, and its leading k x k block
    # is not, so with a far-apart cloud (Z close to I) the pivot of row k is exactly 0
    X = np.arange(400, dtype=np.float64)[:, None] * 100.0
    X[k] = X[k - 1]
    _, _, bd = mag.factor32(dev(X), 1.0)
    assert bd == k + 1
