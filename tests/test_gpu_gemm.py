"""FP32 matrix kernels of the network's training at the edges of their tiles
(32 and 64, K stages of 64 and 32) and on both sides of the tile rule, against
a plain FP64 forward and backward."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1, 1), (31, 33, 64, 32), (64, 32, 65, 31), (63, 65, 2049, 64),
                                  (129, 64, 4608, 512), (65, 128, 4609, 513)])
def test_gradient_tiles(dims):
    import torch
    import paper_2103_10203_amd as mor
    i, h, o, B = dims
    net = mor.MLP(i, h, o, seed=11)
    rng = np.random.default_rng(i + h)
    X = rng.normal(size=(B, i)).astype(np.float32)
    T = rng.normal(size=(B, o)).astype(np.float32)
    loss = net.grad(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
    P = [p.astype(np.float64) for p in net.split(net.params())]
    y, cache = omlp.forward(P, X.astype(np.float64))
    want = omlp.backward(P, cache, y, T.astype(np.float64))
    assert abs(loss - omlp.mse(y, T)) < 1e-5 * abs(omlp.mse(y, T))
    # chains of up to 4609 FP32 products: 4609 * 2^-24 = 3e-4 of the sum of
    # magnitudes at worst, its root in practice
    for g, w in zip(net.split(net.grads()), want):
        assert np.max(np.abs(g - w)) <= 1e-4 * np.max(np.abs(w)) + 1e-12
