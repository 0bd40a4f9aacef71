"""The preconditioner network at box edges around its kernels' tiles (4 x 8 x 16 and 8 x 8 x 16
points, lines of 16 x 16), against the FP64 oracle, and with an infinite input value.

Bars: a layer is a sum of at most 216 products, FP32 in any order: a few times
sqrt(216) 2^-24 ~ 1e-6 of its largest value, three layers deep; 5e-6 for the outputs.  A gradient
entry sums the same errors over the points, and an activation within rounding of zero may fall
on either side of the ReLU: 1e-4 of the largest entry.
"""

import numpy as np
import pytest
import torch

from oracle import convnet

pytestmark = pytest.mark.gpu


def _net(seed, positive=False):
    import paper_2405_01522_amd as ace
    rng = np.random.default_rng(seed)
    vec = convnet.flatten(convnet.init_params(rng, scale=1.0))
    vec = torch.from_numpy(np.abs(vec) + 0.01 if positive else vec).to(torch.bfloat16)
    return ace.ConvNet(vec.float().numpy()), convnet.unflatten(vec.double().numpy())


@pytest.mark.parametrize("n,nb", [(1, 1), (3, 2), (4, 1), (8, 3), (15, 1), (16, 2), (17, 3), (33, 2)])
def test_edges(n, nb):
    net, params = _net(10 * n + nb)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(nb, n, n, n)).astype(np.float32)
    t = rng.normal(size=(nb, n, n, n)).astype(np.float32)
    y = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    loss, grad = net.gradient(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    lref, gref = 0.0, 0.0
    for b in range(nb):
        yr, cache = convnet.forward(params, x[b].astype(np.float64))
        assert np.max(np.abs(y[b] - yr)) < 5e-6 * np.max(np.abs(yr)), (n, b)
        lref += convnet.loss(yr, t[b].astype(np.float64)) / nb
        gref = gref + convnet.flatten(convnet.backward(params, cache, yr, t[b].astype(np.float64))) / nb
    assert abs(loss - lref) < 1e-5 * lref
    assert np.max(np.abs(grad - gref)) < 1e-4 * np.max(np.abs(gref))


@pytest.mark.parametrize("n", [9, 33])
def test_infinity_reaches_its_neighbours_only(n):
    """With positive weights an infinite value makes the outputs within three points infinite and
    leaves every other one as it is."""
    net, params = _net(5, positive=True)
    rng = np.random.default_rng(3)
    x = np.abs(rng.normal(size=(1, n, n, n))).astype(np.float32)
    yr, _ = convnet.forward(params, x[0].astype(np.float64))
    c = (n // 2, n // 3, n // 2 + 1)
    x[0][c] = np.inf
    y = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()[0]
    near = np.ones_like(y, dtype=bool)
    for ax in range(3):
        d = np.abs(np.arange(n) - c[ax]) <= 3
        near &= d.reshape([-1 if k == ax else 1 for k in range(3)])
    assert np.all(np.isposinf(y[near]))
    assert np.max(np.abs(y[~near] - yr[~near])) < 5e-6 * np.max(np.abs(yr))
