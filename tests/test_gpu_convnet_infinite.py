"""The preconditioner network with infinite weights: the kernels' exact splits into BF16 parts and
their zero operands must not turn an infinite sum into NaN.  Values are compared by kind only
(+inf, -inf, NaN, finite) with sums in FP64, so there is no tolerance."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = ((8, 1), (8, 8), (1, 8))  # outputs, inputs of a layer


def _layers(rng):
    """(w, b) of each layer: positive multiples of 1/4, which are BF16 values."""
    out = []
    for co, ci in SIZES:
        w = rng.integers(1, 5, size=(co, ci, 27)) * 0.25
        out.append([w, np.full(co, 0.25)])
    return out


def _net(layers):
    import paper_2405_01522_amd as ace
    return ace.ConvNet(np.concatenate([np.concatenate([w.reshape(-1), b])
                                       for w, b in layers]).astype(np.float32))


def _shift(a, t):
    d = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
    n = a.shape[-1]
    out = np.zeros_like(a)
    src = tuple(slice(max(0, k), n + min(0, k)) for k in d)
    dst = tuple(slice(max(0, -k), n - max(0, k)) for k in d)
    out[(Ellipsis,) + dst] = a[(Ellipsis,) + src]
    return out


def _forward(layers, x):
    """Activations before and after each layer, sums product by product."""
    acts = [x[None]]
    for li, (w, b) in enumerate(layers):
        y = np.broadcast_to(b[:, None, None, None], (len(b),) + x.shape).copy()
        for t in range(27):
            s = _shift(acts[-1], t)
            for i in range(w.shape[1]):
                y += w[:, i, t][:, None, None, None] * s[i]
        acts.append(np.fmax(y, 0.0) if li < 2 else y)
    return acts


def _kind(a):
    return np.where(np.isnan(a), 2, np.where(np.isinf(a), np.sign(a), 0))


@pytest.mark.parametrize("n", [9, 17])
@pytest.mark.parametrize("layer,tap,value", [(2, 13, np.inf), (2, 13, -np.inf), (2, 0, np.inf),
                                             (2, 26, np.inf), (1, 13, np.inf), (1, 4, np.inf)])
def test_infinite_weight(n, layer, tap, value):
    """Inputs are small integers, so the activations fit in 16 bits and have parts that are zero."""
    rng = np.random.default_rng(n + tap)
    layers = _layers(rng)
    layers[layer][0][0, 3, tap] = value
    x = rng.integers(1, 4, size=(2, n, n, n)).astype(np.float32)
    net = _net(layers)
    y = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    with np.errstate(all="ignore"):
        for k in range(2):
            ref = _forward(layers, x[k].astype(np.float64))[-1][0]
            assert np.array_equal(_kind(y[k]), _kind(ref)), np.unique(_kind(y[k]))
    # the loss form of the last layer: an infinite output makes the loss infinite, not NaN
    if (layer, tap) == (2, 13):
        loss, _ = net.gradient(torch.from_numpy(x).cuda(), torch.zeros((2, n, n, n), device="cuda"))
        assert loss == np.inf


def _gradient(layers, acts, t):
    """Gradient of each layer's (w, b), each sum product by product over the output's points, with
    zeros for inputs outside the box."""
    g = ((acts[-1][0] - t) / t.size)[None]
    grads = []
    for li in (2, 1, 0):
        w = layers[li][0]
        if li < 2:
            g = np.where(acts[li + 1] > 0, g, 0.0)
        gw = np.empty_like(w)
        ga = np.zeros_like(acts[li])
        for q in range(27):
            s = _shift(acts[li], q)
            for o in range(w.shape[0]):
                for i in range(w.shape[1]):
                    gw[o, i, q] = np.sum(g[o] * s[i])
            gs = _shift(g, 26 - q)
            for i in range(w.shape[1]):
                for o in range(w.shape[0]):
                    ga[i] += w[o, i, q] * gs[o]
        grads = [gw.reshape(-1), g.sum(axis=(1, 2, 3))] + grads
        g = ga
    return np.concatenate(grads)


@pytest.mark.parametrize("where", ["inside", "tile edge", "face", "corner"])
def test_gradient_of_an_infinite_input(where):
    """An infinite input reaches the activations of three points around it, across tile edges (y = 8)
    and on faces of the box."""
    n = 16
    c = {"inside": (6, 5, 8), "tile edge": (7, 8, 7), "face": (0, 7, 8), "corner": (15, 0, 15)}[where]
    rng = np.random.default_rng(1)
    layers = _layers(rng)
    x = rng.integers(1, 4, size=(1, n, n, n)).astype(np.float32)
    x[0][c] = np.inf
    t = rng.normal(size=(1, n, n, n)).astype(np.float32)
    loss, grad = _net(layers).gradient(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    assert loss == np.inf
    with np.errstate(all="ignore"):
        acts = _forward(layers, x[0].astype(np.float64))
        ref = _gradient(layers, acts, t[0].astype(np.float64))
    assert np.array_equal(_kind(grad), _kind(ref)), np.nonzero(_kind(grad) != _kind(ref))


@pytest.mark.parametrize("c", [(5, 7, 8), (0, 7, 8), (15, 15, 0)])
def test_gradient_of_an_infinite_target(c):
    n = 16
    rng = np.random.default_rng(2)
    layers = _layers(rng)
    x = rng.integers(1, 4, size=(1, n, n, n)).astype(np.float32)
    t = rng.normal(size=(1, n, n, n)).astype(np.float32)
    t[0][c] = np.inf
    loss, grad = _net(layers).gradient(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    assert loss == np.inf
    with np.errstate(all="ignore"):
        acts = _forward(layers, x[0].astype(np.float64))
        ref = _gradient(layers, acts, t[0].astype(np.float64))
    assert np.array_equal(_kind(grad), _kind(ref)), np.nonzero(_kind(grad) != _kind(ref))
