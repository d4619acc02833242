"""Predictor kernels at the edges of their 16-row tiles and block counts, with
operands off the vector alignments."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp as ref
from tests.test_gpu_mlp import _data, _dev, _params, _relerr, resoct, torch

pytestmark = pytest.mark.gpu

# FP16 operands (2^-11 relative each, as in the tests of the whole network)
TOL = 1e-2


def _half(a):
    return np.asarray(a, np.float16).astype(np.float64)


def _network(p, x, y, m):
    """Logits, gradients and loss in FP64 with the products' operands rounded
    to FP16, as they are defined: with few rows, a hidden unit within a
    rounding of zero makes 2 % of the unrounded gradients."""
    W1, W2, W3 = _half(p["W1"]), _half(p["W2"]), _half(p["W3"])
    b1, b2, b3 = (p[k].astype(np.float64) for k in ("b1", "b2", "b3"))
    a1 = x @ W1 + b1
    h1 = _half(np.maximum(a1, 0.0))
    a2 = h1 @ W2 + b2
    h2 = _half(np.maximum(a2, 0.0))
    z = h2 @ W3 + b3
    n = max(m.sum(), 1.0)
    dz = m * (ref.sigmoid(z) - y)
    d2 = (_half(dz) @ W3.T) * (a2 > 0)
    d1 = (_half(d2) @ W2.T) * (a1 > 0)
    g = dict(W3=h2.T @ _half(dz), b3=dz.sum(0), W2=h1.T @ _half(d2), b2=d2.sum(0), W1=x.T @ _half(d1), b1=d1.sum(0))
    return z, {k: v / n for k, v in g.items()}, ref.loss(z, y, m)


def _off(a, by):
    """The array on the device, `by` elements past a 256-byte boundary."""
    t = _dev(a)
    buf = torch.zeros(t.numel() + by, dtype=t.dtype, device="cuda")
    buf[by:].copy_(t.reshape(-1))
    return buf[by:].view(t.shape)


# one tile and its neighbours, a block and one more tile, more tiles than the
# blocks of a launch have waves
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 64, 65, 16 * 4 * 256 + 1, 16 * 4 * 512 + 17])
@pytest.mark.parametrize("by", [0, 1])
def test_tiles(rows, by):
    x, y, m = _data(rows, rows)
    p = _params(3)
    net = resoct.Mlp()
    net.set_weights(p)
    z = _off(np.full((rows, 16), 7.0, np.float32), by)
    X, Y, M = _off(x, by), _off(y, by), _off(m, by)
    net.forward(X, z)
    zr, gr, want = _network(p, x[:, :24].astype(np.float64), y[:, :9].astype(np.float64), m[:, :9].astype(np.float64))
    got = z.cpu().numpy()
    assert np.abs(got[:, :9] - zr).max() <= TOL * max(np.abs(zr).max(), 1e-6)
    assert np.all(got[:, 9:] == 0.0)
    g, loss = net.gradients(X, Y, M)
    assert abs(loss - want) <= 1e-3 * abs(want)
    for k in gr:
        assert _relerr(g[k], gr[k]) <= TOL, k
    assert net.train_step(X, Y, M, 1e-3, want_loss=True) == loss


def test_rows_do_not_mix():
    """Infinite inputs of one row leave the other rows of its tile as they were."""
    x, _, _ = _data(8, 48)
    net = resoct.Mlp()
    net.set_weights(_params(9))
    a = net.forward(_dev(x)).cpu().numpy()
    x[19, 3] = np.inf
    b = net.forward(_dev(x)).cpu().numpy()
    rest = np.arange(48) != 19
    assert np.array_equal(a[rest], b[rest])
