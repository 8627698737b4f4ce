"""The network's many-row kernels at the edges of their 16-row groups and of
their grid (256 workgroups of 16 rows) against the FP64 oracle."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

# float32 products of inner length up to 64 and sums over the rows: each value
# carries at most about (64 + 64 + 16) roundings of 2^-24 of its terms
TOL = 144 * 2.0 ** -24


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 65, 4096, 4101, 9001])
def test_gradient_loss_and_scores(qs_lib, rows):
    params = omlp.init_params(3)
    g = np.random.default_rng(rows)
    X = g.uniform(-1.0, 1.0, (rows, 32)).astype(np.float32).astype(np.float64)
    y = (g.random(rows) < 0.3).astype(float)
    w = omlp.flatten(params).astype(np.float32).astype(np.float64)
    params = omlp.unflatten(w)
    net = qs_lib.MLP(w)
    grad, loss = net.grad(X, y)
    want = omlp.flatten(omlp.backward(params, X, y))
    # the sum of absolute terms bounds what the roundings act on
    assert np.linalg.norm(grad - want) <= 4 * TOL * max(np.linalg.norm(want), 1.0 / np.sqrt(rows))
    assert abs(loss - omlp.loss(params, X, y)) <= TOL
    np.testing.assert_allclose(net.forward(X), omlp.forward(params, X)["score"], atol=TOL)
    net.free()


@pytest.mark.parametrize("rows,batch", [(40, 7), (300, 300), (5000, 4500)])
def test_one_adam_step(qs_lib, rows, batch):
    """After one step every parameter has moved by lr g / (|g| + eps): compared
    where the gradient is far above its rounding."""
    g = np.random.default_rng(batch)
    X = g.uniform(-1.0, 1.0, (rows, 32)).astype(np.float32).astype(np.float64)
    y = (g.random(rows) < 0.3).astype(float)
    w = omlp.flatten(omlp.init_params(4)).astype(np.float32).astype(np.float64)
    grad = omlp.flatten(omlp.backward(omlp.unflatten(w), X[:batch], y[:batch]))
    net = qs_lib.MLP(w)
    net.train(X, y, steps=1, batch=batch, lr=0.125)
    moved = net.get_params().astype(np.float64) - w
    big = np.abs(grad) > 1e-3 * np.abs(grad).max()
    np.testing.assert_allclose(moved[big], -0.125 * np.sign(grad[big]), atol=2e-5)
    assert np.all(np.abs(moved) <= 0.125 * (1 + 1e-5))
    net.free()
