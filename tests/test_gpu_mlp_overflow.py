"""A network whose weights have grown infinite: rows that fill up a group of 16
leave no trace in the gradient."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def diverged(qs_lib):
    """One step of an oversized learning rate from weights chosen so that the
    first layer's weights on input 0 and its biases become infinite, with
    alternating signs, and the other layers' stay finite."""
    P = np.zeros(6337, np.float32)
    w1, b1, w2, b2, w3 = 0, 2048, 2112, 6208, 6272
    P[w1:w1 + 64] = 1e38
    P[w2:b2] = np.repeat(np.where(np.arange(64) % 2, -1e4, 1e4), 64)
    P[b2:w3] = 0.5
    P[w3:w3 + 64] = 1.0
    net = qs_lib.MLP(P)
    X = np.zeros((1, 32), np.float32)
    X[0, 0] = 1e-38
    net.train(X, np.zeros(1, np.float32), steps=1, batch=1, lr=3e38, beta1=0.0, beta2=0.0, eps=1e-34)
    got = net.get_params()
    assert np.isinf(got[:64]).all() and np.isfinite(got[w2:]).all()
    return net


@pytest.mark.parametrize("rows", [1, 2, 4, 8])
def test_gradient_of_part_of_a_group(qs_lib, rows):
    net = diverged(qs_lib)
    g = np.random.default_rng(rows)
    X = np.abs(g.standard_normal((rows, 32))).astype(np.float32)
    y = (np.arange(rows) % 2).astype(np.float32)
    # the mean over the rows repeated to a whole group is the same, exactly: the
    # sums are of halves, quarters, ... of ones
    part, _ = net.grad(X, y)
    whole, _ = net.grad(np.tile(X, (16 // rows, 1)), np.tile(y, 16 // rows))
    assert np.isfinite(whole).all() and np.any(whole != 0)
    np.testing.assert_array_equal(part, whole)
    net.free()
