"""MLP kernels at the edges of their tiles: widths and batches around 16 and 32
(rows, columns and inner blocks that end inside a tile), one layer, a batch
that shrinks after a larger one (stale rows in the transposed operands), the
loss trace over several calls; against the bfloat16-emulating NumPy oracle with
the bound of the other MLP tests (1e-2 of the largest magnitude)."""
import numpy as np
import pytest

from oracle import mlp as OM
from paper_2311_01242_amd.mlp import MLP

pytestmark = pytest.mark.gpu


def _net(widths, seed):
    rng = np.random.default_rng(seed)
    p = []
    for fi, fo in zip(widths[:-1], widths[1:]):
        p += [rng.normal(0.0, np.sqrt(2.0 / fi), fo * fi), rng.normal(0.0, 0.1, fo)]
    net = MLP(widths)
    net.set_params(np.concatenate(p).astype(np.float32))
    return net, np.concatenate(p).astype(np.float32).astype(np.float64), rng


def _check(net, p, widths, B, rng):
    x = rng.normal(size=(B, widths[0])).astype(np.float32)
    y = rng.normal(0.0, 0.3, (B, widths[-1])).astype(np.float32)
    loss, g = net.loss_grad(x, y)
    l_ref, g_ref = OM.loss_and_grad(p, widths, x, y)
    assert abs(loss - l_ref) <= 1e-2 * max(abs(l_ref), 1e-3)
    assert np.abs(g - g_ref).max() <= 1e-2 * np.abs(g_ref).max()
    out = net.forward(x)
    assert out.shape == (B, widths[-1]) and abs(float(((out - y) ** 2).mean()) - loss) <= 1e-5 * loss


@pytest.mark.parametrize("widths", [[1, 1], [5, 3], [16, 32, 17], [33, 31, 15, 64], [37, 300, 48], [8, 8, 8, 8, 8]])
@pytest.mark.parametrize("B", [1, 15, 33, 129, 300])
def test_widths_and_batches(widths, B):
    net, p, rng = _net(widths, sum(widths) + B)
    _check(net, p, widths, B, rng)


def test_shrinking_batch():
    widths = [9, 40, 21]
    net, p, rng = _net(widths, 3)
    for B in (70, 5, 37, 1, 70, 200, 33):
        _check(net, p, widths, B, rng)


def test_trace_and_parameters_over_calls():
    """Two calls of 3 and 4 steps are one call of 7: the same steps, trace and
    parameters, bit for bit."""
    widths = [11, 34, 19]
    a, p, rng = _net(widths, 8)
    b = MLP(widths)
    b.set_params(p.astype(np.float32))
    x = rng.normal(size=(45, 11)).astype(np.float32)
    y = rng.normal(size=(45, 19)).astype(np.float32)
    one = a.train(x, y, 7)
    two = np.concatenate([b.train(x, y, 3), b.train(x, y, 4)])
    assert np.array_equal(one, two) and np.array_equal(a.get_params(), b.get_params())
    assert abs(one[0] - OM.loss_and_grad(p, widths, x, y)[0]) <= 1e-2 * one[0] and one[-1] < one[0]
