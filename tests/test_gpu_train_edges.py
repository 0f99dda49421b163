"""The training kernels at the edges of their decomposition (16-sample chunks,
64-sample passes, one pass per block, several passes per block), against the
FP64 reference (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp_ref as M
from tests.test_gpu_learned import _bf16, _bf16_theta, _cuda, m2c  # noqa: F401

pytestmark = pytest.mark.gpu


def _data(seed, n):
    rng = np.random.default_rng(seed)
    theta = (M.init(6) + 0.02 * rng.standard_normal(M.NPARAM)).astype(np.float32)
    return theta, rng.standard_normal((8, n)).astype(np.float32), rng.standard_normal(n).astype(np.float32)


# The bar is the BF16 operand rounding of 64-term sums (8-bit mantissa): 3 %
# of a tensor's gradient in the 2-norm, 5 % of its largest entry element by
# element, as for the other gradient test; 2 % of the loss.
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 129, 4096, 256 * 64, 256 * 64 + 1, 40000])
def test_gradient_at_the_edges(m2c, n):  # noqa: F811
    theta, X, t = _data(n, n)
    g, loss = m2c.Mlp(theta).grad(_cuda(X), _cuda(t))
    tb = _bf16_theta(theta)
    gr = M.unpack(M.grad(tb, _bf16(X.T), t.astype(np.float64)))
    lr = M.loss(tb, _bf16(X.T), t.astype(np.float64))
    assert abs(loss - lr) <= 2e-2 * max(lr, 1e-2)
    pg = M.unpack(g.astype(np.float64))
    for name, _ in M.SIZES:
        a, b = pg[name].ravel(), gr[name].ravel()
        assert np.linalg.norm(a - b) <= 3e-2 * max(np.linalg.norm(b), 1e-30), (n, name)
        assert np.max(np.abs(a - b)) <= 5e-2 * max(np.max(np.abs(b)), 1e-30), (n, name)


@pytest.mark.parametrize("n", [1, 16, 63, 6144 * 16 + 5])
def test_forward_at_the_edges(m2c, n):  # noqa: F811
    theta, X, _ = _data(3, n)
    y = m2c.Mlp(theta).forward(_cuda(X)).cpu().numpy()
    yr = M.forward(_bf16_theta(theta), _bf16(X.T))
    assert np.max(np.abs(y - yr)) <= 2e-2 * max(1.0, np.max(np.abs(yr)))


@pytest.mark.parametrize("n,batch", [(100, 4096), (1000, 16), (5000, 4999)])
def test_one_epoch_is_adam_on_the_gradients(m2c, n, batch):  # noqa: F811
    """Training equals its own definition: Adam steps on the gradients that
    the gradient call returns, minibatch by minibatch.  Both sums are FP32
    over the same products; Adam's first steps divide by the root of the same
    gradients, so parameters agree to FP32 rounding of the update (1e-3 of a
    step of 1e-3, in all but entries whose gradient is itself rounding)."""
    theta, X, t = _data(11, n)
    net = m2c.Mlp(theta)
    net.train(_cuda(X), _cuda(t), epochs=1, batch=batch, lr=1e-3, lr_final=1e-3)
    got = net.params().astype(np.float64)
    p, m, v = theta.astype(np.float64), np.zeros(M.NPARAM), np.zeros(M.NPARAM)
    for k, i in enumerate(range(0, n, batch)):
        g, _ = m2c.Mlp(p.astype(np.float32)).grad(_cuda(X[:, i:i + batch].copy()), _cuda(t[i:i + batch].copy()))
        p, m, v = M.adam_step(p, g.astype(np.float64), m, v, k + 1, lr=1e-3)
    steps = -(-n // batch)
    assert np.linalg.norm(got - p) <= 1e-3 * np.linalg.norm(p - theta.astype(np.float64)) * steps
