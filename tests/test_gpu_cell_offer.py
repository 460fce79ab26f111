"""Calls that are not offered the cell form (points of a unit box in too many cells for their
number) sweep directly: the same bits as fused=False and mode="lockstep"."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _points(rng, d, T, M):
    g = W.gmm_params(rng, 5, d, 0.03, 0.12)
    return [torch.as_tensor(a, device="cuda") for a in (W.random_walk(rng, T, d), W.gmm_sample(rng, g, M))]


@pytest.mark.parametrize("eps,offered", [(0.001, False), (0.01, True)])
def test_single(ct, eps, offered):
    x, y = _points(np.random.default_rng(1), 2, 3001, 9001)
    kw = dict(eps=eps, iters=70, value=True)
    a, b = ct.sinkhorn_grad(x, y, **kw), ct.sinkhorn_grad(x, y, fused=False, **kw)
    assert torch.equal(a.grad_x, b.grad_x) != offered and (offered or torch.equal(a.value, b.value))


@pytest.mark.parametrize("eps,offered", [(0.005, False), (0.02, True)])
def test_batch(ct, eps, offered):
    rng = np.random.default_rng(2)
    xs, ys = zip(*[_points(rng, 2, 2000 + 100 * i, 7000 - 300 * i) for i in range(8)])
    kw = dict(eps=eps, iters=60)
    a, b = ct.sinkhorn_grad_batched(xs, ys, **kw), ct.sinkhorn_grad_batched(xs, ys, mode="lockstep", **kw)
    assert all(torch.equal(u, v) for u, v in zip(a.grad_x, b.grad_x)) != offered
