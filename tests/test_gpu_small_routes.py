"""Which execution small calls take by default: the same bits as the forced one-workgroup solve
below the thresholds, others above (their sums run in another order)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,value,one_workgroup", [
    (64, True, True), (65, True, False), (20, False, True), (21, False, False),
])
def test_default_execution(ct, n, value, one_workgroup):
    rng = np.random.default_rng(n)
    g = W.gmm_params(rng, 3, 3, 0.05, 0.12)
    x, y = (torch.as_tensor(a, device="cuda") for a in (W.random_walk(rng, n, 3), W.gmm_sample(rng, g, n)))
    kw = dict(eps=0.01, iters=50, value=value, potentials=True)
    a, b = ct.sinkhorn_grad(x, y, **kw), ct.sinkhorn_grad(x, y, fused="tiny", **kw)
    assert torch.equal(a.pot, b.pot) == one_workgroup
    assert torch.allclose(a.grad_x, b.grad_x, rtol=0, atol=1e-5 * b.grad_x.abs().max().item())
