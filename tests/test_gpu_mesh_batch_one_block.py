"""Batches whose problems all fit one block of the exchange solve (at most 128 points a side)
against the FP64 oracle: edges of the form, unequal problems, more problems than compute units,
and replays of a captured graph.  The tolerance is that of the other executions' tests."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import rel
from test_gpu_fused import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _problems(d, sizes):
    rng = np.random.default_rng(7)
    out = []
    for T, M in sizes:
        g = W.gmm_params(rng, 3, d, 0.05, 0.12)
        out.append((W.random_walk(rng, T, d), W.gmm_sample(rng, g, M), W.positive_weights(rng, M)))
    return out


@pytest.mark.parametrize("d,sizes", [
    (2, [(1, 1), (128, 128), (64, 65), (17, 3), (127, 1), (2, 90)]),
    (3, [(128, 100)] * 3 + [(33, 64), (1, 128)]),
    (3, [(5 + i % 9, 4 + i % 7) for i in range(300)]),
])
@pytest.mark.parametrize("value", [False, True])
def test_matches_oracle(ct, d, sizes, value):
    P = _problems(d, sizes)
    xs, ys, ws = [[torch.as_tensor(p[i], device="cuda") for p in P] for i in range(3)]
    print(f"one-block batch d={d} B={len(P)} value={value}", flush=True)
    bs = ct.BatchedSinkhorn(xs, ys, ws, eps=0.01, iters=30, value=value, grad_w=value, mode="mesh")
    bs.run()
    torch.cuda.synchronize()
    gx, want = bs.split(bs.grad_x, bs.T_off), bs.grad_x.clone()
    gw = bs.split(bs.grad_w, bs.M_off) if value else None
    for b in list(range(min(6, len(P)))) + [len(P) - 1]:
        r = oracle.sinkhorn(*P[b], eps=0.01, iters=30)
        assert rel(gx[b].cpu().numpy(), r.grad_x) < TOL, (b, sizes[b])
        if value:
            assert rel(gw[b].cpu().numpy(), r.grad_w) < TOL, (b, sizes[b])
            assert abs(bs.value[b].item() - r.value) < TOL * abs(r.value), (b, sizes[b])
    g = bs.capture()
    for _ in range(3):
        bs.grad_x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(bs.grad_x, want)
        ct.sinkhorn_grad(xs[0], ys[0], eps=0.01, iters=5)
        torch.cuda.synchronize()
