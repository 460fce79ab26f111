"""Rescued self rows of the exchange solve's one-block form (65 to 128 points a side, the default
route) against the FP64 oracle: restarts far from the fixed point, with every row's shift
unusable, and with those of one 64-row half only (the two halves are finished by different
waves).  The tolerance is that of the other executions' rescue tests; repeats are bit-equal."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_fused import TOL, _errs, _run

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,T,M", [(2, 128, 128), (3, 128, 97), (2, 65, 128), (3, 100, 100)])
@pytest.mark.parametrize("which", ["all", "first", "second"])
def test_far_restart_matches_oracle(ct, d, T, M, which):
    x, y, _w, _g = W.config_inputs(W.CONFIGS["grad_2d" if d == 2 else "autograd_3d"], T=T, M=M)
    w = W.positive_weights(np.random.default_rng(13), M)
    eps, K = 0.01, 20
    base = oracle.sinkhorn(x, y, w, eps=eps, iters=40)
    p, q = base.p.copy(), base.q.copy()
    rows = {"all": slice(None), "first": slice(0, 64), "second": slice(64, None)}[which]
    p[rows] = -2.0
    q[rows] = -2.0
    init = np.concatenate([base.f, base.g, p, q]).astype(np.float32)
    print(f"one-block far restart d={d} T={T} M={M} {which}", flush=True)
    g = _run(ct, x, y, w, eps, K, fused=None, init=init)
    assert g["aux"][4] > 0, "rescue path was not exercised"
    i = init.astype(np.float64)
    r = oracle.sinkhorn(x, y, w, eps=eps, iters=K,
                        init=(i[:T], i[T:T + M], i[T + M:2 * T + M], i[2 * T + M:]))
    e = _errs(g, r, T, M, w)
    assert max(e.values()) < TOL, e
    for _ in range(3):
        again = _run(ct, x, y, w, eps, K, fused=None, init=init)
        for k in ("grad_x", "grad_w", "value", "pot"):
            assert np.array_equal(g[k], again[k]), k
