"""Plans of the exchange solve's rows per block (8 to 64 rows, and one block of up to 128
without an exchange) against the FP64 oracle: the one-block form at its edges, single and
odd rows, row counts just past a power of two (idle row slots), blocks without rows of one
set, and in a batch.  The tolerance is that of the other executions' tests."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import rel
from test_gpu_fused import TOL, _errs, _run

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,T,M,rows,fused", [
    (3, 17, 1, 0, None), (2, 1, 17, 0, None), (3, 128, 128, 0, None), (2, 127, 65, 0, "mesh"),
    (2, 129, 129, 0, "mesh"), (3, 129, 5, 8, "mesh"), (3, 100, 333, 16, "mesh"),
    (2, 260, 90, 32, "mesh"), (3, 333, 470, 64, "mesh"), (2, 1025, 40, 0, "mesh"),
])
def test_rows_match_oracle(ct, monkeypatch, d, T, M, rows, fused):
    if rows:
        monkeypatch.setenv("CT_MESH_ROWS", str(rows))
    x, y, _w, _g = W.config_inputs(W.CONFIGS["grad_2d" if d == 2 else "autograd_3d"], T=T, M=M)
    w = W.positive_weights(np.random.default_rng(5), M)
    print(f"exchange rows d={d} T={T} M={M} rows={rows}", flush=True)
    for safe in (False, True):
        g = _run(ct, x, y, w, 0.01, 20, fused=fused, safe=safe)
        e = _errs(g, oracle.sinkhorn(x, y, w, eps=0.01, iters=20), T, M, w)
        assert max(e.values()) < TOL, (safe, e)
        assert g["aux"][6] == 0.0


@pytest.mark.parametrize("rows", [8, 32, 64])
def test_batch_rows_match_oracle(ct, monkeypatch, rows):
    monkeypatch.setenv("CT_MESH_ROWS", str(rows))
    P = [W.config_inputs(W.CONFIGS["autograd_3d"], T=T, M=M)[:2] for T, M in ((1, 9), (70, 64), (129, 33))]
    t = lambda i: [torch.as_tensor(p[i], device="cuda") for p in P]
    g = ct.sinkhorn_grad_batched(t(0), t(1), eps=0.01, iters=20, mode="mesh")
    for b, (x, y) in enumerate(P):
        r = oracle.sinkhorn(x, y, None, eps=0.01, iters=20)
        assert rel(g.grad_x[b].cpu().numpy(), r.grad_x) < TOL, b
