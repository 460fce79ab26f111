"""The cell form of the sweeps (the default of large calls; CT_CELL_MIN_PAIRS lets these
sizes take it) against the direct sweeps on the same inputs (fused=False) and the FP64 oracle: both dimensions, chunk
and tile remainders, warm start, cached reference, no debiasing, weights, one dense cell,
points that do not fit the coded box, non-finite inputs, small workspaces and graphs.

Tolerance: 1e-5 norm-wise, the float32 path's bar against the oracle; two float32 paths that
each meet it differ by at most twice that."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.fixture(autouse=True)
def _small_calls_take_the_cell_form(monkeypatch):
    monkeypatch.setenv("CT_CELL_MIN_PAIRS", "1.5e7")


def _inputs(d, T, M, seed=0):
    cfg = W.CONFIGS["grad_2d" if d == 2 else "autograd_3d"]
    x, y, _w, _g = W.config_inputs(cfg, T=T, M=M)
    w = W.positive_weights(np.random.default_rng(seed), M)
    return [torch.as_tensor(a, device="cuda") for a in (x, y, w)]


def _both(ct, x, y, w, **kw):
    kw = dict(dict(value=True, potentials=True, aux=True), **kw)
    a = ct.sinkhorn_grad(x, y, w, **kw)
    b = ct.sinkhorn_grad(x, y, w, fused=False, **kw)
    torch.cuda.synchronize()
    return a, b


def _close(a, b, T, M, debias=True):
    parts = {"f": (0, T), "g": (T, T + M)}
    if debias:
        parts.update(p=(T + M, 2 * T + M), q=(2 * T + M, 2 * T + 2 * M))
    errs = {"grad_x": rel(a.grad_x.cpu().numpy(), b.grad_x.cpu().numpy())}
    if a.grad_w is not None:
        errs["grad_w"] = rel(a.grad_w.cpu().numpy(), b.grad_w.cpu().numpy())
    for k, (i, j) in parts.items():
        errs[k] = rel(a.pot[i:j].cpu().numpy(), b.pot[i:j].cpu().numpy())
        errs[k + "+"] = rel(a.pot_plus[i:j].cpu().numpy(), b.pot_plus[i:j].cpu().numpy())
    errs["value"] = abs(a.value.item() - b.value.item()) / abs(b.value.item())
    bad = {k: v for k, v in errs.items() if not v <= TOL}
    assert not bad, (bad, errs)


@pytest.mark.parametrize("d,T,M,eps,iters", [
    (2, 2000, 6000, 0.005, 30),     # few chunks
    (2, 4097, 16383, 0.005, 12),    # one point past and short of whole tiles
    (2, 1031, 40009, 0.02, 9),      # large cells: chunks of one cell, 512 keys each
    (3, 1500, 33333, 0.02, 12),
    (3, 20011, 1201, 0.05, 8),
])
def test_matches_direct_sweeps(ct, d, T, M, eps, iters):
    x, y, w = _inputs(d, T, M)
    a, b = _both(ct, x, y, w, eps=eps, iters=iters, grad_w=True)
    assert not torch.equal(a.grad_x, b.grad_x)   # the two forms round differently
    _close(a, b, T, M)


def test_matches_oracle(ct):
    T, M, eps, K = 1500, 5003, 0.004, 25
    x, y, w = _inputs(2, T, M)
    a = ct.sinkhorn_grad(x, y, w, eps=eps, iters=K, value=True, grad_w=True)
    r = oracle.sinkhorn(*(t.cpu().numpy() for t in (x, y, w)), eps=eps, iters=K)
    assert rel(a.grad_x.cpu().numpy(), r.grad_x) < 1e-5
    assert rel(a.grad_w.cpu().numpy(), r.grad_w) < 1e-5
    assert abs(a.value.item() - r.value) < 1e-5 * abs(r.value)


@pytest.mark.parametrize("option", ["warm", "ref", "plain", "no_value"])
def test_options(ct, option):
    T, M, eps, K = 3001, 7001, 0.005, 15
    x, y, w = _inputs(2, T, M)
    kw = dict(eps=eps, iters=K)
    if option == "warm":
        kw["init"] = ct.sinkhorn_grad(x, y, w, eps=eps, iters=10, value=True, potentials=True).pot
    if option == "ref":
        kw["ref_q"] = ct.reference_self_potential(y, w, eps=eps, iters=K)
    if option == "plain":
        kw["debias"] = False
    if option == "no_value":
        a = ct.sinkhorn_grad(x, y, w, **kw).grad_x
        b = ct.sinkhorn_grad(x, y, w, fused=False, **kw).grad_x
        assert rel(a.cpu().numpy(), b.cpu().numpy()) < TOL
        return
    a, b = _both(ct, x, y, w, **kw)
    _close(a, b, T, M, debias=option != "plain")


def test_dense_cell_and_far_points(ct):
    """Most points in one cell (chunks of a cell, tiles of a cell), then a few far outside the
    coded box (the direct sweeps serve the call).  Both inputs cancel: near-equal clouds have
    potentials near zero, far points exponents of 10^5, so the direct sweeps themselves are
    beyond 1e-5 of the oracle; the default may be no worse than twice their error."""
    rng = np.random.default_rng(3)
    T, M = 3000, 9000
    x = torch.as_tensor((0.5 + 0.01 * rng.standard_normal((T, 2))).astype(np.float32), device="cuda")
    y = torch.as_tensor((0.5 + 0.01 * rng.standard_normal((M, 2))).astype(np.float32), device="cuda")
    for far in (False, True):
        if far:
            y[:3] += 50.0
        a, b = _both(ct, x, y, None, eps=0.01, iters=10)
        r = oracle.sinkhorn(x.cpu().numpy(), y.cpu().numpy(), None, eps=0.01, iters=10)
        for got, direct, want in ((a.grad_x, b.grad_x, r.grad_x), (a.pot[:T], b.pot[:T], r.f),
                                  (a.pot[T:T + M], b.pot[T:T + M], r.g),
                                  (a.pot[T + M:2 * T + M], b.pot[T + M:2 * T + M], r.p),
                                  (a.pot[2 * T + M:], b.pot[2 * T + M:], r.q)):
            e, e0 = rel(got.cpu().numpy(), want), rel(direct.cpu().numpy(), want)
            assert e <= max(1e-5, 2.0 * e0), (far, e, e0)


def test_nonfinite_inputs_are_counted(ct):
    x, y, w = _inputs(2, 2500, 6500)
    x[17, 0] = float("nan")
    y[5, 1] = float("inf")
    w[9] = 0.0
    a, b = _both(ct, x, y, w, eps=0.01, iters=8)
    assert a.aux[5].item() == b.aux[5].item() == 3.0


def test_repeatable_and_workspace_without_cells(ct):
    """Two calls agree bit for bit; a workspace of the size without the cell form's arrays
    serves the direct sweeps; so does the static scratch where they do not fit it."""
    from paper_2511_11514_amd import _lib
    x, y, w = _inputs(2, 3000, 9000)
    kw = dict(eps=0.005, iters=10, value=True)
    a, b = ct.sinkhorn_grad(x, y, w, **kw), ct.sinkhorn_grad(x, y, w, **kw)
    assert torch.equal(a.grad_x, b.grad_x) and torch.equal(a.value, b.value)
    direct = ct.sinkhorn_grad(x, y, w, fused=False, **kw)
    L = _lib.lib()
    o = _lib.SinkhornOpts(2, 10, 0.005, _lib.CT_DEBIAS | _lib.CT_VALUE)
    full = L.ct_sinkhorn_workspace_size(3000, 9000, ctypes.byref(o))
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    gx, val = torch.empty_like(x), torch.empty(1, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = L.ct_sinkhorn_grad(p(x), 3000, p(y), p(w), 9000, ctypes.byref(o), p(gx), None, p(val), None,
                            None, None, p(ws), full - 256 * 1024, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    assert rel(gx.cpu().numpy(), direct.grad_x.cpu().numpy()) < TOL


def test_graph_replays(ct):
    x, y, w = _inputs(2, 3000, 9000)
    kw = dict(eps=0.005, iters=10, value=True, grad_w=True)
    want = ct.sinkhorn_grad(x, y, w, **kw)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ct.sinkhorn_grad(x, y, w, **kw)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = ct.sinkhorn_grad(x, y, w, **kw)
    for _ in range(3):
        out.grad_x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.grad_x, want.grad_x) and torch.equal(out.grad_w, want.grad_w)
        assert torch.equal(out.value, want.value)
        ct.sinkhorn_grad(y, x, None, eps=0.01, iters=9)   # eager work between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("d,sizes", [
    (2, [(900, 9000), (3000, 700), (2049, 5121), (1, 3), (400, 12000)]),   # mixed: some problems sweep directly
    (3, [(600, 20000), (2500, 2600)]),
])
def test_batch_matches_direct_sweeps(ct, d, sizes):
    """The lockstep launches' cell form against mode="lockstep" (direct sweeps), eagerly and as a
    replayed graph with other calls between the replays."""
    rng = np.random.default_rng(d)
    t = lambda a: torch.as_tensor(a, device="cuda")
    xs, ys, ws = [], [], []
    for T, M in sizes:
        g = W.gmm_params(rng, 4, d, 0.03, 0.12)
        xs.append(t(W.random_walk(rng, T, d)))
        ys.append(t(W.gmm_sample(rng, g, M)))
        ws.append(t(W.positive_weights(rng, M)))
    kw = dict(eps=0.01, iters=10, value=True, grad_w=True)
    a = ct.sinkhorn_grad_batched(xs, ys, ws, **kw)
    b = ct.sinkhorn_grad_batched(xs, ys, ws, mode="lockstep", **kw)
    assert any(not torch.equal(u, v) for u, v in zip(a.grad_x, b.grad_x))
    for u, v in list(zip(a.grad_x, b.grad_x)) + list(zip(a.grad_w, b.grad_w)):
        if v.numel() > 8:
            assert rel(u.cpu().numpy(), v.cpu().numpy()) < TOL
    assert rel(a.value.cpu().numpy(), b.value.cpu().numpy()) < TOL
    bs = ct.BatchedSinkhorn(xs, ys, ws, **kw)
    bs.run()
    torch.cuda.synchronize()
    g = bs.capture()
    for _ in range(3):
        bs.grad_x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(bs.grad_x, torch.cat(a.grad_x)) and torch.equal(bs.value, a.value)
        ct.sinkhorn_grad(ys[0], xs[0], None, eps=0.01, iters=9)
        torch.cuda.synchronize()
