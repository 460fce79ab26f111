"""The cell form of the 2-D Stein sum (from 32768 points on) against the flow's definition in
float64 for a sample of the points, and against the direct sum of a call whose workspace has
no room for it.

phi_i = 1/T sum_j k_ij [score_j + (2/h)(x_i - x_j)].  Point sets: one cell's worth, clusters with
empty cells between them, all points on a line, a size that is no multiple of a tile, a spread
over more cells than the form takes, a score that is not finite (the last two sum directly).  The
tolerance is that of the direct sum's tests at these sizes: 2e-5 of the flow's norm."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 2e-5


def _points(name, T, rng):
    if name == "one cell":
        return 5.0 + 0.01 * rng.random((T, 2)), 1.0
    if name == "clusters":
        c = rng.random((7, 2)) * [3.0, 1.0] - 1.0
        return c[rng.integers(0, 7, T)] + 0.02 * rng.standard_normal((T, 2)), None
    if name == "line":
        t = rng.random(T)
        return np.stack([t, 0.25 * np.ones(T)], 1), 0.01
    if name == "many cells":
        return rng.random((T, 2)), 2e-4
    return rng.random((T, 2)), None


def _flow64(x, s, h, idx):
    out = np.empty((len(idx), 2))
    for k, i in enumerate(idx):
        d = x[i] - x
        w = np.exp(-(d * d).sum(1) / h)
        out[k] = (w[:, None] * (s + (2.0 / h) * d)).sum(0) / len(x)
    return out


@pytest.mark.parametrize("name,T", [("one cell", 32768), ("clusters", 32769), ("line", 40000),
                                    ("uniform", 33001), ("many cells", 32768)])
def test_flow_matches_its_definition(ct, name, T):
    rng = np.random.default_rng(len(name))
    x, h = _points(name, T, rng)
    x = x.astype(np.float32)
    s = (10.0 * rng.standard_normal((T, 2)) + 3.0).astype(np.float32)
    xt, st = torch.as_tensor(x, device="cuda"), torch.as_tensor(s, device="cuda")
    print(f"stein cells {name} T={T}", flush=True)
    phi, hu = ct.svgd_grad_score(xt, st, h)
    again, _ = ct.svgd_grad_score(xt, st, h)
    assert torch.equal(phi, again)
    idx = np.concatenate([[0, T - 1], rng.integers(0, T, 200)])
    ref = _flow64(x.astype(np.float64), s.astype(np.float64), float(hu), idx)
    err = np.linalg.norm(phi.cpu().numpy()[idx] - ref) / np.linalg.norm(ref)
    assert err < TOL, err


def test_smaller_workspace_takes_the_direct_sum(ct):
    from paper_2511_11514_amd import _lib as L
    T, h = 32768, 0.01
    rng = np.random.default_rng(1)
    x = torch.as_tensor(rng.random((T, 2)).astype(np.float32), device="cuda")
    s = torch.as_tensor(rng.standard_normal((T, 2)).astype(np.float32), device="cuda")
    full = L.lib().ct_svgd_workspace_size(T, 2)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    out = []
    for nbytes in (full, full - 256):
        ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        phi = torch.empty_like(x)
        at = ctypes.c_void_p((ws.data_ptr() + 255) // 256 * 256)
        assert L.lib().ct_svgd_grad_score(p(x), T, 2, p(s), ctypes.c_float(h), p(phi), None, at,
                                          nbytes, stream) == L.CT_OK
        out.append(phi.cpu().numpy().astype(np.float64))
    assert np.linalg.norm(out[0] - out[1]) < TOL * np.linalg.norm(out[1])
    assert not np.array_equal(out[0], out[1])     # two different summations


def test_a_score_that_is_not_finite_spreads_as_in_the_direct_sum(ct):
    T = 32768
    rng = np.random.default_rng(2)
    x = torch.as_tensor(rng.random((T, 2)).astype(np.float32), device="cuda")
    s = torch.zeros(T, 2, device="cuda")
    s[77, 0] = float("nan")
    phi, _ = ct.svgd_grad_score(x, s, 0.01)
    assert torch.isnan(phi[:, 0]).all() and torch.isfinite(phi[:, 1]).all()
