"""ct_sinkhorn_workspace_size asks for the cell form's arrays only where a call may take it."""
import ctypes

import pytest

from paper_2511_11514_amd import _lib

DB, VAL, GW, REF = _lib.CT_DEBIAS, _lib.CT_VALUE, _lib.CT_GRAD_W, _lib.CT_REF_CACHED


def _size(d, T, M, flags, iters=200, eps=0.005):
    return _lib.lib().ct_sinkhorn_workspace_size(
        T, M, ctypes.byref(_lib.SinkhornOpts(d, iters, eps, flags)))


@pytest.mark.parametrize("T,M", [(4096, 16384), (20000, 20001)])
def test_options_that_rule_the_form_out(T, M):
    base = _size(2, T, M, DB | VAL | _lib.CT_UNFUSED)
    for f in (_lib.CT_DIFFERENCE, _lib.CT_SAFE_LSE, _lib.CT_MESH, _lib.CT_FUSED, _lib.CT_TINY):
        assert _size(2, T, M, DB | VAL | f) == base
    assert _size(2, T, M, DB | VAL, iters=7) == base
    assert _size(2, T, M, DB | VAL) > base


def test_calls_below_the_limits():
    # too little work in all; 3-D sweeps of too few pairs
    assert _size(2, 4096, 16384, DB | VAL, iters=10) == _size(2, 4096, 16384, DB | VAL | _lib.CT_UNFUSED)
    assert _size(3, 16381, 16381, DB | VAL) == _size(3, 16381, 16381, DB | VAL | _lib.CT_UNFUSED)


def test_buffers_of_the_sweeps_that_run():
    """Each self problem's moments only where the options ask for it; a cached reference with a
    value still sweeps it once."""
    T, M = 20000, 40000
    sizes = [_size(2, T, M, f) for f in (0, DB, DB | VAL)]
    assert sizes[0] < sizes[1] < sizes[2]
    assert _size(2, T, M, DB | GW) == sizes[2] == _size(2, T, M, DB | VAL | REF)
    assert _size(2, T, M, VAL) == sizes[0]
    # 3-D: only the reference's own sweeps are large enough
    size = lambda f: _size(3, 16384, 65536, f, iters=300, eps=0.01)
    y = size(DB | VAL) - size(DB | VAL | _lib.CT_UNFUSED)
    assert 384 << 20 < y < 800 << 20
    assert size(DB) == size(DB | _lib.CT_UNFUSED)


def _batch(d, sizes, flags, eps, iters=100):
    off = lambda k: (ctypes.c_int64 * (len(sizes) + 1))(*[sum(s[k] for s in sizes[:i])
                                                          for i in range(len(sizes) + 1)])
    return _lib.lib().ct_sinkhorn_batched_workspace_size(
        len(sizes), off(0), off(1), ctypes.byref(_lib.SinkhornOpts(d, iters, eps, flags)))


@pytest.mark.parametrize("eps,offered", [(1e-4, False), (1e-3, False), (0.005, True), (0.02, True), (0.2, True)])
def test_offered_where_a_unit_box_has_few_cells(eps, offered):
    base = _size(2, 4096, 16384, DB | VAL | _lib.CT_UNFUSED, eps=eps)
    assert (_size(2, 4096, 16384, DB | VAL, eps=eps) > base) == offered


@pytest.mark.parametrize("sizes,eps,offered", [
    ([(4000, 20000)] * 12, 0.01, True), ([(4000, 20000)] * 12, 0.0005, False),
    ([(2500, 6000)] * 8, 0.005, False), ([(600, 900)] * 300, 0.1, False),
])
def test_batches_offered_where_it_pays(sizes, eps, offered):
    assert (_batch(2, sizes, DB, eps) > _batch(2, sizes, DB | _lib.CT_UNFUSED, eps)) == offered
