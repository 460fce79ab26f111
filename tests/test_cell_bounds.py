"""What the truncated expansions leave out of a pair's own term, as include/ct.h states it: the
soft-min's cell form (cells.h) and the Stein sum's (stein.h), for all pairs of corners of a cell,
where the term is smallest and the left-out part largest, and for points between them."""
import math
import os
import re

import numpy as np
import pytest

from test_cell_terms import _bessel, _dim, _table

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_11514_amd", "csrc")


def _points(d):
    rng = np.random.default_rng(d)
    corner = np.array(np.meshgrid(*[[-1.0, 1.0]] * d)).reshape(d, -1).T
    s = np.concatenate([rng.uniform(-1, 1, (3000, d))] + [corner] * len(corner))
    u = np.concatenate([rng.uniform(-1, 1, (3000, d))] + [np.repeat(c[None], len(corner), 0) for c in corner])
    return s, u


def _left_out(terms, lam, s, u):
    """|kept - whole| / whole of e^(lambda s.u) at points s, u of [-1, 1]^d."""
    d = s.shape[1]
    F = int(terms.max()) + 1
    phi = np.stack([(2 if n else 1) * _bessel(n, lam * s) for n in range(F)])
    cheb = np.stack([np.cos(n * np.arccos(u)) for n in range(F)])
    got = sum(np.prod([phi[t[a], :, a] * cheb[t[a], :, a] for a in range(d)], axis=0) for t in terms)
    want = np.exp(lam * (s * u).sum(1))
    return np.max(np.abs(got - want) / want)


def _stated(text):
    """The bounds that the header states, in order: soft-min 2-D, 3-D, Stein."""
    flat = re.sub(r"[\s*]+", " ", text)
    a = re.search(r"truncated expansions that leave out less than ([\d.e-]+) of any pair's term \(([\d.e-]+) in 3-D\)", flat)
    b = re.search(r"truncated expansions that leave out less than ([\d.e-]+) of any pair's term;", flat)
    return float(a.group(1)), float(a.group(2)), float(b.group(1))


def test_header_states_what_is_left_out():
    soft2, soft3, stein = _stated(open(os.path.join(ROOT, "include", "ct.h")).read())
    for d, bound in ((2, soft2), (3, soft3)):
        e = _left_out(_table(d), _dim(d, "lambda"), *_points(d))
        assert 0.5 * bound < e < bound, (d, e, bound)
    src = open(os.path.join(CSRC, "stein.h")).read()
    side = float(re.search(r"kSteinSide = ([\d.]+)f", src).group(1))
    terms = np.array([[i % 8, i // 8] for i in range(64)])
    e = _left_out(terms, 0.5 * math.log(2.0) * side * side, *_points(2))
    assert 0.5 * stein < e < stein, (e, stein)


@pytest.mark.parametrize("d", [2, 3])
def test_side_gives_lambda(d):
    src = open(os.path.join(CSRC, "cells.h")).read()
    body = re.search(r"struct CellDim<%d> \{(.*?)\};" % d, src, re.S).group(1)
    num, den = map(float, re.search(r"side = ([\d.]+) / (\d+);", body).groups())
    assert abs(_dim(d, "lambda") - 0.5 * math.log(2.0) * (num / den) ** 2) < 1e-7
    assert math.log2(den).is_integer() and num < 1024
