"""The cell form's truncated expansion (paper_2511_11514_amd/csrc/cells.h) on the CPU: the
products that the kernels keep, against e^(lambda s.u) itself, whatever the two points."""
import math
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2511_11514_amd", "csrc")


def _table(d):
    src = open(os.path.join(CSRC, "cells.hip")).read()
    body = re.search(r"kTerms%d\[[^\]]*\] = \{(.*?)\};" % d, src, re.S).group(1)
    codes = [int(v, 16) for v in re.findall(r"0x[0-9a-f]+", body)]
    return np.array([[(c >> (4 * t)) & 15 for t in range(d)] for c in codes])


def _dim(d, name):
    src = open(os.path.join(CSRC, "cells.h")).read()
    body = re.search(r"struct CellDim<%d> \{(.*?)\};" % d, src, re.S).group(1)
    return float(re.search(r"\b%s = ([0-9.]+);" % name, body).group(1))


def _bessel(n, z):
    return sum((z / 2) ** (n + 2 * m) / (math.factorial(m) * math.factorial(n + m)) for m in range(12))


@pytest.mark.parametrize("d", [2, 3])
def test_kept_products_reproduce_the_kernel(d):
    terms, lam = _table(d), _dim(d, "lambda")
    assert len(terms) == _dim(d, "N") and terms.max() < _dim(d, "F")
    assert len({tuple(t) for t in terms.tolist()}) == len(terms)
    rng = np.random.default_rng(d)
    s, u = rng.uniform(-1, 1, (400, d)), rng.uniform(-1, 1, (400, d))
    # the corners, where the left-out terms are largest
    corner = np.array(np.meshgrid(*[[-1.0, 1.0]] * d)).reshape(d, -1).T
    s[:len(corner)], u[:len(corner)] = corner, 1.0
    F = int(terms.max()) + 1
    phi = np.stack([(2 if n else 1) * _bessel(n, lam * s) for n in range(F)])       # [F, n, d]
    cheb = np.stack([np.cos(n * np.arccos(u)) for n in range(F)])
    got = sum(np.prod([phi[t[a], :, a] * cheb[t[a], :, a] for a in range(d)], axis=0) for t in terms)
    want = np.exp(lam * (s * u).sum(1))
    # stated in cells.h: the left-out terms add up to less than 9e-8
    assert np.max(np.abs(got - want)) < 9e-8
