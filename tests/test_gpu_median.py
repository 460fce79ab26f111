"""The median bandwidth's selection at sizes where its units of 64 rows and columns, its two
targets and its passes can go wrong: h = med^2 / ln T against the sorted float32 distances
of the host (each squared distance is within 3 roundings of 2^-24, and so is h: 1e-6 covers them)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _median(x):
    T, d = x.shape
    c = x.astype(np.float32)
    i, j = np.triu_indices(T, 1)
    sq = ((c[i].astype(np.float64) - c[j]).astype(np.float32).astype(np.float64) ** 2).sum(1)
    sq = np.sort(np.sqrt(sq))
    n = len(sq)
    return 0.5 * (sq[(n - 1) // 2] + sq[n // 2])


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("T", [2, 3, 63, 64, 65, 127, 129, 1000, 4033])
def test_median_of_all_pairs(ct, d, T):
    rng = np.random.default_rng(T)
    scale = 10.0 ** rng.integers(-3, 4)
    x = (scale * rng.standard_normal((T, d))).astype(np.float32)
    print(f"median T={T} d={d}", flush=True)
    s = torch.zeros(T, d, device="cuda")
    for _ in range(2):
        _phi, h = ct.svgd_grad_score(torch.as_tensor(x, device="cuda"), s)
        m = _median(x)
        assert abs(float(h) - m * m / np.log(T)) < 1e-6 * m * m / np.log(T)


def test_two_targets_with_different_prefixes(ct):
    """The two middle ranks in different bins of the first pass: on a line 0, 1, 3, 64 the six
    distances are 1, 2, 3, 61, 63, 64 with middles 3 and 61."""
    x = np.array([[0, 0], [1, 0], [3, 0], [64, 0]], dtype=np.float32)
    _phi, h = ct.svgd_grad_score(torch.as_tensor(x, device="cuda"), torch.zeros(4, 2, device="cuda"))
    assert abs(float(h) - 32.0 ** 2 / np.log(4)) < 1e-6 * 32.0 ** 2
