"""The wide solver's plain steps are steered by trace X and |X|_F^2 in 64 bits.  2 tr X - |X|_F^2 doubles what the
carried trace is off by in every growth step, and a small eigenvalue m needs forty of them: in 32 bits the
trace then says "square" where it should not, five to seven times a solve (the answer stays right, the maps
keep the order)."""
import numpy as np
import pytest
from scipy.stats import random_correlation

from gpu_util import announce
from near_copies import factor

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def steps_of(ev, m):
    """Steps of a first solve on eigenvalues ev: folded growth from x_{m+1} <= 1 / (m + 1), then plain steps until the
    bounds of the lower eigenvalues' sum and the upper ones' distances from 1, squared in turn, are below 1e-12."""
    x, H, k = ev / ev.sum(), 1.0001 / (m + 1), 0
    g = H
    while 1 - g >= 0.5 and k < 40:
        c = min(max(2 / (1 + H), 1), 2)
        x, g, H = 1 - (1 - c * x) ** 2, 1 - (1 - c * g) ** 2, min(1 - (1 - c * H) ** 2, 1 - (1 - c) ** 2)
        k += 1
    square = False
    while True:
        t, F = x.sum(), (x * x).sum()
        if t - F < 0.02 and abs(t - m) < 0.25:
            break
        x, square = x * x if square else 2 * x - x * x, (F if square else 2 * t - F) > m
        k += 1
    A, B = (0.5 * (1.02 * (t - F) + s * (t - m)) for s in (1, -1))
    while True:
        A, B = (A * A, 2 * B) if square else (2 * A, B * B)
        square = A > B
        k += 1
        if max(A, B) < 1e-12:
            return k


@pytest.mark.parametrize("p,m", [(48, 47), (50, 49), (63, 62), (60, 59), (33, 32)])
def test_a_small_eigenvalue_takes_no_more_steps_than_in_64_bits(p, m):
    from paper_2302_05865_amd import FlagAggregator
    announce("steering", p, m)
    ev = 1e-11 ** (np.arange(p) / (p - 1))
    K = random_correlation.rvs(ev / ev.sum() * p, random_state=100 * p + m, tol=1e-8)
    R = factor(K)
    agg = FlagAggregator(n_max=1 << 20, p_max=64)
    agg.fa_irls(K, m, 0.0, 1, 0.0)
    x = agg.fa_get_info()
    agg.close()
    expected = steps_of(np.maximum(np.sort(np.linalg.eigvalsh(R @ R.T))[::-1], 0), m)
    print(p, m, x.rank, x.sweeps, expected)
    assert x.status == 0 and x.rank == len(R) == p
    assert abs(x.sweeps - expected) <= 1
