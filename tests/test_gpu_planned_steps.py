"""Purification steps that need no trace: planned from the previous solve's gap (16 < p <= 64: where the
guess holds, where it does not and the solve is done again, every tile count) and the folded first
growth steps (p <= 16: every width class of the solver)."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def gram_of(p, seed, n=200):
    """Workers around a common direction (or none), some of them replaced by scaled noise or
    copies: the gap at m moves by orders of magnitude from one solve to the next."""
    r = np.random.default_rng(seed)
    G = r.standard_normal((p, n)) * 0.5 + (r.standard_normal((1, n)) if r.random() < 0.7 else 0)
    for i in range(r.integers(0, p // 2)):
        G[i] = r.choice([-4, 5, 0.01]) * r.standard_normal(n) + r.choice([0, 1]) * G[-1]
    return G @ G.T


# the first nine: a NumPy model of the steps says that a guess fails in one of the solves
@pytest.mark.parametrize("p,m,lam,seed", [
    (17, 5, 0.1, 636078391), (27, 6, 0.1, 604592858), (25, 23, 0.0, 746945520),
    (21, 20, 4.0, 614711476), (26, 23, 0.1, 651383795), (23, 8, 0.0, 515711975),
    (18, 2, 0.0, 981457606), (31, 30, 0.1, 656153625), (17, 5, 0.1, 403139253),
    (17, 16, 1.0, 1), (32, 1, 1.0, 2), (33, 17, 1.0, 3), (48, 24, 0.1, 4), (48, 47, 1.0, 5),
    (49, 3, 1.0, 6), (64, 32, 0.1, 7), (64, 63, 4.0, 8), (64, 1, 0.0, 9)])
def test_planned_steps_give_the_jacobi_solvers_answer(p, m, lam, seed):
    _compare_with_jacobi(p, m, lam, seed)


@pytest.mark.parametrize("p", [2, 4, 5, 8, 9, 12, 13, 16])
def test_folded_growth_gives_the_jacobi_solvers_answer(p):
    """m = 1 (no folded step: the bound is 1/2 already) to m = p (no purification at all); widths on
    both sides of every count of matrix instructions per product."""
    for m in sorted({1, 2, p // 2, p - 1, p}):
        _compare_with_jacobi(p, m, 0.3, 11 * p + m)


def _compare_with_jacobi(p, m, lam, seed):
    """Both solvers start from the same K in fp64.  Each solve's projector is good to eps p / gap,
    and passes that on to the next solve's weights; the objective after every solve and the
    coefficients agree to 1e-8 where the relative gap at m stays above 1e-5."""
    from paper_2302_05865_amd import FlagAggregator
    announce("planned steps", p, m, lam, seed)
    K = gram_of(p, seed)
    got = []
    for solver in ("auto", "jacobi"):
        agg = FlagAggregator(n_max=1 << 20, p_max=64, solver=solver)
        agg.fa_irls(K, m, lam, 8, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    a, j = got
    assert a.status == 0 and j.status == 0 and a.rank == j.rank and a.iters_done == 8
    assert np.max(np.abs(a.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-8
    scale = np.sqrt(np.diag(K))
    assert np.linalg.norm((a.c - j.c) * scale) <= 1e-8 * np.linalg.norm(j.c * scale)
    assert np.max(np.abs(a.A.T @ K @ a.A - np.eye(m))) <= 1e-9
