"""Where the wide solver hands a solve to the Jacobi kernel behind it: before the first purification step
(wide_spin_budget = 0), and at the step limit, where the purification cannot end.  Any other budget means
nothing: no wavefront polls.  (A guess that fails and is redone: test_gpu_planned_steps.py.)"""
import numpy as np
import pytest

from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# tiles 2, 3 and 4, a general exponent, blocks of k columns at one, two and four tiles
PROBLEMS = [(20, 1, 2.0), (40, 1, 2.0), (64, 1, 2.0), (20, 1, 4.0), (10, 2, 2.0), (32, 4, 2.0), (60, 2, 2.0)]


def answer(G, p, k, a, m, lam, iters, **kw):
    from paper_2302_05865_amd import FlagAggregator
    agg = FlagAggregator(n_max=G.shape[1], p_max=p, exponent_a=a, **kw)
    if k == 1:
        agg.fa_aggregate(G, m, lam, iters, 0.0)
    else:
        agg.fa_aggregate_grouped(G, [k] * (p // k), m, lam, iters, 0.0)
    info = agg.fa_get_info()
    agg.close()
    return info


@pytest.mark.parametrize("p,k,a", PROBLEMS)
def test_only_a_budget_of_zero_hands_the_solve_over(p, k, a):
    """Same K (fp64, the same kernel) in front of both solvers; projectors good to eps p / gap, the gap at m
    here above 1e-3: 1e-8 on the objective, the coefficients and the basis."""
    n, m, iters = 400, (p + 2) // 2, 4
    r = np.random.default_rng(p + k)
    G = to_device((r.standard_normal((p, n)) * 0.5 + r.standard_normal((1, n))).astype(np.float32))
    ref = answer(G, p, k, a, m, 1.0, iters, solver="jacobi")
    scale = np.sqrt(np.diag(ref.K))
    announce("spin budget", p, k, a)
    zero, one, default = (answer(G, p, k, a, m, 1.0, iters, **kw)
                          for kw in ({"wide_spin_budget": 0}, {"wide_spin_budget": 1}, {}))
    assert zero.status == 0 and zero.sweeps == ref.sweeps and np.array_equal(zero.c, ref.c)
    assert one.sweeps == default.sweeps != ref.sweeps and np.array_equal(one.c, default.c)
    assert one.status == 0 and one.rank == ref.rank and one.iters_done == iters
    assert np.max(np.abs(one.objective - ref.objective) / (1.0 + np.abs(ref.objective))) <= 1e-8
    assert np.linalg.norm((one.c - ref.c) * scale) <= 1e-8 * np.linalg.norm(ref.c * scale)
    assert np.max(np.abs(one.A.T @ one.K @ one.A - np.eye(m))) <= 1e-9


@pytest.mark.parametrize("p,k,a", PROBLEMS)
def test_a_purification_that_cannot_end_hands_the_solve_over(p, k, a):
    """Unit vectors: M is a multiple of the identity, to the bit, and no map takes its eigenvalues apart.  Every role
    leaves at the step limit, and the Jacobi kernel answers, bit for bit."""
    m, iters = (p + 2) // 2, 3
    G = to_device(np.eye(p, 400, dtype=np.float32))
    announce("no end", p, k, a)
    ref = answer(G, p, k, a, m, 0.0, iters, solver="jacobi")
    got = answer(G, p, k, a, m, 0.0, iters)
    assert got.status == 0 and got.rank == p and got.iters_done == iters
    assert got.sweeps == ref.sweeps and np.array_equal(got.c, ref.c) and np.array_equal(got.A, ref.A)
    assert np.max(np.abs(got.A.T @ got.A - np.eye(m))) <= 1e-12
