"""The wide solver's bounded wait with budgets that run out somewhere inside a purification: a few
polls, so that a wavefront may give up on any word, the one that says "this is the result" among
them.  Whatever the polls make of it, the answer is the Jacobi solver's."""
import numpy as np
import pytest

from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BUDGETS = [*range(1, 17), *range(18, 65, 2), 96, 128]


@pytest.mark.parametrize("p,k,a", [(20, 1, 2.0), (40, 1, 2.0), (64, 1, 2.0), (20, 1, 4.0),
                                   (10, 2, 2.0), (32, 4, 2.0), (60, 2, 2.0)])
def test_a_wait_that_runs_out_in_any_step_hands_the_solve_over(p, k, a):
    """Tiles 2, 3 and 4, a general exponent, blocks of k columns at one, two and four tiles.  Same K
    (fp64, the same kernel) in front of both solvers; projectors good to eps p / gap, the gap at m
    here above 1e-3: 1e-8 on the objective, the coefficients and the basis."""
    from paper_2302_05865_amd import FlagAggregator
    n, m, iters = 400, (p + 2) // 2, 4
    r = np.random.default_rng(p + k)
    G = to_device((r.standard_normal((p, n)) * 0.5 + r.standard_normal((1, n))).astype(np.float32))

    def answer(**kw):
        agg = FlagAggregator(n_max=n, p_max=p, exponent_a=a, **kw)
        if k == 1:
            agg.fa_aggregate(G, m, 1.0, iters, 0.0)
        else:
            agg.fa_aggregate_grouped(G, [k] * (p // k), m, 1.0, iters, 0.0)
        info = agg.fa_get_info()
        agg.close()
        return info

    ref = answer(solver="jacobi")
    scale = np.sqrt(np.diag(ref.K))
    for budget in BUDGETS:
        announce("spin budget", p, k, a, budget)
        got = answer(wide_spin_budget=budget)
        assert got.status == 0 and got.rank == ref.rank and got.iters_done == iters, budget
        assert np.max(np.abs(got.objective - ref.objective) / (1.0 + np.abs(ref.objective))) <= 1e-8, budget
        assert np.linalg.norm((got.c - ref.c) * scale) <= 1e-8 * np.linalg.norm(ref.c * scale), budget
        assert np.max(np.abs(got.A.T @ got.K @ got.A - np.eye(m))) <= 1e-9, budget
