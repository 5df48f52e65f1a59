"""Purification steps that need no trace: planned from the previous solve's gap (16 < p <= 64: where the
guess holds, where it does not and the solve is done again, every tile count, single columns and
blocks, a general exponent) and the folded first growth steps (p <= 16: every width class of the
solver).  info.sweeps counts steps, those of a solve that is done again among them."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def stand_by(p):
    """The solver that a purification which fails is handed to."""
    return "jacobi" if p > 16 else "jacobi16"


def grads_of(p, seed, n=200):
    """Workers around a common direction (or none), some of them replaced by scaled noise or
    copies: the gap at m moves by orders of magnitude from one solve to the next."""
    r = np.random.default_rng(seed)
    G = r.standard_normal((p, n)) * 0.5 + (r.standard_normal((1, n)) if r.random() < 0.7 else 0)
    for i in range(r.integers(0, p // 2)):
        G[i] = r.choice([-4, 5, 0.01]) * r.standard_normal(n) + r.choice([0, 1]) * G[-1]
    return G


def gram_of(p, seed):
    G = grads_of(p, seed)
    return G @ G.T


# the first nine: the gap moves by orders of magnitude between the first two solves
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


@pytest.mark.parametrize("p,rank", [(16, 16), (16, 13), (16, 9), (15, 4), (12, 11), (9, 8), (8, 5), (7, 7), (5, 2),
                                    (4, 4), (3, 2)])
def test_steering_with_and_without_copies(p, rank):
    """p <= 16: the steps run on 2X - I with the identity of the rank, which need not be p; the last ones
    are counted from the measured distance.  Same bounds as test_every_remainder_of_the_last_tile."""
    from paper_2302_05865_amd import FlagAggregator
    announce("steering", p, rank)
    K = _with_copies(p, rank, 7 * p + rank)
    scale = np.sqrt(np.diag(K))
    for m in sorted({1, (rank + 1) // 2, rank - 1}):
        got = []
        for solver in ("auto", stand_by(p)):
            agg = FlagAggregator(n_max=1 << 20, p_max=16, solver=solver)
            agg.fa_irls(K, m, 0.5, 9, 0.0)
            got.append(agg.fa_get_info())
            agg.close()
        a, j = got
        assert a.status == 0 and j.status == 0 and a.rank == j.rank == rank and a.sweeps != j.sweeps, m
        assert np.max(np.abs(a.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-8, m
        assert np.linalg.norm(K @ (a.c - j.c) / scale) <= 1e-8 * np.linalg.norm(K @ j.c / scale), m


def _compare_with_jacobi(p, m, lam, seed):
    """Both solvers start from the same K in fp64.  Each solve's projector is good to eps p / gap,
    and passes that on to the next solve's weights; the objective after every solve and the
    coefficients agree to 1e-8 where the relative gap at m stays above 1e-5."""
    from paper_2302_05865_amd import FlagAggregator
    announce("planned steps", p, m, lam, seed)
    K = gram_of(p, seed)
    got = []
    for solver in ("auto", stand_by(p)):
        agg = FlagAggregator(n_max=1 << 20, p_max=64, solver=solver)
        agg.fa_irls(K, m, lam, 8, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    a, j = got
    assert m >= a.rank or a.sweeps != j.sweeps          # the Jacobi solver did not do it
    assert a.status == 0 and j.status == 0 and a.rank == j.rank and a.iters_done == 8
    assert np.max(np.abs(a.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-8
    scale = np.sqrt(np.diag(K))
    assert np.linalg.norm((a.c - j.c) * scale) <= 1e-8 * np.linalg.norm(j.c * scale)
    assert np.max(np.abs(a.A.T @ K @ a.A - np.eye(m))) <= 1e-9


def _steps(p, m, lam, seed, mode):
    """Steps of each of eight solves, as planned and (from launches of one solve each, which know no
    previous gap) without; the answer after them and the Jacobi solver's."""
    from paper_2302_05865_amd import FlagAggregator
    announce("steps", p, m, lam, seed, mode)
    G = torch.from_numpy(grads_of(p, seed).astype(np.float32)).cuda()
    a = 4.0 if mode == "exponent" else 2.0
    agg, ref = (FlagAggregator(n_max=256, p_max=64, exponent_a=a, solver=s) for s in ("auto", "jacobi"))

    def call(ctx, iters):
        if mode == "blocks":
            ctx.fa_aggregate_grouped(G, [1] * p, m, lam, iters, 0.0)
        else:
            ctx.fa_aggregate(G, m, lam, iters, 0.0)
        return ctx.fa_get_info()

    steps, plain, before = [], [], 0
    for iters in range(1, 9):
        info = call(agg, iters)
        steps.append(info.sweeps - before)
        before = info.sweeps
        agg.fa_aggregate_restream(G, m, lam, iters)
        plain.append(agg.fa_get_info().sweeps)
    j = call(ref, 8)
    # projectors good to eps p / gap and the relative gap at m above 1e-7 throughout
    assert info.status == 0 and j.status == 0 and info.rank == j.rank and info.sweeps != j.sweeps
    assert np.max(np.abs(info.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-7
    scale = np.sqrt(np.diag(j.K))
    assert np.linalg.norm((info.c - j.c) * scale) <= 1e-7 * np.linalg.norm(j.c * scale)
    agg.close()
    ref.close()
    return np.array(steps), np.array(plain)


# a gap that closes in or opens up; ends beyond the last solve's folds; the second solve's gap elsewhere
@pytest.mark.parametrize("p,m,lam,seed,mode", [
    (54, 1, 0.0, 759667580, "exponent"), (48, 47, 1.0, 5, "plain"), (48, 47, 1.0, 5, "blocks"),
    (17, 16, 1.0, 1, "plain"), (64, 63, 4.0, 8, "plain"), (21, 20, 4.0, 614711476, "plain"),
    (17, 5, 0.1, 636078391, "plain"), (27, 6, 0.1, 604592858, "blocks"), (23, 8, 0.0, 515711975, "exponent"),
    (18, 2, 0.0, 981457606, "plain")])
def test_planned_steps_cost_no_more_than_plain_ones(p, m, lam, seed, mode):
    """Rounding moves a solve by a step or so; 10 % covers that and the last check of a plan."""
    steps, plain = _steps(p, m, lam, seed, mode)
    assert steps.sum() <= 1.1 * plain.sum(), (steps, plain)


@pytest.mark.parametrize("p,m,lam,seed", [(17, 5, 0.1, 636078391), (27, 6, 0.1, 604592858),
                                          (23, 8, 0.0, 515711975), (17, 5, 0.1, 403139253)])
@pytest.mark.parametrize("mode", ["plain", "blocks"])
def test_planned_steps_are_taken_and_fewer(p, m, lam, seed, mode):
    steps, plain = _steps(p, m, lam, seed, mode)
    assert np.all(np.abs(steps[:2] - plain[:2]) <= 1)                 # no guess yet
    assert steps[2:].sum() <= 0.9 * plain[2:].sum(), (steps, plain)


@pytest.mark.parametrize("p,m,lam,seed,mode", [
    (25, 23, 0.0, 195971021, "plain"), (31, 30, 0.1, 926618490, "plain"), (27, 24, 0.0, 822271859, "plain"),
    (17, 14, 0.0, 574192913, "blocks"), (31, 28, 0.0, 1042215544, "blocks"),
    (64, 62, 0.0, 233228967, "exponent"), (37, 36, 0.0, 172104776, "exponent"),
    (25, 21, 4.0, 611524802, "exponent")])
def test_a_guess_that_fails_costs_one_more_solve(p, m, lam, seed, mode):
    """The third solve's gap is not near the second's: that solve takes its plain steps and the
    planned ones before them, and is over well before the 64 steps after which a guess is dropped."""
    steps, plain = _steps(p, m, lam, seed, mode)
    assert 12 <= steps[2] - plain[2] <= 45, (steps, plain)
    assert np.all(steps[3:] <= plain[3:] + 10), (steps, plain)


@pytest.mark.parametrize("p,m,lam,iters,seed,a", [
    (59, 55, 1.0, 14, 954815241, 2.0), (51, 47, 0.1, 14, 801768823, 2.0), (59, 57, 0.1, 14, 636697993, 4.0),
    (26, 22, 4.0, 9, 556645660, 2.0)])
def test_long_plans_keep_the_projector_symmetric(p, m, lam, iters, seed, a):
    """Eigenvalues m and m + 1 at 1e-7 of the trace: up to forty planned steps with no square among
    them, so whatever is not symmetric in X_0 meets the maps' linear coefficients only (product 1e13
    here; the objective was wrong by 6e-4 in the first case).  Workers with two gradients.  Both
    projectors are good to eps p / gap, 1e-15 * 64 / 5e-8 = 1e-6 at worst in a single vector pair;
    weights and coefficients see its square and its product with a small component."""
    from paper_2302_05865_amd import FlagAggregator
    announce("long plans", p, m, lam, iters, seed, a)
    G = torch.from_numpy(grads_of(p, seed).astype(np.float32)).cuda()
    got = []
    for solver in ("auto", "jacobi"):
        agg = FlagAggregator(n_max=256, p_max=64, exponent_a=a, solver=solver)
        agg.fa_aggregate_grouped(G, [2] * (p // 2) + [1] * (p % 2), m, lam, iters, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    x, j = got
    assert x.status == 0 and j.status == 0 and x.sweeps != j.sweeps
    scale = np.sqrt(np.diag(j.K))
    assert np.max(np.abs(x.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-9
    assert np.linalg.norm((x.c - j.c) * scale) <= 2e-9 * np.linalg.norm(j.c * scale)
    assert np.max(np.abs(x.A.T @ x.K @ x.A - np.eye(m))) <= 1e-9


def _with_copies(p, rank, seed):
    """Gram matrix of `rank` gradients and p - rank exact copies of them."""
    r = np.random.default_rng(seed)
    G = r.standard_normal((rank, 200)) * 0.5 + r.standard_normal((1, 200))
    G = G[np.concatenate([np.arange(rank), r.integers(0, rank, p - rank)])[r.permutation(p)]]
    return G @ G.T


@pytest.mark.parametrize("p,rank", [(p, p) for p in (17, 20, 21, 24, 25, 28, 29, 32, 33, 37, 41, 45, 48, 49, 53,
                                                    57, 61, 64)] +
                         [(20, 16), (32, 7), (40, 32), (48, 20), (64, 48), (64, 33), (60, 61 - 16)])
def test_every_remainder_of_the_last_tile(p, rank):
    """A product stops at the rank: one to four matrix instructions of the last tile, or none of it
    needed.  Against the Jacobi solver from the same K: projectors good to eps p / gap with gaps above
    1e-5, so 1e-8 on the objective and the aggregate (copies' coefficients are not unique, K c is)."""
    from paper_2302_05865_amd import FlagAggregator
    announce("last tile", p, rank)
    K = _with_copies(p, rank, 5 * p + rank)
    m, got = (rank + 2) // 2, []
    for solver in ("auto", "jacobi"):
        agg = FlagAggregator(n_max=1 << 20, p_max=64, solver=solver)
        agg.fa_irls(K, m, 0.5, 6, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    a, j = got
    assert a.status == 0 and j.status == 0 and a.rank == j.rank == rank and a.sweeps != j.sweeps
    assert np.max(np.abs(a.objective - j.objective) / (1.0 + np.abs(j.objective))) <= 1e-8
    scale = np.sqrt(np.diag(K))
    assert np.linalg.norm(K @ (a.c - j.c) / scale) <= 1e-8 * np.linalg.norm(K @ j.c / scale)
