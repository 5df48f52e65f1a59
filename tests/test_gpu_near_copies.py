"""Workers that send nearly the same vector, as colluding ones do.  A pair adds to the trace of the
weighted-PCA matrix M its weight times |r_i - r_j|^2 / D_ij^2, and that ratio is 1 only while
R^T R is the Gram matrix to the accuracy of D_ij^2.  With entries good to 1e-10, as the
bf16 matrix core makes them, the factorisation of near copies stops short and the ratio is
anything up to hundreds: the purification has to be scaled by the trace of M itself.  Scaled by the weights' sum, 17 of
the 25 chosen matrices ended in the stand-by and 5 on another projector than the leading one."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device
from near_copies import irls, near_copies

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


STAND_BY = ("jacobi16", "jacobi")       # what a purification that fails is handed to, p <= 16 and above


def compare(x, j, K, m, lam, iters):
    """x: the library's info, j: the Jacobi solver's of the same K (which only says that x is not its answer).
    R's last rows are good to eps / D^2, M's entries to that times their size, projectors to that over the gap;
    a factor 4 p for the sums.  An answer that is not the leading projector is off by 1.4."""
    assert x.status == 0 and x.iters_done == iters
    assert x.sweeps != j.sweeps, "the stand-by's answer"
    objective, R, P, gap, near, _ = irls(K, m, lam, iters)
    bound = 4 * len(K) * 2.3e-16 / near / gap
    assert bound < 0.05, "not a test"
    U = R @ x.A
    got = [np.max(np.abs(x.objective - objective) / objective), np.linalg.norm(U @ U.T - P),
           np.max(np.abs(U.T @ U - np.eye(m)))]
    print(x.rank, x.sweeps, "gap %.1e" % gap, "bound %.1e" % bound, ["%.1e" % g for g in got])
    assert x.rank == len(R)
    assert got[0] <= bound and got[1] <= bound and got[2] <= bound


# in each of these trace M is 1.5 to 9 times the sum of the weights in one of the five solves at least
WIDE = [(20, 2, 4.0, 15, 1e-10), (20, 2, 4.0, 18, 1e-10), (20, 2, 1.0, 36, 1e-10), (20, 2, 4.0, 37, 5e-10),
        (20, 2, 1.0, 38, 5e-10), (20, 2, 4.0, 39, 5e-10), (42, 1, 1.0, 3, 5e-10), (42, 1, 4.0, 8, 1e-10),
        (42, 1, 4.0, 11, 5e-10), (42, 1, 1.0, 19, 1e-10), (60, 2, 4.0, 202, 5e-10), (60, 2, 1.0, 358, 5e-10),
        (60, 2, 1.0, 460, 5e-10), (60, 2, 1.0, 468, 5e-10)]
NARROW = [(7, 4, 4.0, 2, 1e-10), (7, 2, 4.0, 2, 5e-10), (7, 2, 4.0, 12, 1e-10), (7, 2, 4.0, 20, 1e-10),
          (7, 4, 4.0, 20, 5e-10), (15, 2, 4.0, 4, 5e-10), (15, 2, 4.0, 6, 5e-10), (15, 2, 4.0, 12, 5e-10),
          (15, 2, 4.0, 16, 5e-10), (15, 2, 4.0, 18, 1e-10), (15, 2, 4.0, 21, 1e-10)]


@pytest.mark.parametrize("p,m,lam,seed,noise", WIDE + NARROW)
def test_the_purification_is_scaled_by_the_trace_itself(p, m, lam, seed, noise):
    from paper_2302_05865_amd import FlagAggregator
    announce("near copies", p, m, lam, seed, noise)
    K, got = near_copies(p, max(3, p // 3), 4e-6, 400, seed, noise), []
    for solver in ("auto", STAND_BY[p > 16]):
        agg = FlagAggregator(n_max=1 << 20, p_max=64, solver=solver)
        agg.fa_irls(K, m, lam, 5, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    compare(*got, K, m, lam, 5)


# (a = 4 at p >= 40 with lambda = 1 has gaps of 1e-6, where the bound says nothing)
@pytest.mark.parametrize("p,blocks,a,lam", [(p, k, 2.0, lam) for lam in (1.0, 100.0) for p, k in (
    (8, 1), (16, 1), (20, 1), (40, 1), (60, 1), (10, 2), (20, 2), (40, 4), (60, 2))] + [
    (16, 1, 4.0, 1.0), (20, 1, 4.0, 1.0), (20, 1, 4.0, 100.0), (40, 1, 4.0, 100.0), (60, 1, 4.0, 100.0), (60, 2, 4.0, 100.0)])
def test_close_pairs_of_an_exact_matrix_against_the_jacobi_solver(p, blocks, a, lam):
    """K in fp64: every gradient has a pivot, and pairs closer than the solver lets the weights stand for the
    trace.  Every tile count of every mode.  The same K in front of both solvers; bounds as above."""
    from paper_2302_05865_amd import FlagAggregator
    announce("close pairs", p, blocks, a, lam)
    n, m, r = 400, 5 if p > 10 else 3, np.random.default_rng(p + blocks)
    G = (r.standard_normal((p, n)) * 0.5 + r.standard_normal((1, n))).astype(np.float32)
    copies = r.permutation(p // blocks)[:max(2, p // blocks // 3)]
    for b in range(blocks):
        v = np.float32(r.standard_normal(n))
        for i in copies:
            G[i * blocks + b] = v + np.float32(5e-4) * np.float32(r.standard_normal(n))
    G, got = to_device(G), []
    for solver in ("auto", STAND_BY[p > 16 or blocks > 1]):
        agg = FlagAggregator(n_max=n, p_max=64, exponent_a=a, solver=solver)
        if blocks > 1:
            agg.fa_aggregate_grouped(G, [blocks] * (p // blocks), m, lam, 5, 0.0)
        else:
            agg.fa_aggregate(G, m, lam, 5, 0.0)
        got.append(agg.fa_get_info())
        agg.close()
    x, j = got
    s = np.diag(x.K)
    both = s[:, None] + s[None]
    near = np.min(((both - 2 * x.K) / both)[~np.eye(p, dtype=bool)])
    bound = 4 * p * 2.3e-16 / near / j.eigengap
    agree = [np.max(np.abs(x.objective - j.objective) / j.objective),
             np.linalg.norm(x.K @ (x.c - j.c) / np.sqrt(s)) / np.linalg.norm(x.K @ j.c / np.sqrt(s))]
    print(p, blocks, lam, x.rank, j.rank, x.sweeps, "near %.1e gap %.1e bound %.1e" % (near, j.eigengap, bound),
          ["%.1e" % g for g in agree])
    assert x.status == 0 and j.status == 0 and x.sweeps != j.sweeps and x.rank == j.rank == p
    assert near < 1e-6 and max(agree) <= bound < 0.1


@pytest.mark.parametrize("p,dtype", [(20, "f32"), (42, "f32"), (60, "f32"), (15, "bf16"), (24, "bf16")])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_colluding_workers_take_the_fast_route(p, dtype, seed):
    """The Gram matrix from the bf16 matrix core.  fp32: a third of the workers within 1e-6..8e-6 of one vector;
    bf16: copies of one with a few coordinates one unit in the last place off."""
    from paper_2302_05865_amd import FlagAggregator
    announce("colluding", p, dtype, seed)
    n, r = 1 << 20, np.random.default_rng(100 * p + seed)
    x = (r.standard_normal((p, n), dtype=np.float32) * 0.5 + r.standard_normal((1, n), dtype=np.float32))
    v = r.standard_normal(n, dtype=np.float32)
    x = x if dtype == "f32" else si.f32_to_bf16_bits(x)
    for i in r.permutation(p)[:p // 3]:
        if dtype == "f32":
            x[i] = v + np.float32(4e-6 * r.uniform(0.3, 2)) * r.standard_normal(n, dtype=np.float32)
        else:
            x[i] = si.f32_to_bf16_bits(v[None])[0]
            x[i, r.integers(0, n, r.integers(3, 60))] ^= 1
    G = to_device(x)
    for m in (2, 5):
        agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype)
        agg.fa_aggregate(G, m, 1.0, 5, 0.0)
        a = agg.fa_get_info()
        agg.close()
        ref = FlagAggregator(n_max=n, p_max=p, dtype=dtype, solver=STAND_BY[p > 16])
        ref.fa_irls(a.K, m, 1.0, 5, 0.0)
        j = ref.fa_get_info()
        ref.close()
        assert a.status == 0 and a.sweeps != j.sweeps, m
        objective, R, P, gap, near, _ = irls(a.K, m, 1.0, 5)
        U, bound = R @ a.A, 4 * p * 2.3e-16 / near
        got = np.max(np.abs(U.T @ U - np.eye(m))), np.linalg.norm(U @ U.T - P)
        print(p, dtype, m, a.rank, a.sweeps, "gap %.1e" % gap, "bound %.1e" % bound, ["%.1e" % g for g in got])
        assert a.rank == len(R) and got[0] <= bound
        assert got[1] <= bound / gap or bound / gap > 0.05
