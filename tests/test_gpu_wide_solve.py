"""The solver of 17..64 columns at the edges of its tiles: every remainder of four in the last one, blocks of mixed widths."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device
from oracle import as_f64_matrix, fa_literal, fa_literal_grouped

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIXED = [3, 2, 1, 5, 4, 2, 3, 1, 2, 4, 3, 3]        # 33 columns, blocks over tiles' borders


@pytest.mark.parametrize("a", [2.0, 4.0])
@pytest.mark.parametrize("sizes", [
    [1] * 17, [1] * 20, [1] * 23, [1] * 28, [1] * 32, [1] * 33, [1] * 37, [1] * 43, [1] * 48, [1] * 49, [1] * 54, [1] * 59,
    [1] * 64, [2] * 16, MIXED, MIXED + [15], [1, 31, 32], [7] * 9 + [1], [2, 3, 2, 3, 2, 5], [17, 1, 1]],
    ids=lambda s: "%dx%d" % (len(s), sum(s)))
def test_wide_solve(sizes, a):
    """Aggregate, values and objective against the fp64 definition, from the purification (the Jacobi stand-by, which would
    give the same answer, counts other steps).  The solver is fp64 throughout; the aggregate is rounded
    to fp32 (6e-8), and 1e-6 leaves the rounding of K's eigenvectors (1e-14 times a gap's inverse, here below 1e4) far below."""
    from paper_2302_05865_amd import FlagAggregator
    p, n, iters = sum(sizes), 1_203, 4
    m = max(1, p // 2)
    announce("wide solve", sizes, a)
    G = si.random_dense(p, n, seed=p + len(sizes))
    G += si.random_dense(1, n, seed=1)
    single = len(sizes) == p
    if single:
        ref = fa_literal(as_f64_matrix(G), m, 1.0, iters, 0.0, a=a)
    else:
        ref = fa_literal_grouped(as_f64_matrix(G), sizes, m, 1.0, iters, 0.0, a=a)
    dev, steps = to_device(G), {}
    for solver in ("jacobi", "auto"):
        agg = FlagAggregator(n_max=n, p_max=p, exponent_a=a, solver=solver)
        out = agg.fa_aggregate(dev, m, 1.0, iters, 0.0) if single else agg.fa_aggregate_grouped(dev, sizes, m, 1.0, iters, 0.0)
        out, info = out.cpu().numpy().astype(np.float64), agg.fa_get_info()
        agg.close()
        steps[solver] = info.sweeps
    assert info.status == 0 and info.iters_done == iters
    assert m >= info.rank or steps["auto"] != steps["jacobi"], steps
    assert np.linalg.norm(out - ref["out"]) <= 1e-6 * np.linalg.norm(ref["out"])
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    assert np.allclose(np.asarray(info.v)[first], ref["v"], rtol=0, atol=1e-6)
    # a residual near zero differs by up to 1e-16 of |g|^2 between n rows and K (blocks of one column beside wide ones get
    # there), its a-th root by up to 1e-8 or, a = 4, 1e-4; two such terms
    assert np.allclose(info.objective, ref["objective"], rtol=0, atol=1e-6 + 2.0 * 1e-16 ** (1.0 / a))
