"""A rank threshold above every pivot."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [3, 7, 12, 15, 20, 60])
def test_a_rank_threshold_above_every_pivot_leaves_nothing(p):
    """rank_tol >= 1: no pivot is large enough, rank 0, an empty subspace and a zero aggregate.  Behind a pass over
    NaN gradients, which leaves them in the compute units' LDS: what the solver uses it has to write."""
    from paper_2302_05865_amd import FlagAggregator
    announce("rank 0", p)
    n = 1 << 22
    G = np.random.default_rng(p).standard_normal((p, 50))
    passes = FlagAggregator(n_max=n, p_max=16)
    agg = FlagAggregator(n_max=1 << 20, p_max=64, rank_tol=2.0)
    passes.fa_gram(torch.full((16, n), float("nan"), device="cuda"))
    agg.fa_irls(G @ G.T, 3, 1.0, 4, 0.0)
    x = agg.fa_get_info()
    agg.close()
    passes.close()
    assert x.status == 0 and x.rank == 0 and np.all(x.c == 0) and np.all(x.A == 0)
