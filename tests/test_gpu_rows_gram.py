"""The fp64 Gram pass over interleaved storage, at the edges of its tiles, pitches and types."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(1, 16), (5, 5), (15, 16), (16, 16), (17, 17), (17, 32), (23, 23),
                                     (32, 32), (33, 48), (47, 47), (48, 48), (49, 64), (63, 63),
                                     (64, 64)])
def test_interleaved_gram_matches_worker_major(p, pitch, dtype):
    """Same tiles, same order of rows and sums as over worker-major storage: the same bits, whatever
    the pitch; the places between the rows hold NaN and reach nothing.  Sizes around one tile
    (64 rows fp32, 128 bf16) and around one round of all wavefronts of the widest tiling."""
    from paper_2302_05865_amd import FlagAggregator
    announce("interleaved gram", p, pitch, dtype)
    for n in (1, 63, 64, 65, 127, 129, 2049, 262_145 if p == 17 else 20_003):
        x = si.random_dense(p, n, seed=p + n)
        if dtype == "bf16":
            x = si.f32_to_bf16_bits(x)
        by_worker = to_device(x)
        rows = torch.full((n, pitch), float("nan"), dtype=by_worker.dtype, device="cuda")
        rows[:, :p] = by_worker.t()
        a = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout="row_major")
        b = FlagAggregator(n_max=n, p_max=p, dtype=dtype, gram="fp64")
        K, W = a.fa_gram(rows[:, :p]), b.fa_gram(by_worker)
        assert np.all(np.isfinite(K)) and np.array_equal(K, W), n
        a.close()
        b.close()
