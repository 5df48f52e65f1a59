"""The fp64 Gram pass where the last block of columns, or all there is, is narrow."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["worker_major", "row_major"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 17, 18, 20, 21, 24, 25, 33, 36, 37, 40, 41, 49, 52, 53, 56, 57])
def test_narrow_gram(p, dtype, layout):
    """At most eight columns, at most four and at most eight in the last block and one more, at a tile's edges (64 rows
    fp32, 128 bf16) and with more than a round of all wavefronts.  fp64 products of fp32 values are exact; two orders of
    summing n of them differ by at most n eps of the sums of magnitudes (6e-11 at 262 209 rows) and, rounding at random, by
    some sqrt(n) eps (1e-13), which is what is seen: 2e-12 up to 300 thousand rows and in proportion beyond, below the bound from
    ten thousand rows on.  Identical gradients have identical rows."""
    from paper_2302_05865_amd import FlagAggregator
    announce("narrow gram", p, dtype, layout)
    for n in (1, 63, 64, 127, 128, 129, 2049, 262_145 + 64, (1 << 22) + 5 if p in (5, 8) else 1000):
        x = si.random_dense(p, n, seed=p + n)
        if p > 2:
            x[p - 1] = x[1]
        if dtype == "bf16":
            x = si.f32_to_bf16_bits(x)
        dev = to_device(x)
        agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout=layout, gram="fp64")
        K = agg.fa_gram(dev if layout == "worker_major" else torch.empty((n, p), dtype=dev.dtype, device="cuda").copy_(dev.t()))
        agg.close()
        y = dev.double()
        want, mag = (y @ y.t().contiguous()).cpu().numpy(), (y.abs() @ y.abs().t().contiguous()).cpu().numpy()
        assert np.array_equal(K, K.T), n
        assert np.all(np.abs(K - want) <= 2e-12 * mag * max(1.0, n / 300_000)), n
        if p > 2:
            assert np.array_equal(K[1, :1], K[p - 1, :1]) and K[1, 1] == K[p - 1, p - 1] == K[1, p - 1], n
