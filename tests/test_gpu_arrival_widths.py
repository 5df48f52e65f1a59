"""The Gram matrix built from pieces, at the widths where the passes behind it change."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 15, 16, 17, 18, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gram_from_pieces_at_every_width_class(p, dtype):
    """p <= 16: one pass over a piece once everybody holds it.  p > 16: one over all but the
    missing gradient (first, middle or last place), then that one's row.  Unequal cuts: gradient 0
    lands whole, the others in three pieces, the last one ragged.  Places that have not landed
    hold NaN.  Products and sums are fp64: |K - K_ref| <= n * 2^-53 sum|products|, under 1e-12 of
    sqrt(K_ii K_jj) at n = 3001."""
    from paper_2302_05865_amd import FlagAggregator
    announce("gram from pieces: widths", p, dtype)
    n = 3001
    x = si.random_dense(p, n, seed=p)
    if dtype == "bf16":
        x = si.f32_to_bf16_bits(x)
        wide = np.ascontiguousarray(x.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    else:
        wide = x.astype(np.float64)
    full = to_device(x)
    buf = to_device(np.full(x.shape, 0x7FC0, np.uint16) if dtype == "bf16" else
                    np.full(x.shape, np.nan, np.float32))
    cuts = [0, 1024, 2048, n]
    agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype)
    for last in sorted({0, p // 2, p - 1}):          # whose pieces come last
        buf.fill_(float("nan"))
        agg.fa_gram_begin(p, n)
        order = [i for i in range(p) if i != last] + [last]
        for i in order:
            for a, b in ([(0, n)] if i == 0 else list(zip(cuts, cuts[1:]))):
                buf[i, a:b] = full[i, a:b]
                if i == 0 and last == 0 and p > 1:   # the whole of gradient 0 after the pieces
                    for c, d in zip(cuts, cuts[1:]):
                        agg.fa_gram_update_rows(buf, 0, c, d - c)
                else:
                    agg.fa_gram_update_rows(buf, i, a, b - a)
        agg.fa_aggregate_arrived(buf, max(1, p // 2), 1.0 if p > 1 else 0.0, 1, 0.0)
        K = agg.fa_get_info().K
        ref = wide @ wide.T
        scale = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
        assert np.max(np.abs(K - ref) / scale) <= 1e-12
        assert np.array_equal(K, K.T)
    agg.close()
