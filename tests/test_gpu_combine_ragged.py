"""The aggregate pass over worker-major columns that do not end on a 16-byte piece: the workgroup that their end is in."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p", [1, 2, 7, 8, 9, 15, 16, 17, 24, 33, 64])
def test_ragged_columns(p, dtype):
    """Every remainder of a piece, in the first piece, the first workgroup and the second; fewer columns than are in flight,
    as many, one more.  What lies behind the columns is NaN and reaches nothing.  One rounding of the result (fp32),
    (p + 2) 2^-24 of the sum of magnitudes (bf16, added in fp32)."""
    from paper_2302_05865_amd import FlagAggregator
    announce("ragged columns", p, dtype)
    per = 4 if dtype == "f32" else 8
    most = 256 * per + 3 * per
    G = torch.full((p, most + per), float("nan"), device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    values = torch.randn((p, most), generator=torch.Generator(device="cuda").manual_seed(p), device="cuda").to(G.dtype)
    c = np.random.default_rng(p).standard_normal(p)
    cd = torch.from_numpy(c).cuda()
    agg = FlagAggregator(n_max=most, p_max=p, dtype=dtype)
    for start in (0, 64 * per, 255 * per, 256 * per, 257 * per):
        for n in range(start + 1, start + per + 1):
            G[:, :n], G[:, n:] = values[:, :n], float("nan")
            out = torch.full((n + 8,), float("nan"), device="cuda")
            agg.fa_combine(G[:, :n], c, out[:n])
            assert torch.isnan(out[n:]).all()
            x = values[:, :n].double()
            lim = 2.0 ** -24 * ((cd @ x).abs() * 1.01 if dtype == "f32" else (p + 2) * (cd.abs() @ x.abs())) + 1e-30
            assert bool(((out[:n].double() - cd @ x).abs() <= lim).all()), n
    agg.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_multi_krum_ragged_columns(dtype):
    """The pass that reads the selected columns only, as above: the bits of the one that reads them all, times 0."""
    from paper_2302_05865_amd import FlagAggregator
    announce("krum, ragged columns", dtype)
    per = 4 if dtype == "f32" else 8
    gen = torch.Generator(device="cuda").manual_seed(1)
    for n in range(300 * per + 1, 301 * per + 1):
        G = torch.randn((20, 304 * per), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)[:, :n]
        agg = FlagAggregator(n_max=n, p_max=20, dtype=dtype)
        out, _, sel = agg.fa_multikrum(G, 3, 11)
        assert sel.sum() == 11 and torch.equal(out, agg.fa_combine(G, sel / 11)), n
        agg.close()


def test_ragged_columns_take_no_longer():
    """Three rows past whole pieces (the dispatch alone, the shortest of many): 1.7 of the time without them, where each of
    the 64 columns was waited for 4.3."""
    from paper_2302_05865_amd import FlagAggregator
    announce("ragged columns, time")
    G = torch.randn((64, 100_004), device="cuda")
    agg = FlagAggregator(n_max=100_003, p_max=64, dtype="f32")
    agg.fa_set_profiling(True)
    best = {100_000: 1e9, 100_003: 1e9}
    for _ in range(40):
        for n in best:
            agg.fa_aggregate(G[:, :n], 2, 1.0, 1, 0.0)
            best[n] = min(best[n], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[100_003] <= 2.5 * best[100_000], best
