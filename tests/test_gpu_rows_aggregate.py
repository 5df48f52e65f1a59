"""The aggregate pass over interleaved storage, at the edges of its tiles, pitches, types and batches."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(p, pitch, n, dtype, rng):
    """The places between the rows hold NaN and reach nothing; fp64 sums of exact values, one fp32 rounding of the
    result (2^-24 of it, and of the sum of magnitudes at most p 2^-53 from the order of the additions)."""
    from paper_2302_05865_amd import FlagAggregator
    gen = torch.Generator(device="cuda").manual_seed(p + n % 1013)
    rows = torch.full((n, pitch), float("nan"), device="cuda",
                      dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    step = 1 << 20
    for a in range(0, n, step):
        k = min(step, n - a)
        rows[a:a + k, :p] = torch.randn((k, p), generator=gen, device="cuda").to(rows.dtype)
    c = rng.standard_normal(p)
    agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout="row_major")
    out = torch.full((n + 8,), float("nan"), device="cuda")
    agg.fa_combine(rows[:, :p], c, out[:n])
    agg.close()
    assert torch.isnan(out[n:]).all()
    cd = torch.from_numpy(c).cuda()
    for a in range(0, n, step):
        x = rows[a:min(a + step, n), :p].double()
        want, mag = x @ cd, x.abs() @ cd.abs()
        lim = 2.0 ** -24 * 1.0001 * want.abs() + p * 2.0 ** -53 * mag + 1e-45
        assert bool(((out[a:a + x.shape[0]].double() - want).abs() <= lim).all()), (p, pitch, n, a)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(1, 1), (1, 16), (3, 3), (4, 4), (5, 5), (7, 8), (8, 8), (9, 12), (15, 15), (15, 16),
                                     (16, 16), (17, 17), (20, 20), (21, 24), (23, 23), (24, 24), (28, 28), (31, 32),
                                     (32, 32), (33, 33), (40, 40), (41, 47), (48, 48), (49, 49), (52, 56), (57, 57),
                                     (63, 64), (64, 64)])
def test_rows_around_a_tile(p, pitch, dtype):
    """Rows of whole 16-byte pieces and others, every number of loads a tile; a row, a tile, one short and one over,
    less than a round of all wavefronts and a few rounds."""
    announce("rows aggregate", p, pitch, dtype)
    rng = np.random.default_rng(p)
    for n in (1, 63, 64, 65, 255, 1000, 300_007):
        _check(p, pitch, n, dtype, rng)


@pytest.mark.parametrize("dtype,p,wgs,held", [("f32", 10, 3, 48), ("f32", 12, 3, 64), ("f32", 16, 3, 64), ("f32", 20, 3, 64),
                                              ("f32", 24, 2, 64), ("f32", 37, 2, 64), ("bf16", 17, 4, 32), ("bf16", 32, 4, 32),
                                              ("bf16", 33, 4, 32), ("bf16", 47, 3, 64)])
def test_rows_around_a_batch(p, wgs, held, dtype):
    """The outputs a wavefront holds back (wgs workgroups of four a compute unit, held tiles of 64 rows): one tile
    short of all, all, and one row more (for bf16 rows of 49 to 80 bytes the line to three workgroups, in any case)."""
    announce("rows aggregate, batches", dtype, p, wgs, held)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    full = units * wgs * 4 * 64 * held
    rng = np.random.default_rng(p)
    for n in (full - 64, full, full + 1):
        _check(p, p, n, dtype, rng)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(1, 1), (2, 2), (3, 3), (5, 6), (7, 7), (8, 8), (13, 13), (16, 16), (19, 20), (33, 33),
                                     (10, 10), (15, 15), (20, 20), (30, 30), (29, 30), (60, 60), (58, 60),
                                     (40, 40), (55, 64), (61, 61), (64, 64)])
def test_rows_past_the_last_tile(p, pitch, dtype):
    """One to 63 rows past the whole tiles, with none, one and several of these: whole 16-byte pieces, less than one, and one
    that the last row ends in.  What lies behind the last row is NaN and reaches nothing."""
    from paper_2302_05865_amd import FlagAggregator
    announce("rows aggregate, ragged tile", p, pitch, dtype)
    rng = np.random.default_rng(p)
    gen = torch.Generator(device="cuda").manual_seed(p)
    agg = FlagAggregator(n_max=1 << 12, p_max=p, dtype=dtype, layout="row_major")
    c = rng.standard_normal(p)
    cd = torch.from_numpy(c).cuda()
    for n in [64 * k + r for k in (0, 1, 5) for r in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63)]:
        rows = torch.full((n + 64, pitch), float("nan"), device="cuda",
                          dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
        rows[:n, :p] = torch.randn((n, p), generator=gen, device="cuda").to(rows.dtype)
        out = torch.full((n + 8,), float("nan"), device="cuda")
        agg.fa_combine(rows[:n, :p], c, out[:n])
        assert torch.isnan(out[n:]).all()
        x = rows[:n, :p].double()
        lim = 2.0 ** -24 * 1.0001 * (x @ cd).abs() + p * 2.0 ** -53 * (x.abs() @ cd.abs()) + 1e-45
        assert bool(((out[:n].double() - x @ cd).abs() <= lim).all()), n
    agg.close()


def test_rows_past_the_last_tile_take_no_longer():
    """A set a few rows short of whole tiles takes as long as one that is not (the dispatch alone, the shortest of many);
    a ragged tile read one KiB after the other took 1.6 of it."""
    from paper_2302_05865_amd import FlagAggregator
    announce("rows aggregate, time of a ragged tile")
    sets = [torch.randn((n, 64), device="cuda") for n in (30_016, 30_001)]
    agg = FlagAggregator(n_max=30_016, p_max=64, dtype="f32", layout="row_major")
    agg.fa_set_profiling(True)
    best = [1e9, 1e9]
    for _ in range(40):
        for k, G in enumerate(sets):
            agg.fa_aggregate(G, 2, 1.0, 1, 0.0)
            best[k] = min(best[k], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[1] <= 1.25 * best[0], best


def test_rows_of_many_batches_take_no_longer():
    """Thirty million rows against six (the dispatch alone, the shortest of many): 5.1 of the time; with shorter batches of more
    workgroups 5.7."""
    from paper_2302_05865_amd import FlagAggregator
    announce("rows aggregate, time of many batches")
    G = torch.empty((30_000_000, 16), device="cuda")
    for a in range(0, 30_000_000, 3_000_000):
        G[a:a + 3_000_000].normal_()
    agg = FlagAggregator(n_max=30_000_000, p_max=16, dtype="f32", layout="row_major")
    agg.fa_set_profiling(True)
    best = {6_000_000: 1e9, 30_000_000: 1e9}
    for _ in range(15):
        for n in best:
            agg.fa_aggregate(G[:n], 2, 1.0, 1, 0.0)
            best[n] = min(best[n], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[30_000_000] <= 5.4 * best[6_000_000], best


def test_rows_of_thirty_take_no_longer_than_of_thirty_two():
    """The dispatch alone, the shortest of many: 0.9 of the time; with the rows on one bank of LDS 1.4."""
    from paper_2302_05865_amd import FlagAggregator
    announce("rows aggregate, time of rows of 60 bytes")
    sets = [torch.randn((1_000_000, p), device="cuda").to(torch.bfloat16) for p in (32, 30)]
    agg = FlagAggregator(n_max=1_000_000, p_max=32, dtype="bf16", layout="row_major")
    agg.fa_set_profiling(True)
    best = [1e9, 1e9]
    for _ in range(25):
        for k, G in enumerate(sets):
            agg.fa_aggregate(G, 2, 1.0, 1, 0.0)
            best[k] = min(best[k], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[1] <= 1.15 * best[0], best
