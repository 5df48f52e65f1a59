"""The aggregate pass for large sets (outputs held back on the chip), and the passes that leave out columns."""
import numpy as np
import pytest

from gpu_util import announce

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _gradients(p, n, dtype, seed):
    per = 4 if dtype == "f32" else 8
    gen = torch.Generator(device="cuda").manual_seed(seed)
    G = torch.zeros((p, -(-n // per) * per), device="cuda",
                    dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    for i in range(p):
        G[i, :n] = torch.randn(n, generator=gen, device="cuda")
    return G[:, :n]


def _wave_tiles(dtype):
    """Rows that give every wavefront (four per compute unit) one tile."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    return units * 4 * 64 * (4 if dtype == "f32" else 8)


# ten tiles a wavefront (sixteen below ten columns) are the rule's line; a batch is 55 tiles (fp32, p <= 16),
# 103 (fp32), 28 (bf16, p <= 16) and 51 (bf16): one tile short of it, all of it, one more, and two.  280 tiles of five columns
# are batches of 55, 55, 55, 55, 56 and 4: two tiles end within six columns and the second of them is the first in registers,
# and the last place in registers is filled
@pytest.mark.parametrize("dtype,p,rounds", [
    ("f32", 5, 16), ("f32", 9, 16), ("f32", 10, 10), ("f32", 17, 10), ("bf16", 10, 10), ("bf16", 17, 10),
    ("f32", 5, 32), ("f32", 5, 55), ("f32", 5, 57), ("f32", 5, 280), ("f32", 6, 54), ("f32", 6, 55), ("f32", 7, 110),
    ("f32", 7, 112), ("f32", 9, 32), ("f32", 10, 16), ("f32", 15, 55), ("f32", 15, 56),
    ("f32", 16, 16), ("f32", 17, 16), ("f32", 17, 102), ("f32", 18, 103), ("f32", 19, 104), ("f32", 33, 16),
    ("f32", 64, 17), ("bf16", 10, 16), ("bf16", 11, 27), ("bf16", 12, 28), ("bf16", 13, 29), ("bf16", 16, 56), ("bf16", 17, 50),
    ("bf16", 23, 51), ("bf16", 32, 52), ("bf16", 47, 17), ("bf16", 64, 16)])
def test_held_aggregate_has_the_small_kernels_bits(dtype, p, rounds):
    """The same sums in the same order: pieces of the rows through the kernel for small sets give the same bits.
    Rows short of a tile, of a round of all wavefronts and none, against 64 bits as well: one rounding of
    the result (fp32), (p + 2) 2^-24 of the sum of magnitudes (bf16, added in fp32)."""
    from paper_2302_05865_amd import FlagAggregator
    announce("held aggregate", dtype, p, rounds)
    full = rounds * _wave_tiles(dtype)
    rng = np.random.default_rng(p)
    for n in (full, full + 1, full + 64 * 8 * 5 + 13):
        G = _gradients(p, n, dtype, p + n % 97)
        c = rng.standard_normal(p)
        agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype)
        out = torch.full((n + 8,), float("nan"), device="cuda")
        agg.fa_combine(G, c, out[:n])
        assert torch.isnan(out[n:]).all()
        step = 1 << 20
        for a in range(0, n, step):
            x = G[:, a:a + step]
            assert torch.equal(out[a:a + x.shape[1]], agg.fa_combine(x, c)), (n, a)
        a = max(0, n - (1 << 18))
        x, cd = G[:, a:].double(), torch.from_numpy(c).cuda()
        want, mag = cd @ x, cd.abs() @ x.abs()
        lim = 2.0 ** -24 * (want.abs() * 1.01 if dtype == "f32" else (p + 2) * mag)
        assert bool(((out[a:n].double() - want).abs() <= lim + 1e-30).all())
        agg.close()


@pytest.mark.parametrize("dtype,p,n,f,q", [
    ("f32", 5, 40_003, 1, 1), ("f32", 15, 300_007, 3, 10), ("f32", 15, 9_000_001, 3, 5), ("f32", 15, 9_000_001, 3, 10),
    ("f32", 16, 4_194_304, 2, 14), ("f32", 40, 4_200_005, 5, 12), ("f32", 40, 4_200_005, 5, 17), ("f32", 64, 70_001, 3, 1),
    ("bf16", 15, 9_000_001, 3, 11), ("bf16", 32, 9_000_007, 4, 28), ("bf16", 33, 131_073, 4, 9)])
def test_multi_krum_without_the_other_columns(dtype, p, n, f, q):
    """Columns that were not selected are not read: the bits of the pass that reads them all, times 0."""
    from paper_2302_05865_amd import FlagAggregator
    announce("krum, selected columns", dtype, p, n, f, q)
    G = _gradients(p, n, dtype, p)
    agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype)
    out, _, sel = agg.fa_multikrum(G, f, q)
    assert sel.sum() == q
    assert torch.equal(out, agg.fa_combine(G, sel / q))
    agg.close()


@pytest.mark.parametrize("n", [30_001, 9_000_001])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_multi_krum_carries_nan_and_inf_over(n, bad):
    """A NaN or an infinity in any gradient, selected or not, reaches its coordinate of the result."""
    from paper_2302_05865_amd import FlagAggregator
    announce("krum, non-finite", n, bad)
    G = _gradients(15, n, "f32", 3)
    agg = FlagAggregator(n_max=n, p_max=15, dtype="f32")
    for i in (0, 7, 14):
        x = G.clone()[:, :n]
        x = torch.nn.functional.pad(x, (0, -n % 4))[:, :n]
        x[i, n // 2] = bad
        out, _, sel = agg.fa_multikrum(x, 3, 6)
        assert not torch.isfinite(out[n // 2])
        assert torch.isfinite(out[:n // 2]).all() and torch.isfinite(out[n // 2 + 1:]).all()
    agg.close()


@pytest.mark.parametrize("dtype,p,rounds", [("f32", 5, 16), ("f32", 9, 32), ("f32", 15, 10), ("f32", 64, 16), ("bf16", 10, 10),
                                            ("bf16", 17, 10), ("bf16", 40, 16)])
def test_held_aggregate_past_the_last_tile(dtype, p, rounds):
    """One row past the whole tiles to one short of another: whole 16-byte pieces of a column, less than one, and one that
    the column ends in.  What lies behind the columns is NaN and reaches nothing."""
    from paper_2302_05865_amd import FlagAggregator
    announce("held aggregate, ragged tile", dtype, p, rounds)
    per = 4 if dtype == "f32" else 8
    full, rng = rounds * _wave_tiles(dtype), np.random.default_rng(p)
    G = _gradients(p, full + 64 * per, dtype, p)
    c = rng.standard_normal(p)
    cd = torch.from_numpy(c).cuda()
    agg = FlagAggregator(n_max=G.shape[1], p_max=p, dtype=dtype)
    for r in sorted({1, 2, 3, per - 1, per, per + 1, 2 * per + 3, 17 * per, 63 * per, 63 * per + 1, 64 * per - 1}):
        n = full + r
        kept = G[:, n:].clone()
        G[:, n:] = float("nan")
        out = torch.full((n + 8,), float("nan"), device="cuda")
        agg.fa_combine(G[:, :n], c, out[:n])
        assert torch.isnan(out[n:]).all() and torch.isfinite(out[:n]).all()
        x = G[:, full - 4096:n].double()
        lim = 2.0 ** -24 * ((cd @ x).abs() * 1.01 if dtype == "f32" else (p + 2) * (cd.abs() @ x.abs())) + 1e-30
        assert bool(((out[full - 4096:n].double() - cd @ x).abs() <= lim).all()), r
        G[:, n:] = kept
    agg.close()


def test_held_aggregate_past_the_last_tile_takes_no_longer():
    """The dispatch alone, the shortest of many: 37 pieces past the whole tiles cost 1.02 of a set without them; taken column
    by column behind everything else it was 1.16."""
    from paper_2302_05865_amd import FlagAggregator
    announce("held aggregate, time of a ragged tile")
    full = 16 * _wave_tiles("f32")
    G = _gradients(64, full + 256, "f32", 1)
    agg = FlagAggregator(n_max=full + 256, p_max=64, dtype="f32")
    agg.fa_set_profiling(True)
    best = {full: 1e9, full + 148: 1e9}
    for _ in range(25):
        for n in best:
            agg.fa_aggregate(G[:, :n], 2, 1.0, 1, 0.0)
            best[n] = min(best[n], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[full + 148] <= 1.08 * best[full], best


def test_held_aggregate_takes_no_longer_where_it_begins():
    """Just below the line of sixteen tiles that was there the kernel for small sets took 1.13 of the time it takes for a tile's
    rows more; now that both sides of it are one kernel, 0.94 to 1."""
    from paper_2302_05865_amd import FlagAggregator
    announce("held aggregate, time across its former line")
    full = 16 * _wave_tiles("f32")
    G = _gradients(64, full, "f32", 1)
    agg = FlagAggregator(n_max=full, p_max=64, dtype="f32")
    agg.fa_set_profiling(True)
    best = {full: 1e9, full - 64 * 4: 1e9}
    for _ in range(25):
        for n in best:
            agg.fa_aggregate(G[:, :n], 2, 1.0, 1, 0.0)
            best[n] = min(best[n], float(agg.fa_get_timings()[3]))
    agg.close()
    assert best[full - 64 * 4] <= 1.06 * best[full], best


@pytest.mark.parametrize("dtype,p,rounds", [("f32", 12, 10), ("f32", 20, 11), ("f32", 64, 12), ("bf16", 16, 10), ("bf16", 32, 10)])
def test_held_aggregate_beside_another_sets_solver(dtype, p, rounds):
    """Two sets in flight, a context and a stream each: the solver of one holds a compute unit whose share of the other's
    aggregate waits for it (the wide forms fit beside no solver).  Bit for bit what the calls return alone."""
    from paper_2302_05865_amd import FlagAggregator
    announce("held aggregate, two sets in flight", dtype, p, rounds)
    n = rounds * _wave_tiles(dtype) + 37
    sets = [_gradients(p, n, dtype, p + k) for k in range(2)]
    for G in sets:
        G += _gradients(1, n, dtype, 7)
    aggs = [FlagAggregator(n_max=n, p_max=p, dtype=dtype) for _ in range(2)]
    refs = [aggs[0].fa_aggregate(G, p // 2, 1.0, 8, 0.0).clone() for G in sets]
    outs, streams = [torch.empty_like(r) for r in refs], [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(3):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for i in range(6):
            with torch.cuda.stream(streams[i & 1]):
                aggs[i & 1].fa_aggregate(sets[i & 1], p // 2, 1.0, 8, 0.0, out=outs[i & 1])
        torch.cuda.synchronize()
        for k in range(2):
            assert torch.equal(outs[k], refs[k]), (rep, k)
            assert aggs[k].fa_get_info().status == 0
    for a in aggs:
        a.close()
