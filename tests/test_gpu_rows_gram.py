"""The fp64 Gram pass over interleaved storage, at the edges of its tiles, pitches and types."""
import numpy as np
import pytest

import synth_inputs as si
from gpu_util import announce, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(1, 16), (5, 5), (15, 16), (16, 16), (17, 17), (17, 32), (23, 23),
                                     (32, 32), (33, 48), (47, 47), (48, 48), (49, 49), (49, 64), (50, 52), (53, 60),
                                     (56, 56), (63, 63), (64, 64)])
def test_interleaved_gram_matches_worker_major(p, pitch, dtype):
    """Same tiles, same order of rows and sums as over worker-major storage: the same bits, whatever
    the pitch; the places between the rows hold NaN and reach nothing.  Sizes around one tile
    (64 rows fp32, 128 bf16) and less than a round of all wavefronts."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch,waves", [(9, 9, 12), (15, 16, 12), (17, 17, 16), (30, 32, 16),
                                           (33, 33, 8), (45, 48, 8), (49, 49, 8), (51, 51, 8), (56, 58, 8), (64, 64, 8)])
def test_interleaved_gram_in_its_steady_state(p, pitch, waves, dtype):
    """Two rounds of all wavefronts and a ragged tail: every wavefront has a full tile in LDS while the
    next full one is on its way to its registers, some have a third and one the ragged one (waves: per
    compute unit, of that width's tiling)."""
    from paper_2302_05865_amd import FlagAggregator
    announce("interleaved gram, rounds", p, pitch, dtype)
    tile = 64 if dtype == "f32" else 128
    units = torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device="cuda").manual_seed(p)
    for n in (2 * units * waves * tile, 2 * units * waves * tile + 5 * tile + 3):
        by_worker = torch.zeros((p, -(-n // 8) * 8), device="cuda",
                                dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
        by_worker[:, :n] = torch.randn((p, n), generator=gen, device="cuda")
        rows = torch.full((n, pitch), float("nan"), dtype=by_worker.dtype, device="cuda")
        rows[:, :p] = by_worker[:, :n].t()
        a = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout="row_major")
        b = FlagAggregator(n_max=n, p_max=p, dtype=dtype, gram="fp64")
        K, W = a.fa_gram(rows[:, :p]), b.fa_gram(by_worker[:, :n])
        assert np.all(np.isfinite(K)) and np.array_equal(K, W), n
        a.close()
        b.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(1, 1), (1, 16), (4, 4), (7, 9), (11, 11), (15, 16), (16, 16)])
def test_interleaved_gram_of_many_rows(p, pitch, dtype):
    """p <= 16 from 2^22 rows on: elements scattered to their columns on the way into LDS.  A last tile
    of one row, of all rows but one and none; one row below the rule's line."""
    from paper_2302_05865_amd import FlagAggregator
    announce("interleaved gram, many rows", p, pitch, dtype)
    gen = torch.Generator(device="cuda").manual_seed(p)
    for n in ((1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 22) + 127):
        by_worker = torch.zeros((p, -(-n // 8) * 8), device="cuda",
                                dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
        by_worker[:, :n] = torch.randn((p, n), generator=gen, device="cuda")
        rows = torch.full((n, pitch), float("nan"), dtype=by_worker.dtype, device="cuda")
        rows[:, :p] = by_worker[:, :n].t()
        a = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout="row_major")
        b = FlagAggregator(n_max=n, p_max=p, dtype=dtype, gram="fp64")
        K, W = a.fa_gram(rows[:, :p]), b.fa_gram(by_worker[:, :n])
        assert np.all(np.isfinite(K)) and np.array_equal(K, W), n
        a.close()
        b.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,pitch", [(17, 18), (19, 31), (20, 20), (20, 32), (21, 21), (24, 24), (24, 31), (25, 25),
                                     (33, 33), (36, 36), (37, 48), (40, 40), (41, 41), (50, 50), (52, 64), (53, 53),
                                     (56, 56), (57, 57)])
def test_interleaved_gram_with_a_narrow_last_block(p, pitch, dtype):
    """At most four, at most eight and more columns in the last block of sixteen, full and not, a tile's edge and
    a round of all wavefronts.  fp64 products of fp32 values are exact; the sums differ from numpy's by at
    most n eps of the sums of magnitudes, 2e-12 here."""
    from paper_2302_05865_amd import FlagAggregator
    announce("interleaved gram, narrow last block", p, pitch, dtype)
    for n in (1, 65, 2049, 262_145 + 64):
        x = si.random_dense(p, n, seed=p + n)
        if dtype == "bf16":
            x = si.f32_to_bf16_bits(x)
        by_worker = to_device(x)
        rows = torch.full((n, pitch), float("nan"), dtype=by_worker.dtype, device="cuda")
        rows[:, :p] = by_worker.t()
        a = FlagAggregator(n_max=n, p_max=p, dtype=dtype, layout="row_major")
        K = a.fa_gram(rows[:, :p])
        a.close()
        y = by_worker.double().cpu().numpy()
        assert np.all(np.abs(K - y @ y.T) <= 2e-12 * (np.abs(y) @ np.abs(y).T)), n
