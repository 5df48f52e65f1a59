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


@pytest.mark.parametrize("p,n,dtype", [
    *((p, 20_011, d) for p in (17, 18, 33, 64) for d in ("f32", "bf16")),
    *((p, (1 << 22) + 20_011, d) for p in (18, 33, 34) for d in ("f32", "bf16")),
    (50, (1 << 22) + 20_011, "bf16"), (64, (1 << 22) + 20_011, "bf16")])
def test_gram_from_pieces_in_any_order(p, n, dtype):
    """p > 16.  Small pieces: the pairs of all but one gradient, then the last one's row.  A first
    piece of 2^22 rows or more: the pairs of the first gradients ahead of the others', of all but one
    at once where one of the first is the last or the last but one to hold the rows.  Whole
    gradients and pieces in random order, one worker far behind with its later pieces, pieces of
    eight rows and of many tiles.  fp64 sums as above, in blocks."""
    from paper_2302_05865_amd import FlagAggregator
    announce("gram from pieces: orders", p, n, dtype)
    gen = torch.Generator(device="cuda").manual_seed(p)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    pitch = (n + 7) // 8 * 8
    full = torch.zeros((p, pitch), dtype=tdt, device="cuda")
    for i in range(p):
        full[i, :n] = torch.randn(n, generator=gen, device="cuda").to(tdt)
    ref = np.zeros((p, p))
    for a in range(0, n, 1 << 20):
        x = full[:, a:min(a + (1 << 20), n)].to(torch.float64)
        ref += (x @ x.t().contiguous()).cpu().numpy()
    scale = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    buf = torch.empty_like(full)
    agg = FlagAggregator(n_max=n, p_max=p, dtype=dtype)
    r = np.random.default_rng(p)
    base = n - 20_011
    cuts = [0, base + 4096, base + 4104, base + 16_384, n]
    pieces = list(zip(cuts, cuts[1:]))
    for kind in ("whole", "pieces", "straggler", "mixed"):
        todo = {i: [(0, n)] if kind == "whole" or (kind == "mixed" and i % 3 == 0) else pieces[:]
                for i in range(p)}
        behind = int(r.integers(p)) if kind == "straggler" else -1
        buf.fill_(float("nan"))
        agg.fa_gram_begin(p, n)
        started = False
        while any(todo.values()):
            ready = [i for i in todo if todo[i]]
            # the one behind lands its first piece at once, the others when all are done
            if behind in ready and len(ready) > 1 and started:
                ready.remove(behind)
            i = behind if behind in ready and not started else int(r.choice(ready))
            started = True
            a, b = todo[i].pop(0)
            held = [n if not todo[j] else todo[j][0][0] for j in range(p) if j != i]
            for e in sorted({h for h in held if a < h < b} | {b}):   # cut where others' rows end
                buf[i, a:e] = full[i, a:e]
                agg.fa_gram_update_rows(buf[:, :n], i, a, e - a)
                a = e
        agg.fa_aggregate_arrived(buf[:, :n], p // 2, 1.0, 1, 0.0)
        K = agg.fa_get_info().K
        assert np.max(np.abs(K - ref) / scale) <= 1e-12, kind
        assert np.array_equal(K, K.T)
    agg.close()
