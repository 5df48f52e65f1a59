"""The p x p solvers take the sum of the weights for the trace of the weighted-PCA matrix M where no pair is closer than
FA_CLOSE_PAIR and either every gradient has a pivot or R^T R bears the distances out to FA_TRACE_OFF.  Here: within
1e-7 (what they scale X_0 down by) wherever that rule says so, and far from it on the inputs that it sends to
the measured trace."""
import os
import re

import numpy as np
import pytest

from near_copies import irls, near_copies

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_05865_amd", "csrc",
                      "fa_internal.h")
CLOSE, OFF = (float(re.search(rf"#define {name} (\S+)", open(HEADER).read()).group(1))
              for name in ("FA_CLOSE_PAIR", "FA_TRACE_OFF"))


def weights_will_do(K, R, near):
    s, Q = np.diag(K), R.T @ R
    D2, r2 = s[:, None] + s[None] - 2 * K, np.diag(Q)
    pairs = D2 > 1e-12 * (s[:, None] + s[None])
    off = np.abs((r2[:, None] + r2[None] - 2 * Q) / np.where(pairs, D2, 1) - 1)[pairs]
    return near > CLOSE and (len(R) == len(K) or max(np.max(off), np.max(np.abs(r2 / s - 1))) <= OFF)


@pytest.mark.parametrize("noise", [0.0, 1e-10, 5e-10])
@pytest.mark.parametrize("p", [7, 15, 20, 42, 60])
def test_the_weights_sum_to_the_trace_where_the_rule_says_so(p, noise):
    taken, worst_left = 0, 0.0
    for dist in (3e-6, 1e-4, 1.2e-3, 2e-3, 1e-2, 1.0):
        for seed in range(3):
            K = near_copies(p, max(3, p // 3), dist, 400, seed, noise)
            for m, lam in ((2, 1.0), (p // 2, 4.0)):
                _, R, _, _, near, ratio = irls(K, m, lam, 5)
                off = np.max(np.abs(ratio - 1))
                if weights_will_do(K, R, near):
                    taken += 1
                    assert off <= 1e-7, (dist, seed, m, off)
                else:
                    worst_left = max(worst_left, off)
    assert taken >= 12
    assert worst_left > (0.05 if noise else 1e-8)


@pytest.mark.parametrize("p,rank", [(7, 5), (16, 9), (20, 16), (48, 20), (64, 48)])
def test_exact_copies_need_no_measured_trace(p, rank):
    """Copies, one of them scaled (a distance, but no pivot): nothing is left out."""
    r = np.random.default_rng(p + rank)
    G = r.standard_normal((rank, 200)) * 0.5 + r.standard_normal((1, 200))
    G = G[np.concatenate([np.arange(rank), r.integers(0, rank, p - rank)])]
    G[-1] *= -4
    K = G @ G.T
    _, R, _, _, near, ratio = irls(K, rank // 2, 1.0, 5)
    assert len(R) == rank and weights_will_do(K, R, near)
    assert np.max(np.abs(ratio - 1)) <= 1e-7
