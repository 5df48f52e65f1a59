"""Workers that send nearly the same vector, and the solvers' steps on their Gram matrix in NumPy: the same
factorisation, eigenvectors instead of purifications."""
import numpy as np


def near_copies(p, count, dist, n, seed, noise):
    """Gram matrix of p workers, `count` of them within dist of one vector, its entries off by `noise`."""
    r = np.random.default_rng(seed)
    G = r.standard_normal((p, n)) * 0.5 + r.standard_normal((1, n))
    v = r.standard_normal(n)
    for i in r.permutation(p)[:count]:
        G[i] = v + dist * r.uniform(0.3, 2) * r.standard_normal(n)
    K = G @ G.T
    E = r.standard_normal((p, p)) * noise
    s = np.sqrt(np.diag(K))
    return K + (E + E.T) / np.sqrt(2) * s[:, None] * s[None]


def factor(K, rank_tol=1e-12):
    """The solvers' R: greedy pivots, the largest diagonal entry left as seen in fp32 (64 columns: six bits of its
    mantissa hold the column; 16: four), until none is above rank_tol."""
    p = len(K)
    low = np.uint32(63 if p > 16 else 15)
    s = np.diag(K)
    S = K / np.sqrt(s)[:, None] / np.sqrt(s)[None]
    S[np.diag_indices(p)] = 1.0
    d, left, rows = np.ones(p), np.ones(p), []
    while len(rows) < p:
        pv = int(np.argmax(np.float32(np.maximum(d, 0)).view(np.uint32) & ~low))
        if not d[pv] > rank_tol:
            break
        row = S[pv] * left / np.sqrt(d[pv])
        row[pv] = np.sqrt(d[pv])
        rows.append(row)
        S = S - np.outer(row, row)
        d = d - row * row
        d[pv] = left[pv] = 0
    return np.array(rows) * np.sqrt(s)


def irls(K, m, lam, iters, delta=1e-6, pair_tol=1e-12):
    """Eq. 5's IRLS over span R by eigenvectors: objectives, R, the last projector, the smallest gap at m over
    the largest eigenvalue, the smallest live D_ij^2 / (|g_i|^2 + |g_j|^2), trace M over the sum of the weights."""
    p, s, R = len(K), np.diag(K), factor(K)
    both = s[:, None] + s[None]
    D2 = both - 2 * K
    live = (D2 > pair_tol * both) & ~np.eye(p, dtype=bool)
    inv = np.where(live, 1 / np.where(live, D2, 1), 0)
    w, wp, coef, gap, objective, ratio = np.ones(p), live * 1.0, lam / (p - 1), 1.0, [], []
    for _ in range(iters):
        C = -2 * coef * inv * wp
        C[np.diag_indices(p)] = w / s - C.sum(1)
        M = R @ (C @ R.T)
        ratio.append(np.trace(M) / (w.sum() + coef * wp.sum()))
        ev, Q = np.linalg.eigh(np.tril(M) + np.tril(M, -1).T)
        gap = min(gap, (ev[-m] - ev[-m - 1]) / ev[-1])
        P = Q[:, -m:] @ Q[:, -m:].T
        Z = R - P @ R
        q = Z.T @ Z
        rho = np.maximum(np.diag(q) / s, 0)
        pair = np.maximum(np.diag(q)[:, None] + np.diag(q)[None] - 2 * q, 0) * inv
        objective.append(np.sqrt(rho).sum() + coef * np.sqrt(pair).sum())
        w = np.minimum(1 / np.sqrt(np.maximum(rho, 1e-300)), delta ** -0.5)
        wp = np.where(live, np.minimum(1 / np.sqrt(np.maximum(pair, 1e-300)), delta ** -0.5), 0)
    return np.array(objective), R, P, gap, np.min((D2 / both)[live]), np.array(ratio)
