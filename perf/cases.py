"""The aggregation calls whose time is followed, from one small model to the largest gradient sets.

Every case is one whole call (or one round of calls) through the package's public entry points, on
gradients drawn on the device: honest workers are a common direction plus noise, the Byzantine
ones send sign flips, large noise or a colluding direction.  The shapes are those of the five
configurations the benchmark and the tests use (7 workers x 100 thousand parameters up to 64
workers x 50 million), of the largest worker count the paper reports (60), and ragged sizes in
between, in both storage types and both storage orders.

    listed()            the cases that are timed
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and context a program has in hand before the call
    run(state)          one call; returns its outputs
    work(case)          bytes and operations the call cannot do without
    tolerance(case)     how far another correct implementation may be
    exact(case, seed)   the outputs in 64 bits, from plain torch and numpy
"""
import math
import random

import numpy as np
import torch

from paper_2302_05865_amd import FlagAggregator, fa_aggregate_static


def _case(entry, p, n, m, lam, iters, dtype="f32", layout="worker_major", recipe="mixed", f=1,
          pieces=0, k=1, name=None):
    c = dict(entry=entry, p=p, n=n, m=m, lam=lam, iters=iters, dtype=dtype, layout=layout,
             recipe=recipe, f=f, pieces=pieces, k=k)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a handful of workers on a small model, where launches and the
        # p x p solve are everything
        _case("aggregate", 7, 100_000, 4, 1.0, 10, recipe="signflip", f=1, name="small_p7"),
        # the entry point that allocates nothing, a small residual network's gradient, the
        # paper's own budget of five solves; odd length
        _case("static", 15, 271_117, 8, 1.0, 5, f=3, name="static_p15"),
        # the headline configuration
        _case("aggregate", 15, 11_200_000, 8, 1.0, 20, f=3, name="headline_p15"),
        # gradients stored interleaved, an even worker count, an odd number of coordinates
        _case("aggregate", 20, 3_000_001, 11, 1.0, 10, layout="row_major", f=4,
              name="rows_p20"),
        # interleaved bf16 at the width of two matrix tiles
        _case("aggregate", 32, 8_000_000, 17, 1.0, 10, dtype="bf16", layout="row_major",
              recipe="lowrank", f=6, name="rows_bf16_p32"),
        # ragged in every direction: 23 workers, odd length, bf16
        _case("aggregate", 23, 999_999, 12, 0.1, 12, dtype="bf16", recipe="lowrank", f=4,
              name="ragged_bf16_p23"),
        # the paper's largest setting: 60 workers with 14 Byzantine ones on a small convolutional
        # network, five solves
        _case("aggregate", 60, 1_199_882, 31, 1.0, 5, recipe="cluster", f=14, name="paper_p60"),
        # workers that send two gradients each
        _case("grouped", 32, 2_000_003, 16, 1.0, 15, f=3, k=2, name="grouped_16x2"),
        # the distance-based aggregator on the same passes
        _case("krum", 15, 11_200_000, 10, 0.0, 1, f=3, name="krum_p15"),
        # one round in which every gradient lands in four pieces, then the aggregate
        _case("arrival", 15, 11_200_000, 8, 1.0, 20, f=3, pieces=4, name="arrival_p15"),
        # language-model sized gradients in bf16
        _case("aggregate", 32, 124_000_000, 16, 1.0, 15, dtype="bf16", recipe="lowrank", f=6,
              name="large_bf16_p32"),
        # the widest set at full length
        _case("aggregate", 64, 50_000_000, 32, 1.0, 30, recipe="cluster", f=12,
              name="large_p64"),
    ]


def draw(rng: random.Random):
    entry = rng.choice(["aggregate"] * 6 + ["static", "grouped", "krum", "arrival"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    layout = "worker_major"
    if entry not in ("static", "arrival"):
        layout = rng.choice(["worker_major", "worker_major", "row_major"])
    k = 1
    if entry == "grouped":
        k = rng.choice([2, 3, 4])
        workers = rng.randint(4, 64 // k)
        p = workers * k
    else:
        p = round(math.exp(rng.uniform(math.log(5), math.log(64.49))))
        workers = p
    most = 4_000_000_000 // (p * (4 if dtype == "f32" else 2))
    if layout == "row_major":
        most //= 2
    if entry == "arrival":
        most //= p                       # the pieces read the gradients that are there already
    n = round(math.exp(rng.uniform(math.log(20_000), math.log(max(40_000, most)))))
    f = rng.randint(1, max(1, (workers - 3) // 3))
    m = (p + 2) // 2 if rng.random() < 0.7 else rng.randint(2, p)
    if entry == "krum":
        m = rng.randint(1, p - f)        # how many workers are averaged
    return _case(entry, p, n, m, rng.choice([0.1, 1.0, 1.0]), rng.randint(5, 30), dtype, layout,
                 rng.choice(["mixed", "signflip", "lowrank", "cluster", "student"]), f,
                 rng.randint(1, 6) if entry == "arrival" else 0, k)


# ---- inputs -------------------------------------------------------------------------------------

def _pitch(c):
    """Row pitch in elements: whole 16-byte units per gradient, or p values per coordinate."""
    if c["layout"] == "row_major":
        return c["p"]
    per = 4 if c["dtype"] == "f32" else 8
    return -(-c["n"] // per) * per


def _gradients(c, seed):
    """[p, n] (a view of padded rows), or [n, p] when stored row by row."""
    p, n, f = c["p"], c["n"], c["f"]
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(1000 * seed + 17)
    pick = random.Random(7919 * seed + 13 * p + n % 1009)
    workers = p // c["k"]
    byz = set(pick.sample(range(workers), f))
    rows = c["layout"] == "row_major"
    G = torch.zeros((n, p) if rows else (p, _pitch(c)), dtype=dt, device="cuda")

    def normal():
        return torch.randn(n, generator=gen, device="cuda")

    mu, mu2 = normal(), normal()
    U = [normal() for _ in range(4)] if c["recipe"] == "lowrank" else []
    nb = 0
    for i in range(p):
        w = i // c["k"]
        if w in byz:
            kind = {"signflip": "flip10", "lowrank": "noise", "student": "collude",
                    "cluster": ("flip4", "noise")[nb % 2],
                    "mixed": ("noise", "flip4", "unit")[nb % 3]}[c["recipe"]]
            nb += 1
            if kind == "flip10":
                col = -10.0 * mu
            elif kind == "flip4":
                col = -4.0 * mu
            elif kind == "noise":
                col = 5.0 * normal()
            elif kind == "collude":
                col = -mu + 0.1 * normal()
            else:
                col = normal()
                col *= 1000.0 / col.norm()
        else:
            col = normal()
            if c["recipe"] == "signflip":
                col.mul_(0.1)
            elif c["recipe"] == "student":      # three degrees of freedom, by the definition
                chi = normal() ** 2 + normal() ** 2 + normal() ** 2
                col = 0.5 * col / (chi / 3.0).clamp_min(1e-12).sqrt()
            else:
                col.mul_(0.5)
            col += mu2 if c["recipe"] == "cluster" and pick.random() >= 0.7 else mu
            for u in U:
                col += pick.gauss(0.0, 1.0) * u
        if rows:
            G[:, i] = col.to(dt)
        else:
            G[i, :n] = col.to(dt)
        del col
    return G if rows else G[:, :n]


def prepare(case, seed):
    G = _gradients(case, seed)
    state = dict(case=case, G=G, out=torch.empty(case["n"], dtype=torch.float32, device="cuda"))
    if case["entry"] != "static":
        state["fa"] = FlagAggregator(n_max=case["n"], p_max=case["p"], dtype=case["dtype"],
                                     layout=case["layout"])
    if case["entry"] == "grouped":
        state["sizes"] = [case["k"]] * (case["p"] // case["k"])
    if case["entry"] == "arrival":
        # cuts on whole 16-byte units
        unit = 4 if case["dtype"] == "f32" else 8
        step = max(1, -(-case["n"] // (case["pieces"] * unit))) * unit
        state["cuts"] = [(a, min(step, case["n"] - a)) for a in range(0, case["n"], step)]
    return state


def run(state):
    c, G, out = state["case"], state["G"], state["out"]
    m, lam, iters = c["m"], c["lam"], c["iters"]
    if c["entry"] == "static":
        return fa_aggregate_static(G, m, lam, iters, 0.0, out)
    fa = state["fa"]
    if c["entry"] == "aggregate":
        return fa.fa_aggregate(G, m, lam, iters, 0.0, out)
    if c["entry"] == "grouped":
        return fa.fa_aggregate_grouped(G, state["sizes"], m, lam, iters, 0.0, out)
    if c["entry"] == "krum":
        return fa.fa_multikrum(G, c["f"], m, out)
    fa.fa_gram_begin(c["p"], c["n"])
    for row0, rows in state["cuts"]:         # a round: the workers' pieces come in interleaved
        for i in range(c["p"]):
            fa.fa_gram_update_rows(G, i, row0, rows)
    return fa.fa_aggregate_arrived(G, m, lam, iters, 0.0, out)


# ---- what a call cannot do without ---------------------------------------------------------------

def work(case):
    p, n = case["p"], case["n"]
    size = 4 if case["dtype"] == "f32" else 2
    return {"bytes": p * n * size + 4 * n, "flops": n * p * (p + 1) + 2 * n * p}


def tolerance(case):
    # One fp32 rounding of the result is 2.5e-8, and that is what most cases show against exact().
    # Wide sets from about a million coordinates on take sums of 32 products in fp32 (5e-9 on the
    # Gram matrix), which a subspace whose m-th gap is nearly closed passes on enlarged: up to 2e-6
    # over the listed and two dozen drawn cases.  About four times that; coordinates may be off by
    # forty times the 2-norm.  Which workers are averaged is compared exactly.
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.0}


# ---- the same in 64 bits -------------------------------------------------------------------------

def _irls(K, m, lam, iters, sizes, delta=1e-6, pair_tol=1e-12):
    """Coefficients c of the direction G c, from the exact Gram matrix: repeated weighted PCA of
    the normalised gradients and of the normalised pair differences, all in the coordinates of an
    orthonormal basis of the gradients' span."""
    p, W = K.shape[0], len(sizes)
    blk = np.repeat(np.arange(W), sizes)
    first = np.concatenate([[0], np.cumsum(sizes)])[:-1]
    live = np.diag(K) > 0
    scale = np.where(live, 1 / np.sqrt(np.where(live, np.diag(K), 1)), 0)
    lam0, V = np.linalg.eigh(K * scale[:, None] * scale[None, :])
    keep = lam0 > 1e-12 * lam0[-1]
    L, V = np.sqrt(lam0[keep]), V[:, keep]
    R = (L[:, None] * V.T) / np.where(scale > 0, scale, 1)[None, :] * live[None, :]   # G = Q R
    B = scale[:, None] * V / L[None, :]                                              # R B = I
    r = R.shape[0]
    s = np.array([np.diag(K)[blk == a].sum() for a in range(W)])
    pairs = []
    for a in range(W):
        for b in range(a + 1, W):
            if sizes[a] != sizes[b] or not lam > 0:
                continue
            ia, ib = np.arange(first[a], first[a] + sizes[a]), np.arange(first[b], first[b] + sizes[b])
            d2 = (K[ia, ia] + K[ib, ib] - 2 * K[ia, ib]).sum()
            if d2 > pair_tol * (s[a] + s[b]):
                pairs.append((a, b, ia, ib, d2))
    coef = lam / (W - 1) if W > 1 else 0.0
    w = (s > 0).astype(float)
    D = [R[:, ia] - R[:, ib] for _, _, ia, ib, _ in pairs]
    Dall = np.concatenate(D, 1) if D else np.zeros((r, 0))
    dlen = np.array([d.shape[1] for d in D], dtype=int)
    d2 = np.array([q[4] for q in pairs])
    wp = np.ones(len(pairs))
    for _ in range(iters):
        M = (R * np.where(s[blk] > 0, w[blk] / np.where(s[blk] > 0, s[blk], 1), 0)[None, :]) @ R.T
        if len(pairs):
            M = M + 2 * coef * (Dall * np.repeat(wp / d2, dlen)[None, :]) @ Dall.T
        _, Q = np.linalg.eigh((M + M.T) / 2)
        Q = Q[:, ::-1]
        U, N = Q[:, :m], Q[:, m:]
        res = (N.T @ R) ** 2
        rho = np.array([res[:, blk == a].sum() for a in range(W)]) / np.where(s > 0, s, 1)
        w = np.where(s > 0, np.maximum(rho, delta) ** -0.5, 0)
        if len(pairs):
            rp = np.add.reduceat(((N.T @ Dall) ** 2).sum(0), np.concatenate([[0], np.cumsum(dlen)])[:-1]) / d2
            wp = np.maximum(rp, delta) ** -0.5
    mean = np.concatenate([np.full(k, 1.0 / k) for k in sizes]) / W
    return B @ (U @ (U.T @ (R @ mean)))


def exact(case, seed):
    G = _gradients(case, seed)
    if case["layout"] == "row_major":
        G = G.t()
    p, n = G.shape
    step = max(1, (1 << 27) // p)
    K = torch.zeros((p, p), dtype=torch.float64, device="cuda")
    for a in range(0, n, step):
        x = G[:, a:a + step].to(torch.float64).contiguous()
        K += x @ x.t().contiguous()
    K = K.cpu().numpy()
    scores = None
    if case["entry"] == "krum":
        D = np.diag(K)[:, None] + np.diag(K)[None, :] - 2 * K
        scores = np.array([np.sort(np.delete(D[i], i))[:p - case["f"] - 2].sum() for i in range(p)])
        chosen = np.zeros(p, dtype=np.int32)
        chosen[np.argsort(scores, kind="stable")[:case["m"]]] = 1
        c = chosen / case["m"]
    else:
        c = _irls(K, case["m"], case["lam"], case["iters"], [case["k"]] * (p // case["k"]))
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    cd = torch.from_numpy(np.ascontiguousarray(c, dtype=np.float64)).cuda()
    for a in range(0, n, step):
        out[a:a + step] = cd @ G[:, a:a + step].to(torch.float64).contiguous()
    return out if scores is None else (out, scores, chosen)
