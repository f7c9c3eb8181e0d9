"""Performance cases of the sampler: what its users run, through the Python binding.

Each case is one call (or one round of calls) as a program makes it, with the
parameter ranges of ``paper_2411_16952_amd/workloads.py``, the paper's Tables 1-2
and ``bench.py``.  ``listed`` and ``draw`` give cases, ``prepare`` what a program
holds before the call, ``run`` one pass, ``work`` the operations and bytes the
method cannot do without, ``exact`` the outputs in 64 bits from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2411_16952_amd import tkdv as T

# beta' C3/C2 sqrt(E0) up to which the paper's proposal accepts at least about
# 1e-4 (Tables 1-2; the sweep of workloads.py for K = 16, 32, 64)
P_MAX = {8: 900.0, 16: 2800.0, 32: 7500.0, 64: 18000.0, 128: 40000.0}
PRECISION = {"fp32": T.FP32, "bf16x3": T.BF16X3}
PROPOSAL = {"sigma": T.SIGMA, "uniform": T.UNIFORM}
# VALU operations and matrix flops of one proposal grow as K and K^2; a drawn
# case's proposals are cut so that it costs less than the largest listed one
COST = {8: 0.25, 16: 0.5, 32: 1.0, 64: 2.3, 128: 5.2}


def listed():
    return [
        # The smallest real call: the CPU-sized configuration of the paper's
        # method (K = 8, strong skewness), where launches and latency count.
        dict(name="sample_k8", kind="sample", K=8, E0=1.0, beta=40.0, c=20.0, proposal="sigma", precision="bf16x3",
             mode="proposals", n=10**6, cap=4096, acc=2.8e-3),
        # Table 1's linear row: a million samples where nearly every proposal is
        # accepted, so that writing rows and their statistics is the work.
        dict(name="linear_k16", kind="sample", K=16, E0=1.0, beta=20.0, c=0.0, proposal="sigma", precision="bf16x3",
             mode="accepted", n=10**6, cap=10**6, max_proposals=1 << 32, acc=0.953),
        # The paper's baseline (Table 1's improvement column), FP32 products.
        dict(name="uniform_k16_fp32", kind="sample", K=16, E0=1.0, beta=20.0, c=30.0, proposal="uniform",
             precision="fp32", mode="proposals", n=2 * 10**7 + 11, cap=1 << 16, acc=4e-4),
        # One training point's samples for the learned proposal: few accepted
        # samples of a strongly nonlinear point, an open-ended proposal range.
        dict(name="train_draw_k32", kind="sample", K=32, E0=1.0, beta=100.0 / 3.0, c=270.0, proposal="sigma",
             precision="bf16x3", mode="accepted", n=4096, cap=4096, max_proposals=1 << 36, acc=4.1e-5),
        # The paper's sampler at its main size: one point of the plain benchmark.
        dict(name="sample_k32", kind="sample", K=32, E0=1.0, beta=40.0, c=150.0, proposal="sigma", precision="bf16x3",
             mode="proposals", n=10**9, cap=1 << 20, acc=1.1e-3),
        # The headline: one point of the learned mixture's benchmark.
        dict(name="mixture_k32", kind="mixture", K=32, E0=1.0, beta=40.0, c=225.0, precision="bf16x3", n=10**9,
             cap=1 << 20, acc=7e-3),
        # Several points of the large mode counts in one launch sequence.
        dict(name="batch_k64_k128", kind="batch", K=64, K2=128, points=4, E0=1.0, frac=0.75, precision="bf16x3",
             n=6 * 10**7 + 1, cap=1 << 15, acc=8e-3),
        # A parameter sweep to accepted targets, mixed K, a bounded row store.
        dict(name="sweep_mixed", kind="sweep", K=0, points=24, targets_lo=1e4, targets_hi=3e5, frac=0.8, cap=1 << 12,
             precision="bf16x3", acc=2e-2),
        # An extremes map: 1-in-500 events over a region of parameter space.
        dict(name="map_k32", kind="map", K=32, E0=1.0, nb=8, nc=8, n=500, frac=0.6, precision="bf16x3", acc=5e-2),
        # The search for extreme wave fields among a million stored samples.
        dict(name="extremes_k64", kind="extremes", K=64, E0=1.0, n=10**6 + 3, stride=128, top_k=100),
        # Importance resampling of a strongly nonlinear point, rows wanted.
        dict(name="sir_k32", kind="sir", K=32, E0=1.0, beta=40.0, c=75.0, proposal="sigma", precision="bf16x3",
             n=10**8 + 5, m=10**5),
        # Adam steps of the network between two cutting-plane rounds.
        dict(name="train_k32", kind="train", K=32, points=16, rows=4096, extra=24, hidden=256, steps=30),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sample", "accepted", "uniform", "mixture", "batch", "sweep", "map", "extremes", "sir", "train"])
    E0 = rng.choice([0.5, 1.0, math.pi / 2, 2.0])
    prec = rng.choice(["bf16x3", "bf16x3", "fp32"])
    slow = 4.0 if prec == "fp32" else 1.0
    if kind in ("sample", "uniform"):
        K = rng.choice([8, 16, 32, 64, 128] if kind == "sample" else [8, 16, 32])
        beta = rng.uniform(10.0, 60.0)
        frac = rng.uniform(0.0, 0.95) if kind == "sample" else rng.uniform(0.0, 0.3)
        return dict(kind="sample", K=K, E0=E0, beta=beta, c=frac * P_MAX[K] / (beta * math.sqrt(E0)),
                    proposal="sigma" if kind == "sample" else "uniform", precision=prec, mode="proposals",
                    n=_log_int(rng, 1e4, 8e8 / COST[K] / slow / 4.0), cap=_log_int(rng, 100, 1 << 17),
                    acc=0.95 * math.exp(-8.0 * frac))
    if kind == "accepted":
        K = rng.choice([8, 16, 32, 64])
        beta = rng.uniform(10.0, 60.0)
        frac = rng.uniform(0.0, 0.7)
        n = _log_int(rng, 100, 2e5)
        return dict(kind="sample", K=K, E0=E0, beta=beta, c=frac * P_MAX[K] / (beta * math.sqrt(E0)),
                    proposal="sigma", precision=prec, mode="accepted", n=n, cap=n,
                    max_proposals=1 << rng.randint(30, 36), acc=0.95 * math.exp(-8.0 * frac))
    if kind == "mixture":
        K = rng.choice([8, 16, 32])
        beta = rng.uniform(20.0, 60.0)
        return dict(kind="mixture", K=K, E0=E0, beta=beta,
                    c=rng.uniform(0.6, 1.2) * P_MAX[K] / (beta * math.sqrt(E0)), precision=prec,
                    n=_log_int(rng, 1e5, 3e8 / slow), cap=_log_int(rng, 100, 1 << 17), acc=5e-3)
    if kind == "batch":
        K, K2 = rng.choice([(64, 128), (32, 64), (16, 32), (8, 128)])
        n = _log_int(rng, 1e4, 2e7 / slow)
        # a row store that every point fills
        return dict(kind="batch", K=K, K2=K2, points=rng.randint(2, 9), E0=E0, frac=rng.uniform(0.2, 0.7),
                    precision=prec, n=n, cap=1 + n // 20000, acc=1e-2)
    if kind == "sweep":
        return dict(kind="sweep", K=0, points=rng.randint(3, 40), targets_lo=1e3, targets_hi=rng.choice([1e4, 1e5]),
                    frac=rng.uniform(0.2, 0.8), cap=_log_int(rng, 10, 1 << 12), precision="bf16x3", acc=2e-2)
    if kind == "map":
        return dict(kind="map", K=rng.choice([16, 32, 64]), E0=E0, nb=rng.randint(2, 10), nc=rng.randint(2, 10),
                    n=_log_int(rng, 100, 2000), frac=rng.uniform(0.3, 0.6), precision=prec, acc=5e-2)
    if kind == "extremes":
        K = rng.choice([8, 16, 32, 64, 128])
        return dict(kind="extremes", K=K, E0=E0, n=_log_int(rng, 1e3, 1.2e8 / K), top_k=rng.randint(1, 500),
                    stride=rng.choice([2 * K, 256]))
    if kind == "sir":
        K = rng.choice([8, 16, 32, 64, 128])
        beta = rng.uniform(20.0, 60.0)
        return dict(kind="sir", K=K, E0=E0, beta=beta, c=rng.uniform(0.2, 0.8) * P_MAX[K] / (beta * math.sqrt(E0)),
                    proposal="sigma", precision=prec, n=_log_int(rng, 1e5, 1e8 / COST[K] / slow),
                    m=_log_int(rng, 100, 1e5))
    return dict(kind="train", K=rng.choice([8, 16, 32]), points=rng.randint(2, 20), rows=_log_int(rng, 200, 6000),
                extra=rng.randint(1, 60), hidden=rng.choice([64, 128, 200, 256]), steps=rng.randint(5, 40))


# --------------------------------------------------------------------------
# What a program holds before the call
# --------------------------------------------------------------------------
_CTX = None


def _ctx():
    """One context per process, as a program keeps it."""
    global _CTX
    if _CTX is None:
        _CTX = T.Context(0)
    return _CTX


def _modes(K, r):
    return (np.arange(K) + 1.0) / K if r else np.arange(K) + 1.0


def _mixture(K, plan):
    """A mixture of the shape the trained networks have: D near Sigma, the cos
    block carrying the localised crest, the sin block its steepness."""
    r = _modes(K, True)
    logd = np.log(np.array(plan.sigma2[:K])) - 0.07 + 0.3 * r**6
    V = np.zeros((2 * K, 2))
    V[:K, 0] = 0.68 * (1.0 - r**1.8)
    V[:K, 1] = 0.16 * r * (1.0 - r**6)
    V[K:, 0] = -0.14 * np.sin(math.pi * r)
    V[K:, 1] = 0.40 * np.sin(math.pi * r**0.9)
    s = math.sqrt(32.0 / K)
    return T.make_mixture(K, 0.2, logd, s * V)


def _alpha(K, beta):
    """The root of F(alpha) = 1 - (alpha/K) sum_k 1/(1 + alpha beta' k^2/K^3) (Sec. III.A) by bisection."""
    k2 = _modes(K, False) ** 2
    lo, hi = 1e-9, 1e9
    for _ in range(200):
        mid = math.sqrt(lo * hi)
        if mid * np.sum(1.0 / (1.0 + mid * beta * k2 / K**3)) < K:
            lo = mid
        else:
            hi = mid
    return math.sqrt(lo * hi)


def _sigma2(K, beta):
    return 1.0 / (1.0 + _alpha(K, beta) * beta * _modes(K, False) ** 2 / K**3)


def _spread_points(case, seed):
    """Points of one batch, sweep or map-like call: beta' and the nonlinearity
    spread evenly over their ranges, mixed K, the seed as the Philox key."""
    pts, P = [], int(case["points"])
    for q in range(P):
        if case["kind"] == "sweep":
            K, E0 = (16, 32, 64)[q % 3], (0.5, 1.0, math.pi / 2, 2.0)[q % 4]
        else:
            K, E0 = (int(case["K"]), int(case["K2"]))[q % 2], case["E0"]
        beta = 15.0 + 45.0 * ((q * 0.618034) % 1.0)
        f = case["frac"] * ((0.25 + q * 0.414214) % 1.0)
        pts.append(T.make_point(K, E0, beta, f * P_MAX[K] / (beta * math.sqrt(E0)), seed=seed, point_id=3000 + q))
    return pts


def _rows(K, beta, n, stride, seed):
    """n unit rows x^ of the paper's proposal, row stride `stride` floats, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    buf = torch.empty((n, stride), dtype=torch.float32, device="cuda")
    sg = torch.from_numpy(np.sqrt(_sigma2(K, beta))).to("cuda", torch.float32).repeat(2)
    for r in range(0, n, 1 << 18):
        m = min(1 << 18, n - r)
        x = torch.randn((m, 2 * K), generator=g, device="cuda") * sg
        buf[r:r + m, :2 * K] = x / x.norm(dim=1, keepdim=True)
    return buf[:, :2 * K]


def _train_points(case):
    K, P = int(case["K"]), int(case["points"])
    betas = [20.0 + 40.0 * i / max(P - 1, 1) for i in range(P)]
    return [(b, 9000.0 * (K / 32.0) ** 2 / b) for b in betas]


def _train_rows(case, seed):
    """Per point: accepted-like rows (a crest at a random place plus the
    proposal's background, FP32) and rows near the crest alone (FP64)."""
    K, rng = int(case["K"]), np.random.default_rng(int(seed))
    k = _modes(K, False)
    out = []
    for beta, _ in _train_points(case):
        sg = np.sqrt(_sigma2(K, beta))
        crest = 1.0 - 0.8 * (k / K) ** 2
        sets = []
        for m, amp in ((int(case["rows"]), rng.uniform(0.0, 1.0, (int(case["rows"]), 1))), (int(case["extra"]), 4.0)):
            phi = rng.uniform(-math.pi, math.pi, (m, 1))
            z = rng.standard_normal((m, 2 * K))
            z[:, :K] = z[:, :K] * sg + amp * crest * np.cos(k * phi)
            z[:, K:] = z[:, K:] * sg + amp * crest * np.sin(k * phi)
            sets.append(z / np.linalg.norm(z, axis=1, keepdims=True))
        out.append((sets[0].astype(np.float32), sets[1]))
    return out


def _train_weights(case, seed):
    """Weights as they are between two rounds: Glorot-sized, a small last layer."""
    H, no, rng = int(case["hidden"]), 5 * int(case["K"]), np.random.default_rng(int(seed) + 1)
    sizes = ((3 * H, math.sqrt(6.0 / (3 + H))), (H, 0.02), (H * H, math.sqrt(3.0 / H)), (H, 0.02), (H * no, 0.02),
             (no, 0.02))
    return np.concatenate([a * rng.uniform(-1.0, 1.0, m) for m, a in sizes])


def prepare(case, seed):
    ctx, kind, K = _ctx(), case["kind"], int(case["K"])
    s = {"case": dict(case), "ctx": ctx, "kind": kind}
    if kind in ("sample", "mixture", "sir"):
        pt = T.make_point(K, case["E0"], case["beta"], case["c"], seed=int(seed), point_id=7)
        prop = PROPOSAL[case["proposal"]] if kind != "mixture" else T.SIGMA
        plans, _ = ctx.plan_batch([pt], prop, n_starts=16, seed=1)
        s.update(point=pt, plan=plans[0], proposal=prop)
        if kind == "mixture":
            s["mix"] = _mixture(K, plans[0])
            mp, _ = ctx.plan_mixture_batch([pt], plans, [s["mix"]], n_starts=16, margin=0.02)
            s["plan"] = mp[0]
        if kind != "sir":  # the program's own row store (rows that no sample reaches stay zero)
            s["xhat"] = torch.zeros((int(case["cap"]), 2 * K), device="cuda")
            s["index"] = torch.zeros((int(case["cap"]),), dtype=torch.int64, device="cuda")
    elif kind in ("batch", "sweep"):
        s["points"] = _spread_points(case, int(seed))
        s["plans"], _ = ctx.plan_batch(s["points"], T.SIGMA, n_starts=16, seed=1)
        if kind == "sweep":
            P = len(s["points"])
            lo, hi = math.log(case["targets_lo"]), math.log(case["targets_hi"])
            s["targets"] = [int(math.exp(lo + (hi - lo) * ((0.5 + q * 0.732051) % 1.0))) for q in range(P)]
            s["cap"] = [min(t, int(case["cap"])) for t in s["targets"]]
    elif kind == "map":
        s["betas"] = [15.0 + 45.0 * (i + 0.5) / case["nb"] for i in range(int(case["nb"]))]
        s["c32s"] = [case["frac"] * P_MAX[K] / (60.0 * math.sqrt(case["E0"])) * i / case["nc"]
                     for i in range(int(case["nc"]))]
        s["seed"] = int(seed)
    elif kind == "extremes":
        s["rows"] = _rows(K, 40.0, int(case["n"]), int(case["stride"]), seed)
    elif kind == "train":
        pts = [T.make_point(K, 1.0, b, c, seed=100 + i, point_id=i) for i, (b, c) in enumerate(_train_points(case))]
        plans, _ = ctx.plan_batch(pts, T.SIGMA, n_starts=16, seed=1)
        L = T.Learner(ctx, T.learner_cfg(K, hidden=int(case["hidden"]), eps=0.2, v_amp=0.5, v_scale=1.0, lr=3e-3,
                                         seed=5))
        L.set_points(pts, plans)
        for i, (acc, near) in enumerate(_train_rows(case, seed)):
            L.add_rows(i, torch.from_numpy(acc).cuda(), kind=0)
            L.add_rows(i, near, kind=1)
        s.update(learner=L, w0=_train_weights(case, seed))
    return s


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------
def _i64(v):
    return int(v) if int(v) < 1 << 63 else -1


def _stats(d):
    """The statistics of one point.  Left out: n_fp64_fixups and max_log_a,
    which say how the decisions were reached (how many the FP32 pass left
    open, over which proposals), not what was sampled."""
    return {"counts": np.array([d["n_proposed"], d["n_accepted"], d["n_written"], d["n_exceed_2sigma"],
                                d["n_exceed_4sigma"], d["n_samples_4sigma"], _i64(d["peak_index"]), d["M_raises"]],
                               dtype=np.int64),
            "moments": np.array([d["S1"], d["S2"], d["S3"], d["S4"]]),
            "shape": np.array([d["skewness"], d["kurtosis"], d["p_exceed_2sigma"]]),
            "hist": d["hist_u0"].astype(np.int64), "peak_u": float(d["peak_u"])}


def _many(ds):
    """The statistics of several points, stacked."""
    st = [_stats(d) for d in ds]
    return {k: np.array([q[k] for q in st]) for k in st[0]}


def run(s):
    ctx, case, kind = s["ctx"], s["case"], s["kind"]
    if kind == "sample":
        mode = T.COUNT_ACCEPTED if case["mode"] == "accepted" else T.COUNT_PROPOSALS
        d = ctx.sample(s["point"], int(case["n"]), proposal=s["proposal"], plan=s["plan"], mode=mode,
                       max_proposals=int(case.get("max_proposals", 0)), precision=PRECISION[case["precision"]],
                       capacity=int(case["cap"]), xhat=s["xhat"], index=s["index"])
        return dict(_stats(d), xhat=s["xhat"], index=s["index"])
    if kind == "mixture":
        d = ctx.sample_mixture(s["point"], s["plan"], s["mix"], int(case["n"]),
                               precision=PRECISION[case["precision"]], capacity=int(case["cap"]), xhat=s["xhat"],
                               index=s["index"])
        return dict(_stats(d), xhat=s["xhat"], index=s["index"])
    if kind == "batch":
        P = len(s["points"])
        out, _, _ = ctx.sample_batch(s["points"], [int(case["n"])] * P, plans=s["plans"],
                                     precision=PRECISION[case["precision"]], capacity=[int(case["cap"])] * P)
        return dict(_many(out), xhat=[d["xhat"] for d in out], index=[d["index"] for d in out])
    if kind == "sweep":
        out, _, index = ctx.sample_sweep(s["points"], s["targets"], [10**10] * len(s["points"]), plans=s["plans"],
                                         precision=PRECISION[case["precision"]], capacity=s["cap"])
        # every point meets its target, so every row of the store is written
        return dict(_many(out), index=index, xhat=[d["xhat"] for d in out])
    if kind == "map":
        cells = ctx.extremes_map(int(case["K"]), case["E0"], s["betas"], s["c32s"], int(case["n"]), 10**9,
                                 seed=s["seed"], precision=PRECISION[case["precision"]])
        f = ("alpha_star", "log_M", "acceptance", "skewness", "kurtosis", "p_exceed_2sigma", "p_exceed_4sigma",
             "p_sample_4sigma")
        return {"counts": np.array([[c["n_proposed"], c["n_accepted"], _i64(c["peak_index"]), c["status"],
                                     c["M_raises"]] for c in cells], dtype=np.int64),
                "values": np.array([[c[k] for k in f] for c in cells]),
                "peak_u": np.array([c["peak_u"] for c in cells], dtype=np.float32)}
    if kind == "extremes":
        d = ctx.extremes(s["rows"], int(case["K"]), E0=case["E0"], top_k=int(case["top_k"]))
        return {"rows": d["rows"].astype(np.int64), "umax": d["umax"].astype(np.float32), "jmax": d["jmax"],
                "n_exceed": d["n_exceed"]}
    if kind == "sir":
        d = ctx.sir(s["point"], int(case["n"]), int(case["m"]), 0.5, proposal=s["proposal"], plan=s["plan"],
                    precision=PRECISION[case["precision"]], rows=True)
        return {"sums": np.array([d["W"], d["W2"], d["ess"], d["max_w"]]),
                "moments": np.array([d["mean"], d["m2"], d["m3"], d["m4"]]),
                "over": int(d["n_over_one"]), "index": d["index"], "xhat": d["xhat"]}
    L = s["learner"]
    L.set_weights(s["w0"])
    loss = L.train(int(case["steps"]))
    return {"loss": loss, "weights": L.get_weights()}


# --------------------------------------------------------------------------
# The work of one pass
# --------------------------------------------------------------------------
def _proposal_flops(K):
    """VALU operations of one proposal (Philox, Box-Muller, norms, operands,
    cubes, decision) and the synthesis product in its quarter-period form."""
    return 47.0 * K + 73.0 + 4.0 * K * K


def _row_cost(K, n):
    """(bytes, flops) of n accepted samples: the row and index written, the
    FP32 synthesis and four power sums over N = 4K grid values."""
    return n * (8.0 * K + 8.0), n * (4.0 * K * K + 9.0 * 4 * K)


def work(case):
    kind, K = case["kind"], int(case["K"])
    n = float(case.get("n", 0))
    b = f = 0.0
    if kind in ("sample", "mixture"):
        accepted = case.get("mode") == "accepted"
        prop, acc = (n / case["acc"], n) if accepted else (n, n * case["acc"])
        f = prop * _proposal_flops(K)
        if kind == "mixture":  # y products of 32 shifts, rank 2, and log q_mix
            f += prop * (2.0 * 2 * K * 64 + 10.0 * 32 + 6.0 * K + 35.0)
        b = min(acc, case["cap"]) * (8.0 * K + 8.0)
        f += _row_cost(K, acc)[1]
    elif kind == "batch":
        for q in range(int(case["points"])):
            k = int(case["K"]) if q % 2 == 0 else int(case["K2"])
            f += n * _proposal_flops(k) + _row_cost(k, n * case["acc"])[1]
            b += min(n * case["acc"], case["cap"]) * (8.0 * k + 8.0)
    elif kind == "sweep":
        mean = (case["targets_hi"] - case["targets_lo"]) / math.log(case["targets_hi"] / case["targets_lo"])
        for q in range(int(case["points"])):
            k = (16, 32, 64)[q % 3]
            f += mean / case["acc"] * _proposal_flops(k) + _row_cost(k, mean)[1]
            b += min(mean, case["cap"]) * (8.0 * k + 8.0)
    elif kind == "map":
        cells = case["nb"] * case["nc"]
        f = cells * (n / case["acc"] * _proposal_flops(K) + _row_cost(K, n)[1])
        f += cells * 16 * 300.0 * 32.0 * K * K  # the plans' searches
        b = cells * 136.0
    elif kind == "extremes":
        f, b = n * (4.0 * K * K + 12.0 * K), n * 8.0 * K
    elif kind == "sir":
        f = n * (_proposal_flops(K) + 12.0 * K)
        b = n * 4.0 + case["m"] * (8.0 * K + 8.0)
    else:
        rows, H, out = case["points"] * (case["rows"] + case["extra"]), case["hidden"], 5.0 * K
        nw = 5.0 * H + H * H + H * out + out
        step = rows * 3 * 2.0 * 2 * K * 64 + case["points"] * 6.0 * nw + 12.0 * nw
        f = case["steps"] * step
        b = case["steps"] * (rows * 2 * K * 8.0 + 5 * 8.0 * nw)
    return {"bytes": b, "flops": f}


# --------------------------------------------------------------------------
# The outputs in 64 bits
# --------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _philox(i, pid, block, seed):
    """Philox4x32-10 words of counters (i, pid, block) as int64 tensors."""
    c = [i & _M32, i >> 32, torch.full_like(i, pid), torch.full_like(i, block)]
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & _M32) ^ c[1] ^ k0, b & _M32, ((a >> 32) & _M32) ^ c[3] ^ k1, a & _M32]
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c


def _unit(w):
    return (w.double() + 0.5) * 2.0**-32


def _grid(K, device):
    """Phi [2K, 4K] in 64 bits: cos and sin of k xi_j, xi_j = -pi + 2 pi j/N."""
    N = 4 * K
    k = torch.arange(1, K + 1, device=device)[:, None]
    r = (k * torch.arange(N, device=device)[None, :]) % N
    sign = 1.0 - 2.0 * (k % 2).double()
    ang = r.double() * (2.0 * math.pi / N)
    return torch.cat([sign * torch.cos(ang), sign * torch.sin(ang)])


def _log_ratio(x, K, E0, beta, c, alpha, sigma, phi):
    """log f - log g (the paper's unnormalised g; log f alone for the uniform
    proposal) of unit rows x, and their unscaled grid values."""
    k2 = torch.arange(1, K + 1, device=x.device).double() ** 2
    t = (x[:, :K] ** 2 + x[:, K:] ** 2) @ k2
    u = x @ phi
    H3 = math.pi / (12.0 * K) * (2.0 * E0 / math.pi) ** 1.5 * (u**3).sum(1)
    lr = -beta / (E0 * K * K) * (E0 * t - c * H3)
    return (lr + K * torch.log1p(alpha * beta * t / K**3) if sigma else lr), u


def _log_M(K, E0, beta, c, alpha, sigma):
    """log sup f/g over the sphere: closed form at c = 0, else ascent from the
    Dirichlet kernel, the single mode and random directions."""
    if c == 0.0:
        t = min(max(K**3 * (alpha - 1.0) / (alpha * beta), 1.0), float(K * K)) if sigma else 1.0
        return -beta * t / K**2 + (K * math.log1p(alpha * beta * t / K**3) if sigma else 0.0)
    phi, rng, best = _grid(K, "cpu"), np.random.default_rng(0), -math.inf
    one = np.zeros(2 * K)
    one[0] = 1.0
    for s in [np.concatenate([np.ones(K), np.zeros(K)]), one] + [rng.standard_normal(2 * K) for _ in range(4)]:
        y = torch.tensor(s / np.linalg.norm(s), requires_grad=True)
        opt = torch.optim.LBFGS([y], max_iter=600, history_size=20, tolerance_grad=1e-13, tolerance_change=1e-18,
                                line_search_fn="strong_wolfe")

        def closure():
            opt.zero_grad()
            v = -_log_ratio((y / y.norm())[None, :], K, E0, beta, c, alpha, sigma, phi)[0][0]
            v.backward()
            return v

        opt.step(closure)
        best = max(best, -float(closure().detach()))
    return best


def _proposals64(case, seed, i0, n, alpha, log_M, phi, sig):
    """x^, log a, log U and grid values of proposals i0 .. i0 + n - 1."""
    K, sigma = int(case["K"]), case["proposal"] == "sigma"
    i = torch.arange(i0, i0 + n, device=phi.device)
    x = torch.empty((n, 2 * K), dtype=torch.float64, device=phi.device)
    for b in range(K // 2):
        w = _philox(i, 7, b, int(seed))
        for q in (0, 2):
            r, th = torch.sqrt(-2.0 * torch.log(_unit(w[q]))), 2.0 * math.pi * _unit(w[q + 1])
            x[:, 4 * b + q] = r * torch.cos(th)
            x[:, 4 * b + q + 1] = r * torch.sin(th)
    log_u = torch.log(_unit(_philox(i, 7, K // 2, int(seed))[0]))
    if sigma:
        x *= sig
    x /= x.norm(dim=1, keepdim=True)
    lr, u = _log_ratio(x, K, case["E0"], case["beta"], case["c"], alpha, sigma, phi)
    return x, lr - log_M, log_u, u


def _exact_sample(case, seed):
    K, E0, beta = int(case["K"]), case["E0"], case["beta"]
    sigma, accepted = case["proposal"] == "sigma", case["mode"] == "accepted"
    covered = case["n"] / case["acc"] if accepted else case["n"]
    if covered * K > 4e9 or K > 32:
        return None  # too many proposals for 64-bit passes
    alpha = _alpha(K, beta) if sigma else 1.0
    log_M = _log_M(K, E0, beta, case["c"], alpha, sigma)
    phi = _grid(K, "cuda")
    sig = torch.from_numpy(np.sqrt(_sigma2(K, beta))).cuda().repeat(2)
    amp = math.sqrt(2.0 * E0 / math.pi)
    rows = torch.zeros((int(case["cap"]), 2 * K), dtype=torch.float64, device="cuda")
    got, S, peak, ex = 0, torch.zeros(4, dtype=torch.float64, device="cuda"), -math.inf, 0
    limit, total = (case["n"], 20 * covered) if accepted else (1 << 62, case["n"])
    chunk = (1 << 25) // K
    for i0 in range(0, int(total), chunk):
        x, la, lu, u = _proposals64(case, seed, i0, int(min(chunk, total - i0)), alpha, log_M, phi, sig)
        keep = torch.nonzero(lu < la)[:, 0][: int(limit - got)]
        if keep.numel():
            v = u[keep] * amp
            S += torch.stack([(v**p).sum() for p in (1, 2, 3, 4)])
            ex += int((v > 2.0 * math.sqrt(E0 / math.pi)).sum())
            peak = max(peak, float(v.max()))
            new = x[keep][: max(int(case["cap"]) - got, 0)]
            rows[got:got + new.shape[0]] = new
            got += keep.numel()
        if got >= limit:
            break
    S, cnt = S.cpu().numpy(), max(got * 4 * K, 1)
    m = S / cnt
    return {"counts": None, "moments": S, "hist": None, "peak_u": peak, "index": None,
            "shape": np.array([m[2] / m[1] ** 1.5, m[3] / m[1] ** 2, ex / cnt]) if got else np.zeros(3),
            "xhat": rows}


def _exact_sir(case, seed):
    K, E0, beta = int(case["K"]), case["E0"], case["beta"]
    if case["n"] * K > 4e9 or K > 32:
        return None
    alpha = _alpha(K, beta)
    log_M = _log_M(K, E0, beta, case["c"], alpha, True)
    phi = _grid(K, "cuda")
    sig = torch.from_numpy(np.sqrt(_sigma2(K, beta))).cuda().repeat(2)
    amp = math.sqrt(2.0 * E0 / math.pi)
    W = W2 = mx = 0.0
    S = np.zeros(4)
    chunk = (1 << 25) // K
    for i0 in range(0, int(case["n"]), chunk):
        x, la, _, u = _proposals64(case, seed, i0, min(chunk, int(case["n"]) - i0), alpha, log_M, phi, sig)
        w = torch.exp(la)
        W, W2, mx = W + float(w.sum()), W2 + float((w * w).sum()), max(mx, float(w.max()))
        S += [float((w * (u * amp).pow(p).mean(1)).sum()) for p in (1, 2, 3, 4)]
    # the drawn indices follow the last bits of the weights: no value for them
    return {"sums": np.array([W, W2, W * W / W2, mx]), "moments": S / W, "over": None, "index": None, "xhat": None}


def _exact_extremes(case, seed):
    K, x = int(case["K"]), _rows(int(case["K"]), 40.0, int(case["n"]), int(case["stride"]), seed)
    phi, best = _grid(K, "cuda"), []
    for r in range(0, x.shape[0], 1 << 17):
        best.append((x[r:r + (1 << 17)].double() @ phi).max(1).values)
    u = torch.cat(best) * math.sqrt(2.0 * case["E0"] / math.pi)
    k = min(int(case["top_k"]), u.numel())
    return {"rows": None, "umax": torch.sort(u, descending=True).values[:k].cpu().numpy(), "jmax": None,
            "n_exceed": None}


def _exact_train(case, seed):
    """The Adam steps with torch's autograd in 64 bits."""
    K, H, P, dev = int(case["K"]), int(case["hidden"]), int(case["points"]), "cuda"
    no, S = 5 * K, 32
    W = torch.from_numpy(_train_weights(case, seed)).to(dev)
    eps = S * math.floor(0.2 * 2.0**32 / S) * 2.0**-32
    phi, k = _grid(K, dev), torch.arange(1, K + 1, device=dev).double()
    data = []
    for (beta, c), (acc, near) in zip(_train_points(case), _train_rows(case, seed)):
        a64 = torch.from_numpy(acc).to(dev).double()
        x = torch.cat([a64 / a64.norm(dim=1, keepdim=True), torch.from_numpy(near).to(dev)])
        lf, _ = _log_ratio(x, K, 1.0, beta, c, 1.0, False, phi)
        t = (x[:, :K] ** 2 + x[:, K:] ** 2) @ k**2
        gc = _alpha(K, beta) * beta / K**3
        lg = torch.log1p(gc * k * k).sum() - K * torch.log1p(gc * t)
        ls2 = torch.from_numpy(np.log(_sigma2(K, beta))).to(dev)
        z = torch.tensor([(beta - 40.0) / 20.0, 0.0, c * beta / 1e4 - 1.0], dtype=torch.float64, device=dev)
        data.append((x, lf, lg, ls2, z, acc.shape[0]))
    j = torch.arange(S, device=dev).double()
    cs, sn = (torch.cos(2 * math.pi / S * ((k[:, None] * j) % S)), torch.sin(2 * math.pi / S * ((k[:, None] * j) % S)))
    m, v = torch.zeros_like(W), torch.zeros_like(W)
    loss = None
    for step in range(1, int(case["steps"]) + 1):
        w = W.clone().requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(w, [3 * H, H, H * H, H, H * no, no])
        losses = []
        for x, lf, lg, ls2, z, n_acc in data:
            h = torch.tanh(torch.tanh(z @ W1.view(3, H) + b1) @ W2.view(H, H) + b2)
            o = h @ W3.view(H, no) + b3
            logd = ls2 + o[:K]
            V0 = torch.zeros((2 * K, 2), dtype=torch.float64, device=dev)
            V0[:K, 0] = V0[K:, 1] = 0.5 / math.sqrt(K)
            V = V0 + o[K:].view(2 * K, 2)
            a = torch.exp(-logd).repeat(2)
            G = torch.eye(2, dtype=torch.float64, device=dev) + V.T @ (a[:, None] * V)
            det = G[0, 0] * G[1, 1] - G[0, 1] * G[1, 0]
            aV = a[:, None] * V
            # R_j (A V): coordinate c of x enters R_j^T x
            Bc = cs[:, :, None] * aV[:K, None, :] + sn[:, :, None] * aV[K:, None, :]
            Bs = cs[:, :, None] * aV[K:, None, :] - sn[:, :, None] * aV[:K, None, :]
            y = (x @ torch.cat([Bc, Bs]).reshape(2 * K, 2 * S)).view(-1, S, 2)
            quad = (G[1, 1] * y[..., 0] ** 2 - 2.0 * G[0, 1] * y[..., 0] * y[..., 1] + G[0, 0] * y[..., 1] ** 2) / det
            qf = (x**2 @ a)[:, None] - quad
            lnet = torch.logsumexp(-K * torch.log(qf), 1) - math.log(S) - 0.5 * (2.0 * logd.sum() + torch.log(det))
            lmix = torch.logaddexp(math.log(eps) + lg, math.log1p(-eps) + lnet)
            losses.append(0.05 * torch.logsumexp((lf - lmix) / 0.05, 0) - 0.1 * lnet[:n_acc].mean())
        loss = torch.stack(losses)
        loss.sum().backward()
        g = w.grad
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        W = W - 3e-3 * (m / (1.0 - 0.9**step)) / (torch.sqrt(v / (1.0 - 0.999**step)) + 1e-8)
    return {"loss": loss.detach().cpu().numpy(), "weights": W.cpu().numpy()}


def exact(case, seed):
    """None where the accepted set takes too many 64-bit proposals (the large
    samples, the mixture, batches, sweeps and maps)."""
    fn = {"sample": _exact_sample, "sir": _exact_sir, "extremes": _exact_extremes, "train": _exact_train}
    return fn[case["kind"]](case, seed) if case["kind"] in fn else None
