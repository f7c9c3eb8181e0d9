"""The moment sums S1..S4 are a function of the accepted samples alone.

The same bits for one sequence of accepted samples however it was drawn: a point
alone or beside others, an accepted-count call (which decides some tiles past its
target, how many depends on timing) or the proposal-count call that ends at its
last sample, any launch.  And their values against 64 bits, from the rows that
the call wrote, where the ordered output's runs of ranks begin, end and change
length (R = 1, 2, 4, 8, 16 ranks a run up to 64, 128, 256, 2048 or 4096, 8192
samples and so on, to 2^21 samples for R = 256).

A row's coordinates are FP32 and a grid value is an FP32 product of 2K terms:
within tol = 2e-6 sqrt(K) amp of its 64-bit value.  So a sum of p-th powers is
within the sum of p |u|^(p-1) tol (taken 1.01 times, for the higher orders in tol).
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SUMS = ("S1", "S2", "S3", "S4")


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_16952_amd import tkdv
    return tkdv


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def _plan(T, ctx, pt):
    return ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]


def _equal(a, b):
    assert a["n_accepted"] == b["n_accepted"] > 0
    for k in SUMS:
        assert a[k] == b[k], (k, a[k], b[k])


@pytest.mark.parametrize("K,beta,c,n", [(8, 40.0, 20.0, 1_000_000), (16, 20.0, 0.5, 200_003), (32, 40.0, 75.0, 1_000_000),
                                        (64, 40.0, 150.0, 500_001), (128, 20.0, 300.0, 100_000)])
def test_a_point_beside_others(T, ctx, K, beta, c, n):
    pt = T.make_point(K, 1.0, beta, c, seed=3, point_id=2)
    pl = _plan(T, ctx, pt)
    one = ctx.sample(pt, n, plan=pl, capacity=64)
    for others in ([(8, 0.5, 2_000_000)], [(K, c, n)] * 23, [(16, 30.0, 30_000_000), (64, 100.0, 40_000)]):
        pts = [pt] + [T.make_point(k, 1.0, 40.0, cc, seed=7, point_id=10 + q) for q, (k, cc, _) in enumerate(others)]
        plans = [pl] + ctx.plan_batch(pts[1:], T.SIGMA, n_starts=8)[0]
        out, _, _ = ctx.sample_batch(pts, [n] + [m for _, _, m in others], plans=plans, capacity=[64] * len(pts))
        _equal(out[0], one)


@pytest.mark.parametrize("n_points", [65, 1500])
def test_many_points(T, ctx, n_points):
    """More points than lanes, and than threads of the kernel that lays out the runs; some accept nothing."""
    rng = np.random.default_rng(n_points)
    pts = [T.make_point(int(rng.choice([8, 16, 32, 64])), 1.0, 40.0, float(rng.choice([0.5, 20.0, 60.0])), seed=3, point_id=i)
           for i in range(n_points)]
    plans = ctx.plan_batch(pts, T.SIGMA, n_starts=4)[0]
    n = [int(v) for v in rng.integers(1, 3000, n_points)]
    out, xh, ix = ctx.sample_batch(pts, n, plans=plans, capacity=n)
    off = np.concatenate([[0], np.cumsum(n)]).astype(int)
    assert any(o["n_accepted"] == 0 for o in out) and any(o["n_accepted"] > 500 for o in out)
    for q in sorted(set(rng.integers(0, n_points, 40).tolist() + [0, 63, 64, n_points - 1])):
        one = ctx.sample(pts[q], n[q], plan=plans[q], capacity=n[q])
        w = one["n_written"]
        assert out[q]["n_accepted"] == one["n_accepted"] == w and out[q]["n_proposed"] == n[q]
        assert all(out[q][k] == one[k] for k in SUMS + ("n_exceed_2sigma", "peak_u", "peak_index")), q
        assert np.array_equal(ix[off[q]:off[q] + w].cpu().numpy(), one["index"].cpu().numpy())
        assert np.array_equal(xh[off[q]:off[q] + w, : 2 * pts[q].K].cpu().numpy(), one["xhat"].cpu().numpy())


@pytest.mark.parametrize("K,c,targets", [(8, 20.0, (1, 2_900)), (16, 0.0, (33, 65_536, 1_000_000)),
                                         (32, 75.0, (500, 30_000)), (64, 1.0, (8_193, 200_000)), (128, 1.0, (17, 60_000))])
def test_accepted_count_calls(T, ctx, K, c, targets):
    pt = T.make_point(K, 1.0, 20.0, c, seed=6, point_id=1)
    pl = _plan(T, ctx, pt)
    for n in targets:
        runs = [ctx.sample(pt, n, plan=pl, mode=T.COUNT_ACCEPTED, max_proposals=1 << 32, capacity=8) for _ in range(4)]
        assert all(r["n_accepted"] == n for r in runs)
        whole = ctx.sample(pt, runs[0]["n_proposed"], plan=pl, capacity=8)
        for r in runs:
            _equal(r, whole)


@pytest.mark.parametrize("K,beta,c,n", [(8, 40.0, 60.0, 1 << 28), (8, 60.0, 90.0, 1 << 30), (16, 40.0, 120.0, 1 << 27),
                                        (32, 40.0, 400.0, 1 << 28), (64, 40.0, 1000.0, 1 << 27),
                                        (128, 40.0, 3000.0, 1 << 27)])
def test_hardly_any_accepted(T, ctx, K, beta, c, n):
    """One in 1e6 to 1e9: runs read past many segments without an accepted proposal."""
    pt = T.make_point(K, 1.0, beta, c, seed=2, point_id=3)
    pl = _plan(T, ctx, pt)
    d = ctx.sample(pt, n, plan=pl, capacity=4096)
    idx = d["index"].cpu().numpy()
    assert 0 < d["n_accepted"] == len(idx) == int(d["hist_u0"].sum()) and np.all(np.diff(idx) > 0)
    # up to each third sample alone: the shorter calls cut the words otherwise
    for q in range(len(idx) - 1, max(len(idx) - 20, -1), -3):
        part = ctx.sample(pt, int(idx[q]) + 1, plan=pl, capacity=4096)
        assert np.array_equal(part["index"].cpu().numpy(), idx[:q + 1])
    _equal(ctx.sample(pt, int(idx[-1]) + 1, plan=pl, capacity=4096), d)
    a = ctx.sample(pt, len(idx), plan=pl, mode=T.COUNT_ACCEPTED, max_proposals=n, capacity=4096)
    assert np.array_equal(a["index"].cpu().numpy(), idx)
    _equal(a, d)


def test_mixture_accepted_count(T, ctx):
    K = 32
    pt = T.make_point(K, 1.0, 40.0, 100.0, seed=5, point_id=4)
    pl = T.plan_point(pt, T.SIGMA)
    logd = np.log(np.array(pl.sigma2[:K])) + 0.05 * np.sin(np.arange(1, K + 1))
    V = 0.4 * np.sin(np.arange(2 * K * 2).reshape(2 * K, 2) + 0.5) / np.sqrt(K)
    mx = T.make_mixture(K, 0.2, logd, V)
    mpl, _ = T.plan_mixture(pt, pl, mx, margin=0.02)
    runs = [ctx.sample_mixture(pt, mpl, mx, 2_000, mode=T.COUNT_ACCEPTED, max_proposals=1 << 30, capacity=8)
            for _ in range(3)]
    whole = ctx.sample_mixture(pt, mpl, mx, runs[0]["n_proposed"], capacity=8)
    for r in runs:
        _equal(r, whole)


EDGES = (1, 64, 65, 127, 129, 256, 257, 2_048, 2_049, 4_096, 4_097, 8_191, 8_192, 8_193, 16_384, 16_385, 32_769, 65_536, 65_537,
         131_072, 131_073)


@pytest.mark.parametrize("K,c", [(8, 1.0), (16, 1.0), (32, 1.0), (64, 1.0), (128, 1.0), (32, 60.0)])
def test_values_at_the_edges_of_runs(T, ctx, K, c):
    import torch
    E0 = 1.5
    pt = T.make_point(K, E0, 20.0, c, seed=4, point_id=1)
    pl = _plan(T, ctx, pt)
    N, amp = 4 * K, math.sqrt(2 * E0 / math.pi)
    k = torch.arange(1, K + 1, device="cuda")[:, None]
    ang = -math.pi * k + 2 * math.pi / N * ((k * torch.arange(N, device="cuda")) % N)
    phi = torch.cat([torch.cos(ang.double()), torch.sin(ang.double())])
    tol = 2e-6 * math.sqrt(K) * amp
    for n in EDGES:
        d = ctx.sample(pt, n, plan=pl, mode=T.COUNT_ACCEPTED, max_proposals=1 << 30, capacity=n)
        assert d["n_accepted"] == d["n_written"] == n
        assert int(d["hist_u0"].sum()) == n and d["n_grid_values"] == n * N
        S, B = np.zeros(4), np.zeros(4)
        for r in range(0, n, 1 << 14):
            u = amp * (d["xhat"][r:r + (1 << 14)].double() @ phi)
            S += [float((u**p).sum()) for p in (1, 2, 3, 4)]
            B += [float((p * u.abs() ** (p - 1)).sum()) for p in (1, 2, 3, 4)]
        for p in range(4):
            assert abs(d[SUMS[p]] - S[p]) <= 1.01 * tol * B[p], (n, p + 1, d[SUMS[p]], S[p])
