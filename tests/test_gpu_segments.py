"""The ordered output over segments of every size (8 to 2048 accept words).

Statistics against the rows and indices that the same call wrote: moments,
exceedances, histogram and peak recomputed in 64 bits with torch from the FP32
rows, for ranges whose segments are the shortest, intermediate and the longest,
dense and sparse, with the target inside a segment, and a mixed-K batch.
Rows carry a relative error of a few 2^-24 per coordinate, so a grid value is
within 2e-6 sqrt(K) of its 64-bit value, and sums of n of them within that times n.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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


def _check(d, K, E0):
    import torch
    x, idx = d["xhat"], d["index"]
    n = d["n_accepted"]
    assert d["n_written"] == n == x.shape[0]
    if n == 0:
        return
    assert bool((idx[1:] > idx[:-1]).all()) and int(idx[-1]) < d["n_proposed"]
    N = 4 * K
    k = torch.arange(1, K + 1, device=x.device)[:, None]
    ang = -math.pi * k + 2 * math.pi / N * ((k * torch.arange(N, device=x.device)) % N)
    phi = torch.cat([torch.cos(ang.double()), torch.sin(ang.double())])
    amp, sd = math.sqrt(2 * E0 / math.pi), math.sqrt(E0 / math.pi)
    S, ex2, ex4, smp4, mx = np.zeros(4), [0, 0], [0, 0], [0, 0], []
    tol = 2e-6 * math.sqrt(K) * amp
    hist = torch.zeros(64, dtype=torch.int64, device=x.device)
    for r in range(0, n, 1 << 16):
        xr = x[r:r + (1 << 16)].double()
        u = amp * (xr @ phi)
        S += [float((u**p).sum()) for p in (1, 2, 3, 4)]
        m = u.max(1).values
        mx.append(m)
        for q, t in enumerate((-tol, tol)):
            ex2[q] += int((u > 2 * sd - t).sum())
            ex4[q] += int((u > 4 * sd - t).sum())
            smp4[q] += int((m > 4 * sd - t).sum())
        b = ((xr[:, :K].sum(1) / math.sqrt(K) + 1.0) * 32).floor().clamp(0, 63).long()
        hist += torch.bincount(b, minlength=64)
    umax = math.sqrt(2 * K * E0 / math.pi)
    for p in range(4):
        assert abs(d[f"S{p + 1}"] - S[p]) <= n * N * tol * (p + 1) * umax**p, (p, d[f"S{p + 1}"], S[p])
    assert ex2[0] <= d["n_exceed_2sigma"] <= ex2[1]
    assert ex4[0] <= d["n_exceed_4sigma"] <= ex4[1]
    assert smp4[0] <= d["n_samples_4sigma"] <= smp4[1]
    mx = torch.cat(mx)
    assert abs(d["peak_u"] - float(mx.max())) <= tol
    at = int((idx == int(d["peak_index"])).nonzero()[0])
    assert float(mx[at]) >= float(mx.max()) - 2 * tol
    h = hist.cpu().numpy()
    assert d["hist_u0"].sum() == n and np.abs(d["hist_u0"].astype(np.int64) - h).sum() <= 2 + 1e-4 * n


@pytest.mark.parametrize("K,beta,c,n", [
    (8, 40.0, 20.0, 1), (16, 20.0, 0.0, 255), (16, 20.0, 0.0, 257), (32, 20.0, 0.0, 300_001),  # 8 words, dense
    (32, 40.0, 150.0, 3_000_001),       # 16 words, sparse
    (64, 40.0, 300.0, 2_500_000), (128, 20.0, 1500.0, 500_003),
    (8, 40.0, 20.0, 100_000_007),       # 512 words
    (8, 40.0, 25.0, (1 << 29) + 1)])    # 2048 words
def test_statistics_equal_the_rows(T, ctx, K, beta, c, n):
    pt = T.make_point(K, 1.0, beta, c, seed=2, point_id=9)
    pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
    _check(ctx.sample(pt, n, plan=pl, capacity=min(n, 1 << 21)), K, 1.0)


@pytest.mark.parametrize("K,c,n", [(16, 0.0, 1), (16, 0.0, 100_003), (64, 0.0, 40_001), (32, 100.0, 5_000)])
def test_statistics_stop_at_the_target(T, ctx, K, c, n):
    pt = T.make_point(K, 2.0, 25.0, c, seed=4, point_id=1)
    pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
    d = ctx.sample(pt, n, plan=pl, mode=T.COUNT_ACCEPTED, max_proposals=1 << 30, capacity=n)
    assert d["n_accepted"] == n
    _check(d, K, 2.0)


def test_batch_with_empty_points(T, ctx):
    cfg = [(8, 20.0, 0.0, 5_000), (128, 40.0, 2000.0, 3), (64, 20.0, 0.0, 9_999), (16, 40.0, 60.0, 64),
           (32, 20.0, 0.0, 70_001), (8, 60.0, 60.0, 2)]
    pts = [T.make_point(K, 1.0, b, c, seed=8, point_id=q) for q, (K, b, c, _) in enumerate(cfg)]
    plans, _ = ctx.plan_batch(pts, T.SIGMA, n_starts=8)
    n = [m for *_, m in cfg]
    out, _, _ = ctx.sample_batch(pts, n, plans=plans, capacity=n)
    for p, m, o in zip(pts, n, out):
        assert o["n_proposed"] == m
        _check(o, p.K, 1.0)
