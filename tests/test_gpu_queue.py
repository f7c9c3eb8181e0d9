"""How the decision kernels divide a range among the waves: dealt out evenly up
to 2^20 tiles (2^25 proposals) per call, claimed from queues above, and stopped
early in accepted-count mode.  The division must not show: the accepted
indices and rows of one range are those of any other call that covers it.
"""
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


def _point(T, ctx, K, beta, c, pid=1):
    pt = T.make_point(K, 1.0, beta, c, seed=31, point_id=pid)
    return pt, ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]


@pytest.mark.parametrize("K,beta,c", [(8, 40.0, 20.0), (32, 40.0, 120.0)])
def test_claimed_range_equals_the_dealt_one(T, ctx, K, beta, c):
    pt, pl = _point(T, ctx, K, beta, c)
    n0, n1 = 1 << 25, (1 << 25) + 77   # 2^20 tiles: dealt out; three more: claimed
    a = ctx.sample(pt, n0, plan=pl, capacity=1 << 18)
    b = ctx.sample(pt, n1, plan=pl, capacity=1 << 18)
    ia, ib = a["index"].cpu().numpy(), b["index"].cpu().numpy()
    m = int(np.searchsorted(ib, n0))
    assert m == a["n_accepted"] == len(ia) and b["n_proposed"] == n1
    assert np.array_equal(ia, ib[:m])
    assert np.array_equal(a["xhat"].cpu().numpy(), b["xhat"].cpu().numpy()[:m])
    assert (ib[m:] < n1).all()


@pytest.mark.parametrize("K,beta,c,n", [(16, 20.0, 0.0, 1), (16, 20.0, 0.0, 200_001), (8, 40.0, 20.0, 20_000),
                                        (64, 20.0, 300.0, 3_000), (128, 20.0, 1200.0, 500)])
def test_accepted_count_is_the_prefix(T, ctx, K, beta, c, n):
    pt, pl = _point(T, ctx, K, beta, c)
    a = ctx.sample(pt, n, plan=pl, mode=T.COUNT_ACCEPTED, max_proposals=1 << 32, capacity=n)
    assert a["n_accepted"] == a["n_written"] == n
    b = ctx.sample(pt, a["n_proposed"], plan=pl, capacity=n)
    assert b["n_accepted"] == n
    assert np.array_equal(a["index"].cpu().numpy(), b["index"].cpu().numpy())
    assert a["n_proposed"] == int(b["index"][-1]) + 1
    for k in ("S2", "S3", "S4"):
        assert abs(a[k] - b[k]) <= 1e-12 * abs(b["S2"])
    assert np.array_equal(a["hist_u0"], b["hist_u0"])


def test_batch_of_dealt_and_claimed_points(T, ctx):
    cfg = [(8, 40.0, 20.0, 7_000_001), (32, 40.0, 120.0, 33), (8, 40.0, 20.0, 64), (64, 20.0, 300.0, 400_003),
           (16, 40.0, 30.0, 6_900_000), (8, 30.0, 10.0, 1)]
    pts, plans = zip(*[_point(T, ctx, K, b, c, pid=q) for q, (K, b, c, _) in enumerate(cfg)])
    n = [m for *_, m in cfg]
    out, _, _ = ctx.sample_batch(list(pts), n, plans=list(plans), capacity=[min(m, 1 << 18) for m in n])
    for pt, pl, m, o in zip(pts, plans, n, out):
        s = ctx.sample(pt, m, plan=pl, capacity=min(m, 1 << 18))
        assert o["n_accepted"] == s["n_accepted"] and o["n_proposed"] == m
        assert np.array_equal(o["index"].cpu().numpy(), s["index"].cpu().numpy())
        assert np.array_equal(o["xhat"].cpu().numpy(), s["xhat"].cpu().numpy())
