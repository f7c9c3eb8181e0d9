"""An exact M is not found broken by rounding: C3/C2 = 0, whose M has a closed form.

The supremum of f/(M g) is attained there, so that among some 3e7 proposals at
K = 128 one comes within FP64 rounding of it; a log a of a few 1e-14 is no violation
and M stays as planned.  An M too small by more than rounding is still found.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_16952_amd import tkdv
    return tkdv


@pytest.mark.parametrize("K,beta,n,seeds", [(8, 40.0, 50_000_000, 4), (32, 60.0, 50_000_000, 4), (64, 40.0, 50_000_000, 4),
                                            (128, 20.0, 30_000_000, 4), (128, 40.0, 30_000_000, 16)])
def test_rounding_is_no_violation(T, K, beta, n, seeds):
    ctx = T.Context(0)
    try:
        for seed in range(seeds):
            pt = T.make_point(K, 1.0, beta, 0.0, seed=seed, point_id=3)
            pl = T.plan_point(pt, T.SIGMA)
            d = ctx.sample(pt, n, plan=pl, capacity=1)
            assert d["n_M_violations"] == 0 and d["M_raises"] == 0, (seed, d["max_log_a"])
            assert d["log_M_used"] == pl.log_M
    finally:
        ctx.close()


@pytest.mark.parametrize("K", [8, 16, 32, 64, 128])
def test_a_small_excess_is(T, K):
    ctx = T.Context(0)
    try:
        ctx.set_violation_policy(T.MV_COUNT)
        pt = T.make_point(K, 1.0, 40.0, 0.0, seed=1, point_id=3)
        pl = T.plan_point(pt, T.SIGMA)
        pl.log_M -= 1e-8
        d = ctx.sample(pt, 20_000_000, plan=pl, capacity=1)
        assert d["n_M_violations"] > 0 and d["log_M_used"] == pl.log_M
    finally:
        ctx.close()
