"""The decision kernels settle their tiles in groups (two tiles of 32, four of
16).  A claim that is no multiple of the group draws tiles past its end, and
these must not be counted: with log M set too low many proposals violate the
bound, and their count over a range of odd claims is that of the same range
dealt out in whole groups.  A single wave's ragged ends are the smallest ranges.
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
    c.set_violation_policy(T.MV_COUNT)
    yield c
    c.close()


def _point(T, ctx, K, c):
    pt = T.make_point(K, 1.0, 40.0, c, seed=31, point_id=1)
    pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
    pl.log_M -= 2.0  # near c = 0 every log a is close to 0: most proposals then violate
    return pt, pl


@pytest.mark.parametrize("K,c,prec", [(8, 1.0, 0), (32, 1.0, 0), (32, 1.0, 1), (64, 1.0, 0), (128, 1.0, 0)])
def test_claims_count_their_own_proposals(T, ctx, K, c, prec):
    prec = T.FP32 if prec else T.BF16X3
    pt, pl = _point(T, ctx, K, c)
    n0, n1 = 1 << 25, (1 << 25) + 33  # 2^20 tiles are dealt out in groups; two more: all are claimed
    a = ctx.sample(pt, n0, plan=pl, precision=prec)
    b = ctx.sample(pt, n1, plan=pl, precision=prec)
    assert a["n_M_violations"] > 1000
    assert 0 <= b["n_M_violations"] - a["n_M_violations"] <= n1 - n0
    assert 0 <= b["n_accepted"] - a["n_accepted"] <= n1 - n0
    assert b["max_log_a"] >= a["max_log_a"]


@pytest.mark.parametrize("K", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 97, 2049])
def test_ragged_ends(T, ctx, K, n):
    pt, pl = _point(T, ctx, K, 0.5 * K)
    whole = ctx.sample(pt, 4096, plan=pl, capacity=4096)
    part = ctx.sample(pt, n, plan=pl, capacity=4096)
    idx = whole["index"].cpu().numpy()
    m = int(np.searchsorted(idx, n))
    assert part["n_accepted"] == m
    assert np.array_equal(part["index"].cpu().numpy(), idx[:m])
    assert np.array_equal(part["xhat"].cpu().numpy(), whole["xhat"].cpu().numpy()[:m])
