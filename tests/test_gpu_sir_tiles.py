"""Importance weights settle two tiles at once, over several rounds of
workgroups; the resampling looks at up to 64 tiles per wave before it goes
through those with draws.  Ranges around a tile, around the pairs and around
the waves' shares, with draws fewer and many more than tiles: weights do not
depend on the range, totals are the weights' sums, and the draws are the
systematic ones.
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


@pytest.mark.parametrize("K,prec", [(8, "bf16x3"), (16, "fp32"), (32, "bf16x3"), (64, "bf16x3"), (128, "fp32")])
@pytest.mark.parametrize("n,m", [(1, 3), (31, 5), (33, 40), (64, 1), (97, 1000), (131_072, 7), (131_105, 200_000),
                                 (1_000_003, 1_000), (4_200_001, 100_000)])
def test_weights_and_draws(T, ctx, K, prec, n, m):
    pt = T.make_point(K, 1.0, 30.0, 0.6 * K, seed=12, point_id=4)
    pl = ctx.plan_batch([pt], T.SIGMA, n_starts=6)[0][0]
    u0 = 0.3
    r = ctx.sir(pt, n, m, u0=u0, plan=pl, precision=T.PRECISIONS[prec], rows=m <= 1000, weights=True)
    w = r["weights"].cpu().numpy().astype(np.float64)
    if n <= 131_105:
        more = ctx.sir(pt, n + 77, 0, plan=pl, precision=T.PRECISIONS[prec], weights=True)
        assert np.array_equal(more["weights"].cpu().numpy()[:n].astype(np.float64), w)
    W = w.sum()
    # FP64 sums of n positive terms in two orders
    assert abs(r["W"] - W) <= n * 2.0**-52 * W and abs(r["W2"] - (w * w).sum()) <= n * 2.0**-52 * (w * w).sum()
    assert r["max_w"] == w.max()
    idx = r["index"].cpu().numpy()[:m]
    assert (np.diff(idx) >= 0).all() and idx[0] >= 0 and idx[-1] < n
    # draw q takes the proposal whose cumulative interval holds (u0 + q) W/m; an
    # index may differ only where the point is at a boundary to rounding
    c = np.cumsum(w)
    at = (u0 + np.arange(m)) * (W / m)
    want = np.minimum(np.searchsorted(c, at, side="right"), n - 1)
    off = np.nonzero(idx != want)[0]
    tol = n * 2.0**-51 * W
    for q in off:
        lo, hi = sorted((int(idx[q]), int(want[q])))
        assert abs(at[q] - c[lo]) <= tol or abs(at[q] - c[hi - 1]) <= tol
    if m <= 1000:
        x = r["xhat"].cpu().numpy()[:m].astype(np.float64)
        assert np.allclose((x * x).sum(1), 1.0, atol=2 * K * 2.0**-23)
