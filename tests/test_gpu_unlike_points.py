"""Segments of each point's own size: a dense point's few accept words beside a
sparse point's many are cut finer.  Rows, indices, histograms and statistics of
each point of a batch or a sweep are those of the point sampled alone.
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


def _same(a, b):
    for k in ("n_accepted", "n_grid_values", "n_written"):
        assert a[k] == b[k], k
    assert np.array_equal(a["hist_u0"], b["hist_u0"])
    for k in ("S1", "S2", "S3", "S4"):
        # the same terms in another order: 1e9 of them at most
        assert abs(a[k] - b[k]) <= 1e-12 * max(b["S2"], b["S4"])


# (K, c, accepted or proposals wanted) per point, dense first
CASES = {"dense_and_sparse": [(32, 0.5, 200_000), (32, 250.0, 20)],
         "k64": [(64, 1.0, 150_000), (8, 60.0, 300), (64, 700.0, 30)],
         "one_dense_word": [(128, 1.0, 3), (16, 120.0, 400), (8, 1.0, 1)],
         "many": [(8, 2.0, 40_000)] * 40 + [(16, 150.0, 200)]}


@pytest.mark.parametrize("name", list(CASES))
def test_batch_points_are_the_single_ones(T, ctx, name):
    pts = [T.make_point(K, 1.0, 40.0, c, seed=9, point_id=i) for i, (K, c, _) in enumerate(CASES[name])]
    pls = [ctx.plan_batch([p], T.SIGMA, n_starts=8)[0][0] for p in pts]
    n = [w for _, _, w in CASES[name]]
    cap = [min(w, 500) for w in n]
    st, xh, ix = ctx.sample_batch(pts, n, plans=pls, mode=T.COUNT_ACCEPTED, max_proposals=1 << 27, capacity=cap)
    off = np.concatenate([[0], np.cumsum(cap)]).astype(int)
    for q, p in enumerate(pts):
        one = ctx.sample(p, n[q], plan=pls[q], mode=T.COUNT_ACCEPTED, max_proposals=1 << 27, capacity=cap[q])
        _same(st[q], one)
        w = one["n_written"]
        assert np.array_equal(ix[off[q]:off[q] + w].cpu().numpy(), one["index"].cpu().numpy()[:w])
        assert np.array_equal(xh[off[q]:off[q] + w].cpu().numpy()[:, : 2 * p.K], one["xhat"].cpu().numpy()[:w])
