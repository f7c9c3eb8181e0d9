"""The training step's kernels at the edges of their tiles (16 rows), chunks
(whole tiles of one point, dealt out over the waves of the chip), rows of each
kind and sizes of the hidden layer: losses against the oracle's, gradients
against central differences of the oracle's loss along random directions, and
one Adam step against the update of those gradients.
"""
import numpy as np
import pytest

from oracle import learned as OL

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


# rows of kinds 0, 1, 2 per point
SIZES = {"one": [(1, 0, 0)], "tile": [(16, 0, 0), (15, 0, 1)], "tile+1": [(16, 1, 0), (17, 0, 0)],
         "no_maximum": [(0, 0, 20), (3, 2, 1)], "no_likelihood": [(0, 33, 0)], "empty": [(5, 0, 0), (0, 0, 0), (31, 0, 2)]}


def _learner(T, ctx, K, H, sizes, seed):
    rng = np.random.default_rng(seed)
    L = T.Learner(ctx, T.learner_cfg(K, hidden=H, eps=0.2, v_amp=0.5, v_scale=0.8, temperature=0.3, nll_weight=0.4))
    W = 0.1 * rng.standard_normal(L.n_weights)
    L.set_weights(W)
    opts = [(1.0, 30.0 + 7.0 * i, 40.0 - 5.0 * i) for i in range(len(sizes))]
    pts = [T.make_point(K, E0, bp, c) for E0, bp, c in opts]
    sps = [T.plan_point(p, T.SIGMA) for p in pts]
    L.set_points(pts, sps)
    rows, kinds = [], []
    for i, ns in enumerate(sizes):
        X = rng.standard_normal((sum(ns), 2 * K))
        X /= np.linalg.norm(X, axis=1)[:, None]
        o = 0
        for kd, n in enumerate(ns):
            if n:
                L.add_rows(i, X[o:o + n], kind=kd)
            o += n
        rows.append(X)
        kinds.append([kd for kd, n in enumerate(ns) for _ in range(n)])
    return L, W, opts, [(sp.alpha_star, np.array(sp.sigma2[:K])) for sp in sps], rows, kinds


def _point_loss(K, o, plan, X, kd, mix):
    if not len(kd):
        return 0.0
    if all(k == 2 for k in kd):  # the oracle's soft maximum needs a row: its share taken off
        extra = OL.point_loss(K, *o[:1], o[1], o[2], plan[0], 0.2, *mix, X[:1], [1], 0.3, 0.4)
        return OL.point_loss(K, *o[:1], o[1], o[2], plan[0], 0.2, *mix, np.concatenate([X, X[:1]]), list(kd) + [1], 0.3,
                             0.4) - extra
    return OL.point_loss(K, o[0], o[1], o[2], plan[0], 0.2, *mix, X, kd, 0.3, 0.4)


def _losses(K, H, W, opts, plans, rows, kinds):
    out = []
    for o, pl, X, kd in zip(opts, plans, rows, kinds):
        mix = OL.mixture_params(OL.network(W, H, K, OL.features(o[1], o[0], o[2])), K, pl[1], 0.5, 0.8)
        out.append(_point_loss(K, o, pl, X, kd, mix))
    return np.array(out)


@pytest.mark.parametrize("K", [8, 16, 32])
@pytest.mark.parametrize("name,H", [("one", 12), ("tile", 64), ("tile+1", 256), ("no_maximum", 33), ("no_likelihood", 200),
                                    ("empty", 5)])
def test_step_against_the_oracle(T, ctx, K, name, H):
    L, W, opts, plans, rows, kinds = _learner(T, ctx, K, H, SIZES[name], 3)
    try:
        loss, _, gw = L.gradients()
        want = _losses(K, H, W, opts, plans, rows, kinds)
        # r/T up to 1e2 and 1e2 summands of rounding 2^-53 each
        assert np.allclose(loss, want, rtol=1e-11, atol=1e-10)
        rng = np.random.default_rng(4)
        for _ in range(2):
            d = rng.standard_normal(W.size)
            h = 1e-5
            fd = (_losses(K, H, W + h * d, opts, plans, rows, kinds).sum()
                  - _losses(K, H, W - h * d, opts, plans, rows, kinds).sum()) / (2.0 * h)
            # the difference quotient: h^2 of the third derivative, and 1e-10/h of the losses' rounding
            assert abs(gw @ d - fd) <= 1e-5 * (np.abs(gw * d).sum() + 1.0)
        L.train(1)
        lr, eps = L.cfg.lr, L.cfg.adam_eps
        step = lr * gw / (np.abs(gw) + eps)  # the first step: both moments are the gradient's own
        assert np.allclose(L.get_weights(), W - step, rtol=1e-12, atol=1e-12)
    finally:
        L.close()


@pytest.mark.parametrize("K,rows,points", [(8, 16 * 2100, 1), (32, 16 * 700 + 5, 3), (16, 40000, 2)])
def test_rows_beyond_the_waves(T, ctx, K, rows, points):
    """More tiles than waves: the losses and gradients are those of the rows in
    two learners' halves of the points' sums (soft maxima merged by hand)."""
    rng = np.random.default_rng(7)
    X = rng.standard_normal((points, rows, 2 * K))
    X /= np.linalg.norm(X, axis=2)[:, :, None]
    pts = [T.make_point(K, 1.0, 30.0 + 3.0 * i, 30.0) for i in range(points)]
    sps = [T.plan_point(p, T.SIGMA) for p in pts]

    def run(cut):
        L = T.Learner(ctx, T.learner_cfg(K, hidden=16, eps=0.2, v_amp=0.5, v_scale=0.8, temperature=0.3, nll_weight=0.0))
        L.set_weights(0.1 * np.random.default_rng(1).standard_normal(L.n_weights))
        L.set_points(pts, sps)
        for i in range(points):
            L.add_rows(i, X[i, cut], kind=0)
        out = L.gradients()
        L.close()
        return out
    whole = run(slice(0, rows))
    a, b = run(slice(0, rows // 3)), run(slice(rows // 3, rows))
    t = 0.3
    want = t * np.logaddexp(a[0] / t, b[0] / t)
    assert np.allclose(whole[0], want, rtol=1e-11)
    wa = np.exp((a[0] - want) / t)[:, None]
    g = wa * a[1] + (1.0 - wa) * b[1]
    assert np.allclose(whole[1], g, rtol=1e-8, atol=1e-9 * np.abs(g).max())
