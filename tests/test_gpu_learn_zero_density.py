"""Training rows where the target's density underflows to 0 (log f = -inf) have no
part in the soft maximum, wherever they come among a lane's rows: the loss and the
gradients are those without them.
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


@pytest.mark.parametrize("first", ["zero", "finite"])
def test_rows_of_no_density(T, first):
    K, tiles = 8, 3 * 2048   # tiles of 16 rows, some three to a chunk
    ctx = T.Context(0)
    try:
        # C3/C2 H3 overflows: rows with H3 < 0 have log f = -inf, those of a
        # single mode H3 = 0
        pt = T.make_point(K, 1e4, 40.0, 4e304)
        sp = T.plan_point(T.make_point(K, 1e4, 40.0, 0.0), T.SIGMA)
        rng = np.random.default_rng(3)
        a = rng.uniform(0.0, 2.0 * np.pi, 16 * tiles)
        finite = np.zeros((16 * tiles, 2 * K))
        finite[:, 0], finite[:, K] = np.cos(a), np.sin(a)
        zero = np.zeros((16, 2 * K))
        zero[:, 0], zero[:, 1] = 0.8, -0.6
        res = []
        for with_zero in (False, True):
            L = T.Learner(ctx, T.learner_cfg(K, hidden=16, eps=0.2, v_amp=0.5, v_scale=0.8, temperature=0.3,
                                             nll_weight=0.4))
            L.set_points([pt], [sp])
            rows = finite.reshape(tiles, 16, 2 * K)[0 if first == "finite" else 1::2]
            if with_zero:
                both = [rows, np.broadcast_to(zero, rows.shape)]
                rows = np.stack(both if first == "finite" else both[::-1], axis=1)
            L.add_rows(0, np.ascontiguousarray(rows.reshape(-1, 2 * K)), kind=1)
            res.append(L.gradients())
            L.close()
        for u, v in zip(*res):
            assert np.isfinite(u).all()
            # sums of some 1e5 terms in another order
            assert np.abs(u - v).max() <= 1e-11 * max(np.abs(u).max(), 1e-300), (u, v)
    finally:
        ctx.close()
