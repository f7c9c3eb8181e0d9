"""The search for log M has a kernel for K <= 32, one for K <= 64 and one for
K <= 128, chosen by the largest K of the batch; a point's search is the same to
the bit in each, and its value is the objective at its maximiser.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_16952_amd import tkdv
    return tkdv


@pytest.mark.parametrize("K", [8, 16, 32, 64])
@pytest.mark.parametrize("uniform", [0, 1])
def test_a_points_search_does_not_depend_on_the_batch(T, K, uniform):
    prop = T.UNIFORM if uniform else T.SIGMA
    ctx = T.Context(0)
    try:
        pts = [T.make_point(K, 1.0, 25.0 + 5.0 * i, 2.0 * K * (i + 1), seed=1, point_id=i) for i in range(3)]
        alone, xa = ctx.plan_batch(pts, prop, n_starts=6, seed=3)
        for other in (64, 128):
            if other <= K:
                continue
            more = pts + [T.make_point(other, 1.0, 30.0, 50.0, seed=1, point_id=9)]
            both, xb = ctx.plan_batch(more, prop, n_starts=6, seed=3)
            for q in range(3):
                assert alone[q].log_M == both[q].log_M
                assert alone[q].n_optimiser_evals == both[q].n_optimiser_evals
                assert np.array_equal(xa[q], xb[q])
        for q, p in enumerate(pts):
            x = xa[q][: 2 * K]
            x = x / np.linalg.norm(x)
            want = oracle.log_ratio(x, 1.0, p.beta_p, p.c32, alone[q].alpha_star, 0 if uniform else 1)
            # FP64 sums of 1e2 terms in another order; the plan may add its margin above
            assert abs(want - alone[q].log_M) <= 1e-9 * max(1.0, abs(want))
    finally:
        ctx.close()
