"""The FP64 re-decision on K/2 lanes per proposal (k_fixup) against the oracle.

Points at C3/C2 = 0 send most proposals to within the decision window of the
bound (log a near 0 for the paper's proposal), so the re-decision settles a
large share of them; the list of a mixed-K batch holds every K at once.
Decisions equal the oracle's FP64 ones except within 1e-9 of the threshold.
"""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

AMBIG = 1e-9


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_16952_amd import tkdv
    return tkdv


def _check(pt, plan, n, index, n_fix):
    K = pt.K
    o = oracle.sample(K, pt.E0, pt.beta_p, pt.c32, 1, plan.alpha_star, plan.log_M, pt.seed, pt.point_id, n, 4 * K,
                      want_log=True)
    amb = np.abs(o["log_u"] - o["log_a"]) < AMBIG
    acc = np.zeros(n, dtype=bool)
    acc[index] = True
    print(f"K={K} c={pt.c32} n={n}: {n_fix} re-decided, {int(acc.sum())} accepted", flush=True)
    sys.stdout.flush()
    assert n_fix > 0
    assert not ((acc != o["accept"].astype(bool)) & ~amb).any()


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("K,c,n", [(8, 0.0, 60_001), (16, 0.0, 30_001), (32, 0.0, 20_001), (64, 0.0, 8_001),
                                   (128, 0.0, 4_001), (8, 5.0, 60_001), (128, 200.0, 4_001)])
def test_redecisions_equal_the_oracle(T, K, c, n, prec):
    ctx = T.Context(0)
    pt = T.make_point(K, 1.0, 20.0, c, seed=19, point_id=K)
    plan = ctx.plan_batch([pt], T.SIGMA, n_starts=4)[0][0]
    r = ctx.sample(pt, n, plan=plan, precision=T.PRECISIONS[prec], capacity=n)
    _check(pt, plan, n, r["index"].cpu().numpy(), r["n_fp64_fixups"])
    ctx.close()


def test_mixed_list(T):
    ctx = T.Context(0)
    Ks = [128, 8, 64, 16, 32, 8]
    pts = [T.make_point(K, 1.0, 25.0, 0.0, seed=5, point_id=q) for q, K in enumerate(Ks)]
    plans, _ = ctx.plan_batch(pts, T.SIGMA)
    n = [3_001, 40_003, 6_001, 30_001, 20_005, 17]
    out, _, _ = ctx.sample_batch(pts, n, plans=plans, capacity=n)
    for p, pl, m, o in zip(pts[:5], plans, n, out):
        _check(p, pl, m, o["index"].cpu().numpy(), o["n_fp64_fixups"])
    ctx.close()
