"""Proposals for the FP64 pass: a workgroup keeps up to 256 of them in LDS and
reserves the list once, claims beyond that reserve it themselves.  Near the
linear law a hundredth of the proposals is listed: every accepted index of a
range is that of the same range decided in parts, from no listed proposal at
all over workgroups just below and above their 256 to long ranges, and the
number listed adds up.
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


@pytest.mark.parametrize("K,prec", [(8, "bf16x3"), (16, "fp32"), (32, "bf16x3"), (64, "bf16x3"), (128, "bf16x3")])
def test_listed_proposals(T, K, prec):
    prec = T.PRECISIONS[prec]
    ctx = T.Context(0)
    try:
        pt = T.make_point(K, 1.0, 20.0, 0.5, seed=5, point_id=3)
        pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
        sizes = (40, 4_000, 1 << 18, 3_000_017, (1 << 26) + 99 if K < 64 else 9_000_001)
        runs = [ctx.sample(pt, n, plan=pl, precision=prec, capacity=n if n < 4_000_000 else 1 << 22) for n in sizes]
        last = runs[-1]
        idx = last["index"].cpu().numpy()
        for n, r in zip(sizes[:-1], runs[:-1]):
            m = int(np.searchsorted(idx, n))
            assert r["n_accepted"] == m
            assert np.array_equal(r["index"].cpu().numpy(), idx[:m])
        listed = [r["n_fp64_fixups"] for r in runs]
        assert all(a <= b for a, b in zip(listed, listed[1:]))
        # a share of some 1e-2 of the proposals, the same in every run (5 sigma of the smaller count)
        for n, c in zip(sizes[2:], listed[2:]):
            assert abs(c / n - listed[-1] / sizes[-1]) <= 5.0 * np.sqrt(c) / n
        if K <= 32:  # workgroups of the longest range list more than they keep
            assert listed[-1] > 256 * 1280
    finally:
        ctx.close()
