"""More proposals for the FP64 pass than the workgroups' lists in LDS hold: beyond
256 a workgroup, by the grid that the call itself used.  The accepted indices are
those of a shorter call, whose workgroups keep theirs, and the moments (a function
of the accepted samples, bit for bit) those of an accepted-count call, which deals
out the range otherwise.
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


@pytest.mark.parametrize("K,beta,prec,n", [(8, 20.0, "bf16x3", (1 << 28) + 7), (16, 20.0, "fp32", (1 << 27) + 1),
                                           (32, 20.0, "bf16x3", (1 << 27) + 99), (64, 40.0, "bf16x3", 60_000_001),
                                           (128, 40.0, "bf16x3", 40_000_019), (128, 40.0, "fp32", 40_000_003)])
def test_workgroups_list_more_than_they_keep(T, K, beta, prec, n):
    import torch
    ctx = T.Context(0)
    try:
        pt = T.make_point(K, 1.0, beta, 0.5, seed=5, point_id=3)
        pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
        m = 4_000_000
        d = ctx.sample(pt, n, plan=pl, precision=T.PRECISIONS[prec], capacity=m)
        grid = ctx.timing()["decide_grid"]
        print(f"K={K} {prec}: {d['n_fp64_fixups']} listed, {grid} workgroups", flush=True)
        assert d["n_fp64_fixups"] > 256 * grid
        part = ctx.sample(pt, 1_000_000, plan=pl, precision=T.PRECISIONS[prec], capacity=m)
        k = part["n_written"]
        assert k == part["n_accepted"] and bool(torch.equal(part["index"], d["index"][:k]))
        assert int(d["index"][k]) >= 1_000_000 and bool((d["index"][1:] > d["index"][:-1]).all())
        a = ctx.sample(pt, d["n_accepted"], plan=pl, precision=T.PRECISIONS[prec], mode=T.COUNT_ACCEPTED,
                       max_proposals=n)
        assert a["n_accepted"] == d["n_accepted"]
        for key in ("S1", "S2", "S3", "S4"):
            assert a[key] == d[key], key
    finally:
        ctx.close()
