"""The ordered output of long ranges that accept most of what they propose: more
and shorter segments than sparse ranges of the same length (at least 1024
accepted a segment, 8192 to 65536 segments).  The statistics are the sums over
the same samples whatever the segments: |x^| = 1 fixes S2 per sample (Parseval),
the histogram counts every sample once, and rows and indices are those of a
short call's prefix.
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


@pytest.mark.parametrize("K", [8, 32, 64, 128])
@pytest.mark.parametrize("n", [(1 << 25) + 31, (1 << 26) + 4097])
def test_dense_ranges(T, K, n):
    import torch
    ctx = T.Context(0)
    try:
        # not c = 0, where log a reaches 0 itself and its rounding may raise M
        pt = T.make_point(K, 1.0, 40.0, 1.0, seed=5, point_id=3)
        pl = ctx.plan_batch([pt], T.SIGMA, n_starts=8)[0][0]
        m = 5000
        idx = torch.empty((n,), dtype=torch.int64, device="cuda")
        rows = torch.empty((n if K == 8 else m, 2 * K), dtype=torch.float32, device="cuda")
        a = ctx.sample(pt, m, plan=pl, capacity=m)
        b = ctx.sample(pt, n, plan=pl, capacity=rows.shape[0], xhat=rows, index=idx)
        na, nb = a["n_accepted"], b["n_accepted"]
        assert nb > n // 3 and b["n_written"] == min(nb, rows.shape[0])
        # S2 = n N E0/(2 pi) up to the FP32 rounding of the rows: 2K terms of relative error 2^-24 each
        assert abs(b["S2"] / nb - a["S2"] / na) <= 2 * K * 2.0 ** -24 * a["S2"] / na
        assert int(np.sum(b["hist_u0"])) == nb
        i = idx[: b["n_written"]]
        assert bool((i[1:] > i[:-1]).all())
        w = min(na, b["n_written"])
        assert torch.equal(i[:w], a["index"][:w])
        assert torch.equal(rows[:w], a["xhat"][:w])
    finally:
        ctx.close()
