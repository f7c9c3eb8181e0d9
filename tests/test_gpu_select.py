"""The extremes' selection runs on the device: its list is the first k rows by
(larger maximum, lower row) for every size of the list, of ties and of the
range, and the running maxima keep the lowest grid index of a tie and a valid
one for rows that are not finite.
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


def _run(T, ctx, K, rows, k):
    r = ctx.extremes(rows, K=K, E0=1.0, top_k=k, per_row=True)
    return r, r["umax_rows"].cpu().numpy(), r["jmax_rows"].cpu().numpy()


def _check(r, um, jm, k):
    order = np.lexsort((np.arange(um.size), -um.astype(np.float64)))[:k]
    assert np.array_equal(r["rows"].astype(np.int64), order)
    assert np.array_equal(r["umax"], um[order].astype(np.float64))
    assert np.array_equal(r["jmax"], jm[order])


@pytest.mark.parametrize("K", [8, 32, 64, 128])
@pytest.mark.parametrize("n,k,distinct", [(1, 1, 1), (15, 4, 15), (17, 17, 3), (1025, 700, 1025), (300_007, 4096, 300_007),
                                          (70_001, 300, 40), (65_536, 4096, 1), (262_145, 1000, 777)])
def test_list_is_the_first_k(T, ctx, K, n, k, distinct):
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    base = torch.randn((distinct, 2 * K), generator=g, device="cuda")
    base /= base.norm(dim=1, keepdim=True)
    rows = base[torch.randint(0, distinct, (n,), generator=g, device="cuda")].contiguous()
    r, um, jm = _run(T, ctx, K, rows, k)
    _check(r, um, jm, k)


@pytest.mark.parametrize("K", [64, 128])
def test_ties_and_rows_that_are_not_finite(T, ctx, K):
    import torch
    rows = torch.zeros((40, 2 * K), device="cuda")
    rows[1, 0] = 1.0                  # cos xi: one maximum, at xi = 0
    rows[2, 1] = 1.0                  # cos 2 xi: equal maxima at xi = -pi and 0, the first is kept
    rows[3, K + 1] = 1.0              # sin 2 xi: -3 pi/4 and pi/4
    rows[4, 0] = float("inf")
    rows[5, 0] = float("-inf")
    rows[6, 3] = float("nan")
    rows[7, :] = float("-inf")
    rows[8, K:] = float("inf")
    rows[9, :] = float("nan")
    rows[10, 0] = -1.0                # -cos xi: at +-pi, the same grid point
    r, um, jm = _run(T, ctx, K, rows, 5)
    assert jm[0] == 0 and um[0] == 0.0
    assert jm[1] == 2 * K and jm[2] == 0 and jm[3] == K // 2 and jm[10] == 0
    assert ((jm >= 0) & (jm < 4 * K)).all()
    assert not np.isnan(um).any()     # a row without a comparable value has -inf
    assert um[9] == -np.inf and um[6] == -np.inf
    _check(r, um, jm, 5)
