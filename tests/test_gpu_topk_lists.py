"""The top-k walk's lists: keys entered a super-block at a time, with room in
the list, at the key that fills it and past it, on every row cache and with
ties throughout; against the oracle's k smallest (energy, index) pairs."""
import numpy as np
import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch  # noqa: F401  (torch's HIP runtime starts first)
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


@pytest.mark.parametrize("lo", [-1, -100, -3000000])
@pytest.mark.parametrize("k", [2, 16, 63, 64, 65, 200, 1024])
def test_dense(q, orc, k, lo):
    """n = 19 (512 prefix rows of the default split): packed, int32, and lists
    that fill (64 keys a wave) or never do."""
    Q = inputs.uniform_int(19, lo, -lo, k - lo)
    exp = orc.solve_range(Q, 0, 1 << 19, k=k)
    assert q.solve(Q, k=k)[1] == exp
    assert q.solve(Q, k=k, L=9)[1] == exp          # one wave, one item


@pytest.mark.parametrize("G", [3, 4, 5, 6, 8, 12])
@pytest.mark.parametrize("tier", [2, 4])
def test_row_caches(q, orc, G, tier):
    Q = inputs.uniform_int(20, -3, 3, G)
    if tier == 4:
        got = q.solve(Q, k=130, tier=4, B=11, vgpr_levels=G, L=8)[1]
    else:
        got = q.solve(Q, k=130, tier=2, B=10, vgpr_levels=G, L=9)[1]
    assert got == orc.solve_range(Q, 0, 1 << 20, k=130)


@pytest.mark.parametrize("n,tier", [(22, 4), (24, 2), (30, 2)])
@pytest.mark.parametrize("k", [2, 70, 1000])
def test_all_equal(q, n, tier, k):
    """Every state has energy 0 (n = 30: on wide words): the lowest k indices."""
    r, pairs = q.solve(np.zeros((n, n), dtype=np.int32), k=k, tier=tier)
    assert pairs == [(0, i) for i in range(k)]


@pytest.mark.parametrize("n,k", [(30, 1024), (31, 9), (32, 100)])
def test_wide_equals_int32(q, n, k):
    import torch
    Q = inputs.uniform_int(n, -10000, 10000, k)
    exp = q.solve(Q, k=k, vgpr_levels=3)[1]        # never on wide words
    assert q.solve(Q, k=k)[1] == exp
    assert q.solve_device(torch.from_numpy(Q).cuda(), k=k)[1] == exp
