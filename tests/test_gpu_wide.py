"""The lone walk on wide words (three chunk energies in a 64-bit word): its
eligibility edge and its levels, on single items against the oracle's
exhaustive minimum of their states, and the device's decision against the
host's."""
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


def _gray(i):
    return i ^ (i >> 1)


def _spanning(n, span, seed):
    """Chunk energies of the default split spanning exactly [0, span]: one
    prefix variable and the last column carry the extremes, small entries the
    rest."""
    Q = np.triu(np.random.default_rng(seed).integers(-3, 4, (n, n))).astype(np.int32)
    A = n - 10
    Q[A:, A:] = 0                          # E_s = the diagonal below
    Q[:A, A:] = 0
    Q[A, A] = span // 2                    # E_s in {0, span // 2}
    Q[3, A] = span - span // 2             # and this prefix variable adds the rest
    Q[0, A + 1] = -1
    Q[A + 1, A + 1] = 1                    # keeps the least at 0
    return Q


@pytest.mark.parametrize("span", [2 ** 21 - 1, 2 ** 21, 2 ** 21 + 1, 2 ** 20, 70000])
def test_span_edge(q, orc, span):
    n, L = 32, 8
    Q = _spanning(n, span, span % 97)
    assert q.plan_info(Q)["pack_shift"] == 0 and q.plan_info(Q)["tier"] == 2
    states = 1 << (L + 10)
    for c in (0, 1, 777, (1 << (22 - L)) - 1):
        got = q.solve(Q, L=L, item_first=c, item_count=1)
        assert (got.energy_i, got.index) == orc.solve_range(Q, _gray(c) * states, states, k=1)[0]


@pytest.mark.parametrize("n,lo,L,c", [(32, -10000, 12, 5), (33, -10000, 9, 1234), (40, -30000, 13, 99),
                                      (44, -10000, 14, 1 << 19), (52, -5000, 12, 1 << 29),
                                      (60, -4000, 11, (1 << 31) - 2)])
def test_items_equal_oracle(q, orc, n, lo, L, c):
    """Items of up to 2^14 steps: every level held in LDS flips, and those
    formed from their parts, in both directions."""
    Q = inputs.uniform_int(n, lo, -lo, 10 * n + L)
    info = q.plan_info(Q, L=L)
    assert (info["tier"], info["B"], info["vgpr_levels"]) == (2, 10, 4)
    got = q.solve(Q, L=L, item_first=c, item_count=2)
    states = 1 << (L + 10)
    exp = min(orc.solve_range(Q, _gray(i) * states, states, k=1)[0] for i in (c, c + 1))
    assert (got.energy_i, got.index) == exp


def test_ties_take_the_lowest_index(q, orc):
    """Equal energies all over: a constant on two couplings, too wide a span to
    pack, zero elsewhere."""
    Q = np.zeros((33, 33), dtype=np.int32)
    Q[1, 32] = 200000
    Q[2, 31] = -200000
    got = q.solve(Q)
    assert q.plan_info(Q)["tier"] == 2
    # the lowest index with x_2 = x_31 = 1
    assert (got.energy_i, got.index) == (-200000, (1 << 30) | 2)


@pytest.mark.parametrize("n,lo", [(29, -10000), (30, -10000), (32, -10000), (34, -50000), (35, -400000), (33, -20)])
def test_device_equals_host(q, n, lo):
    import torch
    Q = inputs.uniform_int(n, lo, -lo, n)
    dev = q.solve_device(torch.from_numpy(Q).cuda())
    host = q.solve(Q)
    other = q.solve(Q, tier=2, vgpr_levels=3)          # never on wide words
    assert (dev.energy_i, dev.index) == (host.energy_i, host.index) == (other.energy_i, other.index)
