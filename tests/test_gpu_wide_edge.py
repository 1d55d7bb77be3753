"""Wide words at the edge of their fields: chunk energies that span exactly
2^21 - 1 (the most that three to a word hold), 2^21 and more, with every field
of a word at its largest value where the least is sought; against the oracle's
exhaustive minimum, for host and device Q."""
import numpy as np
import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu

EDGE = 1 << 21


@pytest.fixture(scope="module")
def q():
    import torch  # noqa: F401  (torch's HIP runtime starts first)
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


def _extremes(Q, A):
    """Least and largest chunk energy over all columns and prefixes."""
    Q = Q.astype(np.int64)
    B = Q.shape[0] - A
    s = (np.arange(1 << B)[:, None] >> np.arange(B - 1, -1, -1)) & 1
    E = ((s @ Q[A:, A:]) * s).sum(1)
    M = s @ Q[:A, A:].T
    return int((E + np.minimum(M, 0).sum(1)).min()), int((E + np.maximum(M, 0).sum(1)).max())


def _spanning(n, span, small, seed):
    """Entries of at most `small`, but for variable 3's coupling with suffix
    variable n - 7 (bit 0 of a lane's column number: every other field).  The
    least chunk energy is then below all others by about `span`, and where
    variable 3 is 0 all of a chunk's energies are near the largest."""
    rng = np.random.default_rng(seed)
    Q = np.triu(rng.integers(-small, small, size=(n, n), endpoint=True)).astype(np.int32)
    Q[3, n - 7] = -span // 2
    for _ in range(4):
        lo, hi = _extremes(Q, n - 10)
        Q[3, n - 7] -= span - (hi - lo)
    lo, hi = _extremes(Q, n - 10)
    assert hi - lo == span
    return Q


@pytest.mark.parametrize("small", [0, 5])
@pytest.mark.parametrize("span", [EDGE - 1, EDGE, EDGE + 1, 70000])
def test_items(q, orc, span, small):
    """Single items: variable 3 off (c < 1024 and the last: every energy near the
    top of its field) and on."""
    n, L = 32, 8
    Q = _spanning(n, span, small, span % 97 + small)
    if small == 0:
        Q[:22, :22] = np.triu(inputs.uniform_int(22, -40, 40, 3))   # the prefix's own energies
    info = q.plan_info(Q)
    assert (info["tier"], info["B"], info["vgpr_levels"]) == (2, 10, 4)
    assert info["pack_shift"] == -_extremes(Q, n - 10)[0]
    states = 1 << (L + 10)
    for c in (0, 1, 777, 1023, 1024, 1500, 2047, (1 << 14) - 1):
        got = q.solve(Q, L=L, item_first=c, item_count=1)
        assert (got.energy_i, got.index) == orc.solve_range(Q, (c ^ (c >> 1)) * states, states, k=1)[0], c


@pytest.mark.parametrize("small", [0, 4])
@pytest.mark.parametrize("span", [EDGE - 1, EDGE])
def test_whole_solves(q, orc, span, small):
    """Whole solves and the lowest states, host and device Q: variable 3 made
    costly, so that the answers are chunks whose fields are all near the top."""
    import torch
    n = 30
    Q = _spanning(n, span, small, 11)
    if small == 0:
        Q[:20, :20] = np.triu(inputs.uniform_int(20, -40, 40, 4))
    Q[3, 3] = 4 * EDGE
    assert _extremes(Q, n - 10)[1] - _extremes(Q, n - 10)[0] == span
    assert q.plan_info(Q)["tier"] == 2
    exp = orc.solve_range(Q, 0, 1 << n, k=40)
    Qd = torch.from_numpy(Q).cuda()
    for got in (q.solve(Q), q.solve_device(Qd)):
        assert (got.energy_i, got.index) == exp[0]
    assert q.solve(Q, k=40)[1] == exp
    assert q.solve_device(Qd, k=40)[1] == exp
