"""The walk's interaction rows are formed from a lane part and a column part
per row.  The widest table (n = 60) on single short work items, every lane
width, against the oracle's exhaustive minimum of the item's states."""
import numpy as np
import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


# (B, vgpr_levels, tier, largest |entry|): one word per lane to sixteen, the
# row caches that read level 5 from the parts, and the packed words
CASES = [(6, 12, 1, 1000), (6, 12, 2, 1000), (7, 12, 2, 1000), (8, 12, 2, 1000), (9, 8, 2, 1000),
         (10, 12, 2, 1000), (10, 8, 1, 1000), (10, 6, 2, 1000), (10, 5, 2, 1000), (10, 4, 2, 1000),
         (10, 3, 2, 1000), (9, 12, 4, 3), (10, 8, 4, 3), (11, 4, 4, 3), (11, 3, 4, 3), (11, 5, 4, 3)]


@pytest.mark.parametrize("B,vgpr,tier,span", CASES)
def test_widest_tables_on_single_items(q, orc, B, vgpr, tier, span):
    n = 60
    Q = inputs.uniform_int(n, -span, span, 60 * B + vgpr)
    Q = Q + np.tril(inputs.uniform_int(n, -span, span, 61 * B + vgpr).T, -1)   # both triangles
    states = 1 << (8 + B)
    rng = np.random.default_rng(B)
    # items of 2^8 steps: the first ones and one far out (item numbers are ints)
    for c in (0, 5, int(rng.integers(1 << 20, 1 << 31))):
        got = q.solve(Q, B=B, tier=tier, vgpr_levels=vgpr, L=8, item_first=c, item_count=1)
        assert (got.B, got.tier, got.vgpr_levels) == (B, tier, vgpr)
        exp = orc.solve_range(Q, (c ^ (c >> 1)) * states, states, k=1)[0]
        assert (got.energy_i, got.index) == exp, c


@pytest.mark.parametrize("span", [3, 1000])
def test_widest_tables_topk(q, orc, span):
    """The top-k rescan of selected chunks from the same parts (packed, int32)."""
    n, k = 60, 40
    Q = inputs.uniform_int(n, -span, span, 6060 + span)
    tier, B = (4, 11) if span == 3 else (2, 10)
    c, states = 123456789, 1 << (8 + B)
    res, pairs = q.solve(Q, k=k, B=B, tier=tier, L=8, item_first=c, item_count=1)
    assert pairs == [(int(e), int(i)) for e, i in
                     orc.solve_range(Q, (c ^ (c >> 1)) * states, states, k=k)]
