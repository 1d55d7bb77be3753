"""Requests of large instances beside small ones: items of every length, and
the small requests' results while a large one runs."""
import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch  # noqa: F401  (torch's HIP runtime starts first)
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


# (n, largest |entry|): A = 30 (items of 2^12 steps), A = 32 (2^20 items of 2^12)
# and A = 33, packed and not (of 2^13)
@pytest.mark.parametrize("n,span", [(40, 10000), (42, 10000), (43, 10000), (44, 20)])
def test_large_beside_small(q, n, span):
    big = inputs.uniform_int(n, -span, span, n)
    small = [inputs.uniform_int(15 + i % 8, -100, 100, i) for i in range(12)]
    small += [inputs.normal_fp32(17 + i, i) for i in range(3)]
    s = q.Server(mem_budget_bytes=1 << 30, max_slots=32)
    try:
        t_big = s.submit(big)
        tickets = [s.submit(Q) for Q in small]
        for Q, t in zip(small + [big], tickets + [t_big]):
            got, exp = s.wait(t), q.solve(Q)
            assert (got.energy_i, got.energy, got.index) == (exp.energy_i, exp.energy, exp.index)
    finally:
        s.close()


@pytest.mark.parametrize("n,span,budget", [(38, 10000, 3 << 19), (36, 100, 1 << 20), (26, 100, 6 << 15)])
def test_small_budget(q, n, span, budget):
    """A request whose records fit the budget only on longer items is taken, and
    one that fits on none is refused."""
    Q = inputs.uniform_int(n, -span, span, n)
    s = q.Server(mem_budget_bytes=budget, max_slots=4)
    try:
        got, exp = s.wait(s.submit(Q)), q.solve(Q)
        assert (got.energy_i, got.index) == (exp.energy_i, exp.index)
        assert s.info()["mem_peak"] <= budget
        with pytest.raises(q.QuboError, match="QUBO_ENOMEM"):
            s.submit(inputs.uniform_int(44, -10000, 10000, 1))
    finally:
        s.close()
