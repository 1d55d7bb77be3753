"""The server's kept request memory: bursts of changing sizes under a budget
that holds only some of them, so that blocks are reused, given back and
allocated again; every result equal to the lone solve's."""
import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("budget", [2 << 20, 64 << 20])
def test_bursts_of_changing_sizes(budget):
    import paper_2607_04857_amd as q
    s = q.Server(mem_budget_bytes=budget, max_slots=16)
    for burst, sizes in enumerate([(16, 18, 20, 16), (22, 16, 24, 20, 18), (16, 18, 20, 16), (12, 23, 23, 17)]):
        Qs = [inputs.uniform_int(n, -50, 50, 100 * burst + i) for i, n in enumerate(sizes)]
        Qs.append(inputs.normal_fp32(19, burst))
        tickets = [s.submit(Q) for Q in Qs]
        for Q, t in zip(Qs, tickets):
            got, exp = s.wait(t), q.solve(Q)
            assert (got.energy_i, got.index) == (exp.energy_i, exp.index)
    assert s.info()["mem_in_use"] == 0 and s.info()["mem_peak"] <= budget
    s.close()
