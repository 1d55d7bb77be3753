"""One-shot batches (no handle, no graph) by every way their memory can be had:
small ones in the thread's kept memory, images and jobs too large for it, and
small ones again after those; every kind of instance, against the batch handle
and the oracle."""
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


def _mixed(count, seed, n_lo=6, n_hi=19):
    """Direct (n <= 14), packed, int32-walk and float32 instances, both triangles."""
    out = []
    for i in range(count):
        n = n_lo + (7 * i + seed) % (n_hi - n_lo + 1)
        if i % 3 == 2:
            out.append(inputs.normal_fp32(n, seed + i))
        else:
            s = 40 if i % 3 == 0 else 30000
            Q = inputs.uniform_int(n, -s, s, seed + i)
            out.append(Q + np.tril(inputs.uniform_int(n, -s, s, 100000 + seed + i).T, -1))
    return out


def _key(r):
    return (r.energy_i, r.energy, r.index, r.tol, r.p, r.tier, r.states)


def _check(q, orc, Qs, sample):
    got = q.solve_batch(Qs)
    b = q.Batch(Qs)
    b.run()
    assert [_key(r) for r in got] == [_key(r) for r in b.results()]
    b.close()
    for i in sample:
        if Qs[i].dtype == np.int32:
            assert (got[i].energy_i, got[i].index) == orc.solve(Qs[i], k=1)[0], i
        else:
            alone = q.solve(Qs[i])
            assert (got[i].energy_i, got[i].energy, got[i].index) == (
                alone.energy_i, alone.energy, alone.index), i


@pytest.mark.parametrize("count", [1, 2, 3, 40, 257])
def test_mixed(q, orc, count):
    _check(q, orc, _mixed(count, count), range(min(count, 40)))


def test_direct_only(q, orc):
    Qs = [inputs.uniform_int(1 + i % 14, -9, 9, i) for i in range(30)]
    Qs += [inputs.normal_fp32(1 + i % 14, i) for i in range(30)]
    _check(q, orc, Qs, range(60))


def test_larger_than_kept_and_back(q, orc):
    """7600 instances: an image above 4 MiB (pageable copies) and a job above 128
    MiB (memory of its own); before and after it a small batch, the same matrices
    as one call of three, and a lone call with large lists, on one thread."""
    small = _mixed(12, 5)
    Q = inputs.uniform_int(20, -1000, 1000, 8)
    low = orc.solve_range(Q, 0, 1 << 20, k=300)
    large = _mixed(7600, 77, 14, 18)
    for Qs in (small, large, small, large[:700], small):
        _check(q, orc, Qs, range(0, len(Qs), max(1, len(Qs) // 8)))
        assert q.solve(Q, k=300)[1] == low


def test_thousands_of_equal_small_instances(q, orc):
    """Every item of 2^6 or a few more steps: 4096 copies, replayed and one-shot."""
    for n, s in ((16, 100), (20, 100), (18, 30000)):
        Q = inputs.uniform_int(n, -s, s, n)
        exp = orc.solve(Q, k=1)[0]
        b = q.Batch([Q] * 4096)
        for _ in range(2):
            b.run()
            assert {(r.energy_i, r.index) for r in b.results()} == {exp}
        b.close()
        assert {(r.energy_i, r.index) for r in q.solve_batch([Q] * 4096)} == {exp}


@pytest.mark.parametrize("n,k", [(12, 4), (20, 12), (27, 12)])
def test_outer(q, orc, n, k):
    """The reduced instances of an outer solve: direct ones, and 4096 walked."""
    Q = inputs.uniform_int(n, -300, 300, n + k)
    got = q.solve_outer(Q, k)
    assert (got.energy_i, got.index) == orc.solve(Q, k=1)[0]
