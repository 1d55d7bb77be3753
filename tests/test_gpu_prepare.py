"""The device preparation's fixed-point exponent at and around powers of two
of sum |T|, where a sum in another order could land on the other side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch  # noqa: F401  (torch's HIP runtime starts first)
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


def _matrices():
    rng = np.random.default_rng(2)
    ones = np.eye(16, dtype=np.float32)
    yield "exact power", ones                                   # S = 16
    up, down = ones.copy(), ones.copy()
    up[0, 0] = np.nextafter(np.float32(1), np.float32(2))
    down[0, 0] = np.nextafter(np.float32(1), np.float32(0))
    yield "one ulp above", up
    yield "one ulp below", down
    # many terms whose float64 sum rounds: 2^k + tiny ones
    n = 24
    Q = np.zeros((n, n), dtype=np.float32)
    Q[np.triu_indices(n)] = np.float32(2.0 ** -60)
    Q[0, 0] = 1.0
    yield "power plus dust", Q
    Q = Q.copy()
    Q[np.triu_indices(n)] = np.where(rng.random(n * (n + 1) // 2) < 0.5, 1, -1) * np.float32(0.1)
    yield "tenths", Q
    yield "zero", np.zeros((15, 15), dtype=np.float32)
    yield "random", np.triu(rng.standard_normal((27, 27)).astype(np.float32))
    yield "huge", np.triu(rng.standard_normal((20, 20)).astype(np.float32) * np.float32(1e37))


@pytest.mark.parametrize("name,Q", list(_matrices()), ids=[m[0] for m in _matrices()])
def test_scale_exponent_matches_the_host_planner(q, orc, name, Q):
    import torch
    info = q.plan_info(Q)
    got = q.solve_device(torch.from_numpy(Q).cuda())
    host = q.solve(Q)
    assert got.p == info["p"] == host.p
    assert (got.energy_i, got.energy, got.index, got.tol) == (host.energy_i, host.energy, host.index,
                                                              host.tol)
