"""Graph captures of the caller's own beside the library's calls."""
import threading

import pytest

from paper_2607_04857_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import torch  # noqa: F401  (torch's HIP runtime starts first)
    import paper_2607_04857_amd as qq
    qq.lib()
    return qq


def test_thread_ends_during_a_capture(q, orc):
    """A thread that has solved ends while this one captures in torch's default
    (global) mode: the capture goes on."""
    import torch
    Q = inputs.uniform_int(18, -100, 100, 1)
    solved, end, got = threading.Event(), threading.Event(), []

    def work():
        got.append(q.solve(Q))
        solved.set()
        end.wait(60)

    th = threading.Thread(target=work)
    th.start()
    assert solved.wait(60)
    x = torch.arange(1024, device="cuda:0", dtype=torch.int32)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = x + 1
        end.set()
        th.join()
        z = y * 2
    for _ in range(3):
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, (x + 1) * 2)
    assert (got[0].energy_i, got[0].index) == orc.solve(Q, k=1)[0]
