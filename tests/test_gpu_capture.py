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


def test_refused_on_a_capturing_stream(q, orc):
    """A device solve on a stream that captures is refused with nothing
    recorded: the capture goes on, and so do later solves."""
    import torch
    Q = inputs.uniform_int(18, -100, 100, 2)
    Qd = torch.from_numpy(Q).cuda()
    exp = orc.solve(Q, k=1)[0]
    first = q.solve_device(Qd)
    x = torch.arange(1024, device="cuda:0", dtype=torch.int32)
    torch.cuda.synchronize()
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        y = x + 1
        with pytest.raises(q.QuboError, match="QUBO_EDEVICE"):
            q.solve_device(Qd, stream=s)
        with pytest.raises(q.QuboError, match="QUBO_EDEVICE"):
            q.solve_device(Qd, k=1024, stream=s)
        z = y * 2
    for _ in range(3):
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, (x + 1) * 2)
        for got in (first, q.solve_device(Qd), q.solve_device(Qd, stream=s)):
            assert (got.energy_i, got.index) == exp
