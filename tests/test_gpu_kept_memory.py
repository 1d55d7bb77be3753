"""The memory that a thread keeps between its lone solves: other streams' work
is not waited for, and threads that come and go share nothing that a call has."""
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


def _busy(seconds):
    """A stream with about that much work of one wavefront queued."""
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        torch.cuda._sleep(10 ** 7)
        t1.record()
        s.synchronize()
        torch.cuda._sleep(int(10 ** 7 * seconds * 1e3 / t0.elapsed_time(t1)))
    return s


def test_growth_and_thread_end_wait_for_no_other_stream(q, orc):
    """A thread's first solves, a larger one and its end, beside a second of
    another stream's work."""
    Q = inputs.uniform_int(18, -100, 100, 5)
    exp = orc.solve_range(Q, 0, 1 << 18, k=64)
    q.solve(Q)
    got = []

    def work():
        r = q.solve(Q)
        got.append([(r.energy_i, r.index)])
        got.append(q.solve(Q, k=64)[1])

    side = _busy(1.0)
    th = threading.Thread(target=work)
    th.start()
    th.join()
    still = not side.query()
    side.synchronize()
    assert still, "a solve or its thread's end waited for another stream"
    assert got == [exp[:1], exp]


def test_threads_at_once(q, orc):
    """Lone solves of changing sizes and k from several threads, on memory of
    their own, and from threads that take over ended ones' blocks."""
    cases = [(15 + i % 6, i % 3 == 2, [1, 5, 40][i % 3], i) for i in range(12)]
    mats, exp = [], []
    for n, fp, k, i in cases:
        Q = inputs.normal_fp32(n, i) if fp else inputs.uniform_int(n, -50, 50, i)
        mats.append(Q)
        exp.append(q.solve(Q, k=max(k, 2))[1][:k])
        if not fp:
            assert exp[-1] == orc.solve_range(Q, 0, 1 << n, k=k)
    bad = []

    def work(t):
        for rep in range(4):
            for c in range(len(cases)):
                i = (c * 5 + t + rep) % len(cases)
                k = cases[i][2]
                got = q.solve(mats[i], k=max(k, 2))[1][:k]
                if got != exp[i]:
                    bad.append((t, i, got, exp[i]))

    for wave in range(2):
        th = [threading.Thread(target=work, args=(t,)) for t in range(6)]
        for t in th:
            t.start()
        for t in th:
            t.join()
    assert not bad, bad[:2]
