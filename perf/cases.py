"""Timed cases of the solver's public entry points, from the smallest call to the headline solve.

A case is a dict of plain values.  Its kind names the entry point:

* ``solve``: ``solve(Q)`` on a host matrix (``where`` "host") or
  ``solve_device(Q)`` on a torch tensor ("device"), with ``k`` > 1 the k lowest
  states as well;
* ``batch``: a ``Batch`` handle that the program keeps, replayed and read;
* ``solve_batch``: the one-shot batch, planning included;
* ``serve``: a burst of requests to a running ``Server``, submitted together
  and each waited for.

Entries are i.i.d. uniform integers in [-span, span] or float32 N(0, 1)
(``dtype`` "fp32"), upper-triangular, drawn from the seed; the sizes of a
batch or a burst are spread evenly over [n_lo, n_hi] and do not depend on it.
A "mix" burst is 80% integer and 20% float32 requests.
"""
import math

import numpy as np
import torch

import paper_2607_04857_amd as q


def listed():
    return [
        # a toy problem from host memory: every state evaluated directly
        {"name": "solve_n12", "kind": "solve", "where": "host", "n": 12, "k": 1,
         "dtype": "int32", "span": 100},
        # the small dense instance of the benchmark's first configuration
        {"name": "solve_n24", "kind": "solve", "where": "host", "n": 24, "k": 1,
         "dtype": "int32", "span": 100},
        # a float32 model a program already holds on the GPU
        {"name": "device_n27_fp32", "kind": "solve", "where": "device", "n": 27, "k": 1,
         "dtype": "fp32", "span": 0},
        # a float32 instance from the host, at the upper end of the batch sizes
        {"name": "solve_n33_fp32", "kind": "solve", "where": "host", "n": 33, "k": 1,
         "dtype": "fp32", "span": 0},
        # the mid-size instance of the benchmark's second configuration
        {"name": "solve_n36", "kind": "solve", "where": "host", "n": 36, "k": 1,
         "dtype": "int32", "span": 1000},
        # the headline: one large instance in device memory
        {"name": "device_n44", "kind": "solve", "where": "device", "n": 44, "k": 1,
         "dtype": "int32", "span": 10000},
        # the low end of a spectrum, few states
        {"name": "topk16_n21", "kind": "solve", "where": "host", "n": 21, "k": 16,
         "dtype": "int32", "span": 100},
        # a long low-energy spectrum of a device matrix
        {"name": "topk1024_n31", "kind": "solve", "where": "device", "n": 31, "k": 1024,
         "dtype": "int32", "span": 10000},
        # thousands of instances of uneven size, replayed (the batch configuration)
        {"name": "batch4096", "kind": "batch", "count": 4096, "n_lo": 20, "n_hi": 34,
         "dtype": "int32", "span": 100},
        # many small float32 instances, replayed
        {"name": "batch1000_fp32", "kind": "batch", "count": 1000, "n_lo": 12, "n_hi": 26,
         "dtype": "fp32", "span": 0},
        # one-shot batch of small instances, planned and freed within the call
        {"name": "solve_batch100", "kind": "solve_batch", "count": 100, "n_lo": 15, "n_hi": 25,
         "dtype": "int32", "span": 100},
        # a burst of mixed requests to a running server
        {"name": "serve64", "kind": "serve", "count": 64, "n_lo": 16, "n_hi": 34,
         "dtype": "mix", "span": 100},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: n is the logarithm of the work, so uniform in n."""
    kind = rng.choice(["solve", "solve", "solve", "topk", "topk", "batch", "solve_batch", "serve"])
    dtype = rng.choice(["int32", "int32", "fp32"])
    span = rng.choice([20, 100, 1000, 10000]) if dtype == "int32" else 0
    where = rng.choice(["host", "device"])
    if kind == "solve":
        return {"kind": "solve", "where": where, "n": rng.randint(6, 42), "k": 1,
                "dtype": dtype, "span": span}
    if kind == "topk":
        n = rng.randint(11, 36)
        return {"kind": "solve", "where": where, "n": n, "k": _log_int(rng, 2, 1024),
                "dtype": dtype, "span": span}
    n_lo = rng.randint(10, 22)
    if kind == "batch":
        return {"kind": "batch", "count": _log_int(rng, 16, 4096), "n_lo": n_lo,
                "n_hi": n_lo + rng.randint(0, 11), "dtype": dtype, "span": span}
    if kind == "solve_batch":
        return {"kind": "solve_batch", "count": _log_int(rng, 2, 512), "n_lo": n_lo,
                "n_hi": n_lo + rng.randint(0, 8), "dtype": dtype, "span": span}
    return {"kind": "serve", "count": _log_int(rng, 8, 128), "n_lo": n_lo + 4,
            "n_hi": n_lo + 4 + rng.randint(0, 10), "dtype": "mix", "span": 100}


def _matrix(rng, n, dtype, span):
    if dtype == "fp32":
        return np.triu(rng.standard_normal(size=(n, n)).astype(np.float32))
    return np.triu(rng.integers(-span, span, size=(n, n), endpoint=True)).astype(np.int32)


def _sizes(case):
    """The sizes of a batch or burst, spread evenly over [n_lo, n_hi] in a fixed mixed order."""
    if case["kind"] == "solve":
        return [case["n"]]
    width, count = case["n_hi"] - case["n_lo"] + 1, case["count"]
    sizes = [case["n_lo"] + i % width for i in range(count)]
    return [int(n) for n in np.random.default_rng(count).permutation(sizes)]


def _matrices(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i, n in enumerate(_sizes(case)):
        dtype = case["dtype"]
        if dtype == "mix":
            dtype = "fp32" if i % 5 == 4 else "int32"
        out.append(_matrix(rng, n, dtype, case["span"]))
    return out


def prepare(case, seed):
    Qs = _matrices(case, seed)
    state = {"kind": case["kind"], "k": case.get("k", 1), "Qs": Qs}
    if case["kind"] == "solve":
        state["where"] = case["where"]
        state["Q"] = torch.from_numpy(Qs[0]).to("cuda:0") if case["where"] == "device" else Qs[0]
    elif case["kind"] == "batch":
        state["batch"] = q.Batch(Qs)
    elif case["kind"] == "serve":
        state["server"] = q.Server(mem_budget_bytes=8 << 30, max_slots=512)
    return state


def _one(r):
    return {"energy": r.energy, "energy_i": r.energy_i, "index": r.index, "tol": r.tol, "p": r.p,
            "states": r.states}


def _many(results):
    return {"energy": np.array([r.energy for r in results]),
            "energy_i": np.array([r.energy_i for r in results], dtype=np.int64),
            "index": np.array([r.index for r in results], dtype=np.int64),
            "tol": np.array([r.tol for r in results])}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        call = q.solve_device if state["where"] == "device" else q.solve
        if state["k"] == 1:
            return _one(call(state["Q"]))
        r, pairs = call(state["Q"], k=state["k"])
        return {"best": _one(r), "energies": np.array([e for e, _ in pairs]),
                "indices": np.array([i for _, i in pairs], dtype=np.int64)}
    if kind == "batch":
        state["batch"].run()
        return _many(state["batch"].results())
    if kind == "solve_batch":
        return _many(q.solve_batch(state["Qs"]))
    tickets = [state["server"].submit(Q) for Q in state["Qs"]]
    return _many([state["server"].wait(t) for t in tickets])


def work(case):
    """One add per state (the Gray-code walk's count); Q read once, the answers written once."""
    sizes = _sizes(case)
    answers = len(sizes) * 48 if case.get("k", 1) == 1 else case["k"] * 24
    return {"bytes": sum(4 * n * n for n in sizes) + answers,
            "flops": float(sum(2 ** n for n in sizes))}


def _lowest(Q, k):
    """The k smallest (energy, index) pairs of x^T Q x, by float64 energies of every state."""
    n = Q.shape[0]
    T = torch.from_numpy(Q.astype(np.float64)).to("cuda:0")
    b = min(n, 13)
    a = n - b

    def bits(first, count, width):
        x = torch.arange(first, first + count, device="cuda:0").unsqueeze(1)
        s = torch.arange(width - 1, -1, -1, device="cuda:0").unsqueeze(0)
        return ((x >> s) & 1).double()

    xs = bits(0, 1 << b, b)
    Tss = T[a:, a:].contiguous()
    Es = ((xs @ Tss) * xs).sum(1)
    Tps = (T[:a, a:] + T[a:, :a].t()).contiguous()
    xst = xs.t().contiguous()
    best_e = torch.empty(0, dtype=torch.float64, device="cuda:0")
    best_i = torch.empty(0, dtype=torch.int64, device="cuda:0")
    step = min(1 << a, 1 << 13)
    for first in range(0, 1 << a, step):
        E = Es.unsqueeze(0).expand(step, -1).clone()
        if a:
            xp = bits(first, step, a)
            E += ((xp @ T[:a, :a].contiguous()) * xp).sum(1).unsqueeze(1)
            E += (xp @ Tps) @ xst
        E = E.reshape(-1)
        if k == 1:
            bound = E.min()
        else:
            bound = torch.topk(E, min(k, E.numel()), largest=False).values.max()
        if best_e.numel() >= k:
            if bool(E.min() > best_e[-1]):
                continue
            bound = torch.minimum(bound, best_e[-1])
        at = (E <= bound).nonzero().reshape(-1)
        e = torch.cat([best_e, E[at]])
        i = torch.cat([best_i, at + (first << b)])
        by_i = torch.argsort(i)
        e, i = e[by_i], i[by_i]
        by_e = torch.argsort(e, stable=True)[:k]
        best_e, best_i = e[by_e], i[by_e]
    return best_e.cpu().numpy(), best_i.cpu().numpy()


def exact(case, seed):
    """Energies of the lowest states in float64 from the definition (None beyond 2^36 states)."""
    if sum(2 ** n for n in _sizes(case)) > 2 ** 36:
        return None
    Qs = _matrices(case, seed)
    k = case.get("k", 1)
    found = [_lowest(Q, k) for Q in Qs]
    if case["kind"] == "solve":
        e, i = found[0]
        best = {"energy": float(e[0]), "energy_i": None, "index": int(i[0]), "tol": None, "p": None,
                "states": 2 ** case["n"]}
        if k == 1:
            return best
        fp = case["dtype"] == "fp32"
        return {"best": best, "energies": e if fp else e.astype(np.int64), "indices": i}
    return {"energy": np.array([e[0] for e, _ in found]), "energy_i": None,
            "index": np.array([i[0] for _, i in found]), "tol": None}
