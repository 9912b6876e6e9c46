"""The cases of test_gpu_failures.py, each in a process of its own whose HIP
calls go through the shim: python gpu_failing.py SHIM CASE."""
import ctypes as ct
import os
import sys

SHIM = ct.CDLL(sys.argv[1], mode=ct.RTLD_GLOBAL) if __name__ == "__main__" else None
if SHIM:
    SHIM.shim_launches.restype = ct.c_long
sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import numpy as np  # noqa: E402

from paper_1904_08553_amd import dc  # noqa: E402
from paper_1904_08553_amd import workloads as W  # noqa: E402

OPTIONS = {
    "delta": {},
    "cascade": dict(cascade=(1, 20)),
    "conservative": dict(del_rule=dc.DEL_CONSERVATIVE),
    "all": dict(mode=dc.MODE_ALL),
    "static": dict(mode=dc.MODE_STATIC),
    "learned": dict(mode=dc.MODE_LEARNED, collect=1),
    "slm": dict(algorithm=dc.ALGO_SLM),
}


def _context(case, n, edges):
    g = dc.DynamicCommunities(n, *edges, **OPTIONS[case])
    if case == "learned":
        from oracle import mlp as M
        g.set_screener(M.init_weights(3), 0.0)
    return g


def _seen(g, timed=True):
    """Everything the context tells of its state (timed: its clocks too)."""
    st = {k: v for k, v in g.last_stats().as_dict().items() if timed or not k.startswith("ms_")}
    return (*g.csr(), g.communities(), g.last_R(), g.last_trace(), g.modularity(), st)


def _same(a, b):
    return all(np.array_equal(x, y) if isinstance(x, np.ndarray) else x == y for x, y in zip(a, b))


def out_of_memory(case):
    """A batch whose first `allowed` allocations succeed, for every number that
    is too few: the context is as it was, and the same batch and the next one
    give what they give an undisturbed context."""
    n = 1500
    edges, batches = W.DCSBM(n=n, m=6 * n, blocks=15, dmax=300, seed=5).stream(2, frac=0.05)
    batches = [(b.add_u, b.add_v, b.add_w, b.del_u, b.del_v) for b in batches]
    ref = _context(case, n, edges)
    want = []
    for b in batches:
        ref.apply_batch(*b)
        want.append(_seen(ref, timed=False))
    ref.close()
    for allowed in range(10_000):
        dc.load().dc_trim_device_cache()
        g = _context(case, n, edges)
        before = _seen(g)
        SHIM.shim_allow(ct.c_long(allowed))
        try:
            g.apply_batch(*batches[0])
            failed = False
        except dc.DCError as e:
            assert e.status == -8, f"allowed={allowed}: {e}"
            failed = True
        SHIM.shim_allow(ct.c_long(-1))
        if failed:
            assert _same(_seen(g), before), f"allowed={allowed}: the context changed"
            g.apply_batch(*batches[0])
        for t, b in enumerate(batches):
            if t:
                g.apply_batch(*b)
            assert _same(_seen(g, timed=False), want[t]), f"allowed={allowed}: step {t} differs"
        g.close()
        if not failed:
            break
    print(f"{case}: every allocation of {allowed} failed once", flush=True)
    assert allowed > 20


def server(_):
    """A batch whose memory runs out, one whose kernels never run and one whose
    last sweep never runs: each fails alone, and the server goes on."""
    n = 1500
    edges, batches = W.DCSBM(n=n, m=6 * n, blocks=15, dmax=300, seed=5).stream(2, frac=0.05)
    batches = [(b.add_u, b.add_v, b.add_w, b.del_u, b.del_v) for b in batches]
    ref = dc.DynamicCommunities(n, *edges)
    want = [ref.apply_batch(*b).copy() for b in batches]
    ref.close()
    srv = dc.Server(max_inflight=4)
    oom, front, finish, twin = [srv.add_graph(n, *edges) for _ in range(4)]

    def run(gid, t):
        ticket = srv.submit(gid, *batches[t])
        try:
            return srv.poll(ticket, gid)[0]
        except dc.DCError as e:
            return e.status

    dc.load().dc_trim_device_cache()
    SHIM.shim_allow(ct.c_long(2))
    assert run(oom, 0) == -8
    SHIM.shim_allow(ct.c_long(-1))
    assert np.array_equal(run(oom, 0), want[0])
    print("out of memory: reported, then as if nothing had been", flush=True)

    SHIM.shim_drop_from(ct.c_long(SHIM.shim_launches()))
    assert run(front, 0) == -9
    SHIM.shim_drop_from(ct.c_long(-1))
    assert run(front, 0) == -10
    print("no kernel ran: the graph is out of use", flush=True)

    first = SHIM.shim_launches()
    assert np.array_equal(run(twin, 0), want[0])
    steps = SHIM.shim_launches() - first
    # the last six launches: a sweep's four and the final labels' two
    SHIM.shim_drop_from(ct.c_long(SHIM.shim_launches() + steps - 6))
    assert run(finish, 0) == -9
    SHIM.shim_drop_from(ct.c_long(-1))
    assert run(finish, 0) == -10
    print("the last sweep did not run: the graph is out of use", flush=True)

    for gid in (oom, twin):
        assert np.array_equal(run(gid, 1), want[1])
    srv.close()


if __name__ == "__main__":
    kind, _, arg = sys.argv[2].partition(":")
    {"oom": out_of_memory, "server": server}[kind](arg)
