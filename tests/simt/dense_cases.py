"""Small graphs with skewed or long rows on the CPU emulation, through the
one-workgroup solve of the hybrid schedule where its limits allow: prints one
JSON line per case with the launches it took.  Started by
tests/test_simt_dense.py."""
import json

import numpy as np

from cases import L, P, graph, llpgen, oracle, solve

L.simt_launches.restype = __import__("ctypes").c_ulonglong


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def run(name, e, s):
    for kind in ("sssp", "bfs"):
        before = L.simt_launches()
        code, _, out = solve(kind, graph(e), s, sched=P.SCHED_HYBRID)
        want = oracle.sssp(e.n, e.src, e.dst, e.w, s) if kind == "sssp" else oracle.bfs(e.n, e.src, e.dst, s)
        print(json.dumps({"case": name, "kind": kind, "status": code, "equal": bool(np.array_equal(out, want)),
                          "launches": int(L.simt_launches() - before)}), flush=True)


rng = np.random.default_rng(5)
# few vertices: as many arcs as one workgroup takes, and one more
for n, m in ((3, 50150), (3, 50151), (64, 53200), (64, 53201), (300, 65000), (300, 65001)):
    run(f"limit-{n}-{m}", edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, 20, m)), n - 1)
# rows on both sides of what all waves share: one hub, hubs of one run, hubs of many blocks
for deg in (4095, 4096, 4097, 9000):
    src = np.concatenate([np.full(deg, 8), rng.integers(0, 200, 600)])
    run(f"hub-{deg}", edges(200, src, rng.integers(0, 200, src.size), rng.integers(0, 30, src.size)), 8)
src = np.concatenate([np.repeat(np.arange(4), 1500), np.repeat(np.arange(100, 140), 257), rng.integers(0, 500, 900)])
run("hubs", edges(500, src, rng.integers(0, 500, src.size), rng.integers(0, 30, src.size)), 101)
# several blocks per wave: long and short frontiers, ids that share their low bits
for n in (1023, 1025, 2049, 5000):
    run(f"blocks-{n}", llpgen.uniform_graph(n, 3 * n, 0, 9, seed=n), n // 3)
g = llpgen.rmat_graph(11, ef=8, seed=3, relabel=False)
run("rmat", g, llpgen.max_outdeg_source(g))
i = np.repeat(np.arange(2000 - 3), 3)
run("band", edges(2000, i, i + np.tile([1, 2, 3], 1997), rng.integers(0, 9, i.size)), 0)
