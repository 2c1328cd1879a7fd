"""Runs small graphs under the hybrid schedule on the CPU emulation, through
the one-workgroup solve and (with statistics asked for) through the grid-wide
sweep, and prints one JSON line per case.  Started by tests/test_simt_small.py."""
import ctypes
import json

import numpy as np

from cases import P, graph, llpgen, oracle, solve


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def run(name, e, s, spoil=None, want=None):
    for kind in ("sssp", "bfs"):
        got = []
        for stats in (False, True):
            g = graph(e)
            if spoil:
                spoil(g)
            kw = dict(sched=P.SCHED_HYBRID)
            if stats:
                st = P.Stats()
                kw["stats"] = ctypes.pointer(st)
            code, _, out = solve(kind, g, s, **kw)
            got.append((code, out))
        (c0, o0), (c1, o1) = got
        row = {"case": name, "kind": kind, "status": [c0, c1], "equal": bool(np.array_equal(o0, o1))}
        if want is None and not spoil:
            ref = oracle.sssp(e.n, e.src, e.dst, e.w, s) if kind == "sssp" else oracle.bfs(e.n, e.src, e.dst, s)
            row["oracle"] = bool(np.array_equal(o0, ref))
        print(json.dumps(row), flush=True)


def word(addr, i, v):
    ctypes.cast(addr, ctypes.POINTER(ctypes.c_int32))[i] = v


rng = np.random.default_rng(3)
for n in (3, 63, 64, 65, 130, 1025):
    run(f"uniform-{n}", llpgen.uniform_graph(n, 8 * n, 0, 20, seed=n), n // 2)
for deg in (255, 256, 257, 600):   # hubs, self-loops, duplicates, isolated vertices
    src = np.concatenate([np.full(deg, 0), np.full(deg, 50), rng.integers(0, 90, 300)])
    run(f"hub-{deg}", edges(100, src, rng.integers(0, 90, src.size), rng.integers(0, 30, src.size)), 0)
run("mesh", llpgen.grid_graph(24, 24, 1, 1000, seed=5), 7)
# weights below zero without a negative cycle are taken as they are
dag = edges(60, np.repeat(np.arange(57), 4), np.repeat(np.arange(57), 4) + np.tile([1, 2, 3, 2], 57),
            rng.integers(-3, 50, 228) + 0)
run("below-zero", dag, 0, want=False)
# a distance beyond int32 on the way; ids and offsets out of range
big = edges(40, np.repeat(np.arange(39), 4), np.repeat(np.arange(1, 40), 4), np.full(156, 2**30))
run("overflow", big, 0, want=False)
u = llpgen.uniform_graph(70, 560, 1, 9, seed=1)
run("bad-id", u, 0, spoil=lambda g: word(g.out_dst, 5, 70))
run("bad-id-low", u, 0, spoil=lambda g: word(g.out_dst, 5, -1))
