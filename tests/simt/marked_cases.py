"""Runs graphs wide enough for marked pull rounds on the CPU emulation: the
plain schedule (marked rounds) against a script of pull rounds (candidates
listed), and prints one JSON line per case.  Started by
tests/test_simt_marked.py."""
import ctypes
import json

import numpy as np

from cases import P, graph, llpgen, oracle, solve


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def run(name, e, s, kinds=("sssp", "bfs"), spoil=None, ref=True):
    for kind in kinds:
        got = []
        for sched in (P.SCHED_PLAIN, P.SCHED_SCRIPT):
            g = graph(e)
            if spoil:
                spoil(g)
            got.append(solve(kind, g, s, sched=sched))
        (c0, _, o0), (c1, _, o1) = got
        row = {"case": name, "kind": kind, "status": [c0, c1], "equal": bool(np.array_equal(o0, o1))}
        if ref and not spoil:
            want = oracle.sssp(e.n, e.src, e.dst, e.w, s) if kind == "sssp" else oracle.bfs(e.n, e.src, e.dst, s)
            row["oracle"] = bool(np.array_equal(o0, want))
        print(json.dumps(row), flush=True)


def word(addr, i, v):
    ctypes.cast(addr, ctypes.POINTER(ctypes.c_int32))[i] = v


rng = np.random.default_rng(8)
M = (1 << 18) + 1000


def dense(n, lo, hi, long_row=0):
    """M arcs over n - 60 vertices (the rest have none), one row of long_row more."""
    k = n - 60
    src, dst = rng.integers(0, k, M), rng.integers(0, k, M)
    src = np.concatenate([src, rng.integers(0, k, long_row)])
    return edges(n, src, np.concatenate([dst, np.full(long_row, 7)]), rng.integers(lo, hi, src.size))


run("zero-weights", dense(700, 0, 9), 3, kinds=("sssp",))
run("long-row", dense(2500, 1, 5000, 1400), 0, kinds=("bfs",))
run("overflow", dense(500, 2 ** 30, 2 ** 30 + 5), 1, kinds=("sssp",), ref=False)
u = dense(600, 1, 50)
run("bad-out-id", u, 0, kinds=("sssp",), spoil=lambda g: word(g.out_dst, 70000, 600))
run("bad-in-id", u, 0, kinds=("bfs",), spoil=lambda g: word(g.in_src, 70000, -1))
