"""Runs batches and transitive closures on the CPU emulation
(libllp_simt_wg.so) and prints one JSON line per case.  Started by
tests/test_simt_wg.py in a child process, as a waiting workgroup whose waves
stand at different barriers aborts.  Usage: wg_cases.py batch|closure."""
import ctypes
import json
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))
import llpgen  # noqa: E402
import oracle  # noqa: E402
import paper_2603_13147_amd as P  # noqa: E402

L = ctypes.CDLL(os.path.join(HERE, "_build", "libllp_simt_wg.so"))
L.simt_alloc.restype = ctypes.c_void_p
L.simt_alloc.argtypes = [ctypes.c_size_t]
vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
L.llp_solve_batch.argtypes = [i32, vp, vp, i64, vp, i64, vp, ctypes.POINTER(P.Opts)]
L.llp_solve_tc.argtypes = [i32, i64, vp, vp, vp, ctypes.POINTER(P.Opts)]


def dev(a):
    a = np.ascontiguousarray(a)
    p = L.simt_alloc(max(a.nbytes, 4))
    ctypes.memmove(p, a.ctypes.data, a.nbytes)
    return p


def host(p, n, dtype=np.int32):
    return np.frombuffer((ctypes.c_char * (n * np.dtype(dtype).itemsize)).from_address(p), dtype).copy()


def opts(**kw):
    o = P.Opts()
    o.size = ctypes.sizeof(P.Opts)
    for k, v in kw.items():
        setattr(o, k, v)
    return o


def spoiled(e, late, what, value):
    """Out-CSR of e with one arc's head or weight, or one row's end, replaced in row `late`."""
    c = llpgen.CSRGraph(e, weighted=True, out_weights=True)
    ptr, dst, w = c.out_ptr.copy(), c.out_dst.copy(), c.out_w.copy()
    at = ptr[late] if what != "end" else late + 1
    {"head": dst, "weight": w, "end": ptr}[what][at] = value
    return ptr, dst, w


def batch(instances, block):
    """Solves [(ptr, dst, w, source)] in one workgroup after the other; per-instance status and distances."""
    desc = np.zeros(len(instances), P.INSTANCE_DTYPE)
    words, pos, out = [], 0, 0
    for i, (ptr, dst, w, s) in enumerate(instances):
        n, m = len(ptr) - 1, len(dst)
        desc[i] = (P.KIND_SSSP, n, s, 0, m, pos, out)
        words += [ptr, dst, w]
        pos += n + 1 + 2 * m
        out += n
    outp, stp = dev(np.full(out, -7, np.int32)), dev(np.full(len(desc), -7, np.int32))
    code = L.llp_solve_batch(len(desc), dev(desc), dev(np.concatenate(words).astype(np.int32)), pos, outp, out, stp,
                             ctypes.byref(opts(block=block, chunk=len(desc))))
    dist = host(outp, out)
    return code, host(stp, len(desc)), [dist[d["out_off"]:d["out_off"] + d["n"]] for d in desc]


def batches():
    """A malformed instance that the search reaches some rounds in, on a graph
    of several active blocks, then well-formed ones in the same workgroup."""
    for block in (256, 512):
        for what, value in (("head", 5000), ("weight", -1), ("end", 1 << 30)):
            for seed in range(2):
                e = llpgen.uniform_graph(900, 3600, 1, 9, seed=seed)
                far = oracle.bfs(e.n, e.src, e.dst, 0)
                items, want = [], []
                # taken in order of their arcs, most first
                for k, late in enumerate(np.argsort(far)[[300, 600, 890]]):
                    items.append((*spoiled(e, int(late), what, value), 0))
                    want.append(None)
                    g = llpgen.uniform_graph(700 - 60 * k, 3000 - 400 * k, 1, 50, seed=10 * seed + k)
                    c = llpgen.CSRGraph(g, weighted=True, out_weights=True)
                    items.append((c.out_ptr, c.out_dst, c.out_w, 5))
                    want.append(oracle.sssp(g.n, g.src, g.dst, g.w, 5))
                    # one arc a vertex or none: a shuffled chain, and a loop with tails
                    p = np.random.default_rng(seed + k).permutation(300).astype(np.int32)
                    for src, dst in ((p[:-1], p[1:]), (p, p[np.arange(300) * 7 % 290])):
                        h = llpgen.EdgeList(300, src, dst, (dst % 5).astype(np.int32))
                        c = llpgen.CSRGraph(h, weighted=True, out_weights=True)
                        items.append((c.out_ptr, c.out_dst, c.out_w, int(p[0])))
                        want.append(oracle.sssp(300, h.src, h.dst, h.w, int(p[0])))
                code, st, dist = batch(items, block)
                print(json.dumps({
                    "case": f"{what}-{block}-{seed}", "code": code,
                    "bad": [int(s) for s, w in zip(st, want) if w is None],
                    "good": [int(s) for s, w in zip(st, want) if w is not None],
                    "equal": all(np.array_equal(d, w) for d, w in zip(dist, want) if w is not None)}), flush=True)


def closures():
    """Well-formed graphs against the oracle, then the same with one id or
    offset out of range in a row that only later rounds reach."""
    for n, deg, seed in ((700, 2, 0), (1100, 3, 1), (1500, 2, 2)):
        g = llpgen.uniform_graph(n, deg * n, seed=seed)
        far = oracle.bfs(n, g.src, g.dst, 0)
        order = np.argsort(far)
        for what, value in ((None, 0), ("head", n), ("head", -1), ("end", 1 << 30)):
            for late in order[[n // 2, n - 1]] if what else order[:1]:
                ptr, dst, _ = spoiled(g, int(late), what, value) if what else spoiled(g, 0, "weight", 1)
                words = (n + 31) // 32
                bits = dev(np.zeros(n * words, np.uint32))
                code = L.llp_solve_tc(n, len(dst), dev(ptr), dev(dst), bits, ctypes.byref(opts()))
                row = {"case": f"{n}-{what}", "code": code}
                if not what:
                    want = oracle.transitive_closure(n, g.src, g.dst)
                    row["equal"] = bool(np.array_equal(host(bits, n * words, np.uint32).reshape(n, words), want))
                print(json.dumps(row), flush=True)


if __name__ == "__main__":
    {"batch": batches, "closure": closures}[sys.argv[1]]()
