"""Marked pull rounds (plain schedule: an expansion of at least 2^16 arcs and
n / 8 stamps its targets with plain stores and the rows stamped are evaluated
in arc order): the limits of the rule, rows longer than a wave evaluates and
than a block holds, rows without arcs, weights of zero, and the counters of a
traced solve, against the oracle."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def solve(g, s, bfs=False, **kw):
    dg = llp.DeviceGraph(llpgen.CSRGraph(g, weighted=not bfs, out_weights=True))
    d = (llp.bfs if bfs else llp.sssp)(dg, s, **kw)
    torch.cuda.synchronize()
    return d.cpu().numpy()


def graph(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def hubs(n, deg, long_row, zero, seed):
    """Random arcs over the first 3/4 of the vertices (the rest have none), and
    a row of long_row in-arcs; weights from 0 or 1."""
    rng = np.random.default_rng(seed)
    k = 3 * n // 4
    src = rng.integers(0, k, n * deg)
    dst = rng.integers(0, k, n * deg)
    hs = rng.integers(0, k, long_row)
    src = np.concatenate([src, hs, np.arange(64)])
    dst = np.concatenate([dst, np.full(long_row, 5), (np.arange(64) + 1)])
    w = rng.integers(0 if zero else 1, 50, len(src))
    return graph(n, src, dst, w)


# the graphs of at least 2^18 arcs, 6 a vertex, take the marking kernel; rows of
# 512 (a block), 1024 (a wave) and more arcs
@pytest.mark.parametrize("n,deg,long_row", [(32768, 8, 0), (32767, 8, 511), (40000, 8, 513), (20000, 16, 1025),
                                            (9000, 40, 30000), (43000, 6, 1024), (600, 500, 600)])
@pytest.mark.parametrize("bfs", [False, True])
@pytest.mark.parametrize("zero", [False, True])
def test_against_oracle(n, deg, long_row, bfs, zero):
    g = hubs(n, deg, long_row, zero, n + long_row)
    want = oracle.sssp(g.n, g.src, g.dst, None if bfs else g.w, 0, bag=True)
    assert np.array_equal(solve(g, 0, bfs), want)


def star(arcs):
    """Source 0 with exactly `arcs` out-arcs into 50000 vertices, each with one
    arc on to a second half and enough arcs among the rest to reach 2^18 and 6
    a vertex."""
    n = 50001
    dst = 1 + np.arange(arcs) % 50000
    rng = np.random.default_rng(arcs)
    k = 6 * n
    s2, d2 = rng.integers(1, n, k), rng.integers(1, n, k)
    src = np.concatenate([np.zeros(arcs, np.int64), s2])
    return graph(n, src, np.concatenate([dst, d2]), rng.integers(1, 1000, arcs + k))


@pytest.mark.parametrize("arcs", [65535, 65536, 65537])
def test_round_limit(arcs):
    """The first round expands just below, at and above 2^16 arcs; the traced
    rounds add up to the solve's counters either way."""
    g = star(arcs)
    trace, st = llp.trace_buffer(256), llp.Stats()
    got = solve(g, 0, trace=trace, stats=st, flags=llp.TRACE)
    assert np.array_equal(got, oracle.sssp(g.n, g.src, g.dst, g.w, 0, bag=True))
    rec = llp.trace_records(trace, int(st.rounds))
    assert rec["in_edges"][0] == arcs and rec["out_count"][0] == 50000
    indeg = np.bincount(g.dst, minlength=g.n)
    assert rec["out_edges"][0] == indeg[1:].sum()
    assert rec["out_count"].sum() == st.candidates and rec["out_edges"].sum() == st.edges_inspected
    assert (rec["mode"] & 3 == 0).all()
