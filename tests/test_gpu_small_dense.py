"""GPU parity of small graphs with long rows under the hybrid schedule: few
vertices around the limit on their arcs, hubs whose rows all waves share,
hubs side by side, ids that share their low bits, and frontiers of a few
vertices over many blocks."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def check(g, s):
    dg = llp.DeviceGraph(llpgen.CSRGraph(g, weighted=True, out_weights=True))
    want, levels = oracle.sssp(g.n, g.src, g.dst, g.w, s, bag=True), oracle.bfs(g.n, g.src, g.dst, s)
    for _ in range(3):
        assert np.array_equal(llp.sssp(dg, s, sched=llp.SCHED_HYBRID).cpu().numpy(), want)
        assert np.array_equal(llp.bfs(dg, s, sched=llp.SCHED_HYBRID).cpu().numpy(), levels)


@pytest.mark.parametrize("n,m", [(1, 50050), (1, 50051), (15, 50750), (16, 50800), (64, 53200), (64, 53201), (128, 56400),
                                 (960, 98000), (999, 99950), (1001, 100000)])
def test_arcs_at_the_limit(n, m):
    rng = np.random.default_rng(m)
    check(edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, 100, m)), n - 1)


@pytest.mark.parametrize("n", [90, 1025, 16384])
@pytest.mark.parametrize("deg", [4096, 4097, 48000])
def test_hub(n, deg):
    rng = np.random.default_rng(n + deg)
    src = np.concatenate([np.full(deg, 8), rng.integers(0, n, 3 * n)])[:50000 + 50 * n]
    check(edges(n, src, rng.integers(0, n, src.size), rng.integers(0, 100, src.size)), 8)


@pytest.mark.parametrize("hubs,deg", [(4, 2000), (64, 300), (64, 257), (380, 257)])
def test_hubs_side_by_side(hubs, deg):
    rng = np.random.default_rng(hubs + deg)
    src = np.concatenate([np.repeat(np.arange(hubs), deg), rng.integers(0, 2000, 2000)])
    check(edges(2000, src, rng.integers(0, 2000, src.size), rng.integers(0, 100, src.size)), 1)


@pytest.mark.parametrize("scale,ef", [(8, 60), (11, 16), (13, 6), (14, 4)])
@pytest.mark.parametrize("relabel", [False, True])
def test_rmat(scale, ef, relabel):
    g = llpgen.rmat_graph(scale, ef=ef, seed=scale, relabel=relabel)
    check(g, llpgen.max_outdeg_source(g))
