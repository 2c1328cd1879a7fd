"""GPU parity of small graphs solved by one workgroup (the hybrid schedule
with nothing else asked for) against the oracle, around its limits on
vertices and arcs, with hubs, and repeated on one workspace between solves
of other sizes."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def check(g, s, ws=None):
    dg = llp.DeviceGraph(llpgen.CSRGraph(g, weighted=True, out_weights=True))
    d = llp.sssp(dg, s, ws=ws, sched=llp.SCHED_HYBRID).cpu().numpy()
    assert np.array_equal(d, oracle.sssp(g.n, g.src, g.dst, g.w, s, bag=True))
    lv = llp.bfs(dg, s, ws=ws, sched=llp.SCHED_HYBRID).cpu().numpy()
    assert np.array_equal(lv, oracle.bfs(g.n, g.src, g.dst, s))


@pytest.mark.parametrize("n,deg", [(2, 3), (63, 4), (64, 8), (65, 8), (1000, 16), (1024, 3), (1025, 3), (4096, 8),
                                   (5000, 18), (9999, 9), (10000, 9), (16383, 5), (16384, 5), (16385, 5), (12500, 7)])
def test_uniform(n, deg):
    """m = (deg + 1) n with the cycle: 100000 arcs at (10000, 9) and (12500, 7)."""
    check(llpgen.uniform_graph(n, deg * n, 1, 100, seed=n + deg), n - 1)


@pytest.mark.parametrize("scale", [6, 9, 12])
def test_rmat(scale):
    g = llpgen.rmat_graph(scale, seed=scale)
    check(g, llpgen.max_outdeg_source(g))


@pytest.mark.parametrize("rows,cols", [(8, 8), (32, 32), (33, 32), (100, 100)])
def test_grid(rows, cols):
    check(llpgen.grid_graph(rows, cols, 1, 1000, seed=rows), rows * cols // 2)


def test_one_workspace_for_many_sizes():
    ws = llp.workspace(llp.KIND_SSSP, 20000, 200000)
    for k in range(3):
        for n in (5000, 300, 20000, 64):
            check(llpgen.uniform_graph(n, 8 * n, 0, 50, seed=n + k), k, ws)
