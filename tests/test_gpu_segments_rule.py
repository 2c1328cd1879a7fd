"""The library's own choice of list segments (one workgroup per CU below 2^21
arcs, two from there on): either side of the limit against the oracle, in the
scratch the size query states and with every explicit choice beside it."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


@pytest.mark.parametrize("m", [(1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("bfs", [False, True])
def test_limit(m, bfs):
    n = 30000
    g = llpgen.uniform_graph(n, m - n, seed=m)   # n arcs of a cycle and m - n random ones
    dg = llp.DeviceGraph(llpgen.CSRGraph(g, weighted=not bfs, out_weights=True))
    assert dg.m == m
    want = oracle.sssp(n, g.src, g.dst, None if bfs else g.w, 0, bag=True)
    fn = llp.bfs if bfs else llp.sssp
    ws = llp.workspace(llp.KIND_BFS if bfs else llp.KIND_SSSP, n, m)
    for sched in (llp.SCHED_HYBRID, llp.SCHED_PLAIN):
        for chunk in (0, 1, 2):
            got = fn(dg, 0, sched=sched, chunk=chunk, ws=ws)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want), (sched, chunk)
