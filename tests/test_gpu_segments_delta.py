"""GPU: fixed pull rounds with delta buckets on both sides of their limit of
arcs for one list segment per CU, whatever the workgroups per CU, against the
oracle."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


@pytest.mark.parametrize("m", [(1 << 19) - 1, 1 << 19])
def test_limit(m):
    n = 5000
    g = llpgen.uniform_graph(n, m - n, 1, 100, seed=m)
    dg = llp.DeviceGraph(llpgen.CSRGraph(g, weighted=True, out_weights=True))
    want, levels = oracle.sssp(n, g.src, g.dst, g.w, 0, bag=True), oracle.bfs(n, g.src, g.dst, 0)
    ws = llp.workspace(llp.KIND_SSSP, n, m)
    for chunk in (0, 1, 2):
        for flags in (0, llp.PUSH):
            kw = dict(sched=llp.SCHED_FIXED, flags=flags, delta=40, chunk=chunk, ws=ws)
            assert np.array_equal(llp.sssp(dg, 0, **kw).cpu().numpy(), want), (chunk, flags)
            assert np.array_equal(llp.bfs(dg, 0, **kw).cpu().numpy(), levels), (chunk, flags)
