"""GPU: well-formed batch instances that a workgroup solves after malformed
ones of many active blocks.  The bad id or weight is met some rounds into a
search, while other waves of the workgroup are at work."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


@pytest.mark.parametrize("block,per_claim", [(256, 4), (512, 60), (1024, 60)])
def test_good_instances_after_malformed_ones(block, per_claim):
    items, want = [], []
    for k in range(30):
        n = 4000 - 40 * k
        g = llpgen.uniform_graph(n, 4 * n, 1, 9, seed=k)
        late = int(np.argsort(oracle.bfs(n, g.src, g.dst, 0))[n // 2 + 30 * k])
        arc = int(np.flatnonzero(g.src == late)[0])
        (g.dst if k % 2 else g.w)[arc] = n + 5 if k % 2 else -1
        items.append(("sssp", g, 0))
        want.append(None)
        n = 3980 - 40 * k
        h = llpgen.uniform_graph(n, 4 * n, 0, 50, seed=100 + k)
        items.append(("sssp", h, 5))
        want.append(oracle.sssp(n, h.src, h.dst, h.w, 5))
    b = llp.Batch(items)
    for _ in range(3):
        b.out.fill_(-7)
        with pytest.raises(llp.LLPError):
            b.solve(block=block, chunk=per_claim)
        assert b.status.cpu().tolist() == [llp.E_INPUT if w is None else llp.OK for w in want]
        for got, w in zip(b.results(), want):
            assert w is None or np.array_equal(got, w)
