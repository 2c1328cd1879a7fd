"""GPU parity of the workgroup SSSP inside a batch at the edges of its steps:
blocks of 64 vertices, steps of 256 arc positions, rows of more than 256
arcs, more blocks than a wave looks at at once, multi-arcs, zero weights,
unreachable vertices, overflow and malformed arrays."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def hub_graph(n, deg, seed):
    """Two hubs of deg arcs (duplicates and self-loops among them) on a chain."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([np.full(deg, 0), np.full(deg, n // 2), np.arange(n - 1)])
    dst = np.concatenate([rng.integers(0, n, 2 * deg), np.arange(1, n)])
    return edges(n, src, dst, rng.integers(0, 50, src.size))


def graphs():
    out = []
    for n in (2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 1000, 4095, 4096, 4097, 8191, 8192):
        for deg in (1, 4, 8):
            out.append((llpgen.uniform_graph(n, deg * n, 1, 100, seed=n + deg, cycle=deg != 1), (7 * n) % n))
    for deg in (255, 256, 257, 511, 512, 513, 5000):
        out.append((hub_graph(300, deg, deg), 0))
    rng = np.random.default_rng(1)
    p = rng.permutation(2000)
    out.append((edges(2000, p[:-1], p[1:], rng.integers(0, 9, 1999)), int(p[0])))       # a chain, ids shuffled
    out.append((edges(2000, p[1:], p[:-1], np.zeros(1999)), int(p[-1])))                # all weights zero
    out.append((llpgen.grid_graph(64, 64, 1, 1000, seed=3), 100))
    out.append((edges(100, [0], [1], [2**31 - 2]), 0))
    return out


@pytest.mark.parametrize("shape", [dict(), dict(block=64), dict(block=128, chunk=2), dict(block=256), dict(block=512),
                                   dict(block=1024)], ids=str)
def test_batched_graphs(shape):
    gs = graphs()
    b = llp.Batch([("sssp", g, s) for g, s in gs]).solve(**shape)
    assert not b.status.any().item()
    for (g, s), got in zip(gs, b.results()):
        assert np.array_equal(got, oracle.sssp(g.n, g.src, g.dst, g.w, s, bag=True)), (g.n, g.m)


def test_overflow_and_malformed_instances():
    """Only the instances at fault report it; the kernel checks before use."""
    good = llpgen.uniform_graph(200, 800, 1, 100, seed=2)
    far = edges(3, [0, 1], [1, 2], [2**31 - 2, 5])
    bad_id = edges(3, [0, 1], [1, 7], [1, 1])
    negative = edges(3, [0, 1], [1, 2], [1, -1])
    b = llp.Batch([("sssp", good, 0), ("sssp", far, 0), ("sssp", bad_id, 0), ("sssp", negative, 0), ("sssp", good, 5)])
    with pytest.raises(llp.LLPError):
        b.solve()
    assert b.status.cpu().tolist() == [llp.OK, llp.E_OVERFLOW, llp.E_INPUT, llp.E_INPUT, llp.OK]
    r = b.results()
    assert np.array_equal(r[0], oracle.sssp(200, good.src, good.dst, good.w, 0))
    assert np.array_equal(r[4], oracle.sssp(200, good.src, good.dst, good.w, 5))


def test_graph_replay_after_the_table_changed():
    """A replay measures the limits and the order again in its one preparing launch."""
    items = llpgen.batch_workload(30, 30, seed=4, sssp_nhi=600)
    b = llp.Batch(items)
    want = llp.Batch(items).solve().results()
    desc = b.desc.clone()
    for k in range(4):
        b.out.zero_()
        b.solve(graph=True)
        assert all(np.array_equal(x, y) for x, y in zip(b.results(), want))
        # half of the instances shrink to nothing, then come back
        d = np.frombuffer(desc.cpu().numpy().tobytes(), llp.INSTANCE_DTYPE).copy()
        kn = np.nonzero(d["kind"] == llp.KIND_KNAPSACK)[0][:15]
        d["n"][kn] = 0
        b.desc.copy_(torch.from_numpy(d.view(np.uint8).copy()).cuda())
        b.solve(graph=True)
        out = b.out.cpu().numpy()
        assert all(out[b.out_slices[i][0]] == 0 for i in kn)
        b.desc.copy_(desc)
