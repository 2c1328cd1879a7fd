"""GPU parity of batched graphs with one arc a vertex or none (chains, loops
with tails), and of steps beside it: a vertex with two arcs among them,
overflow at a chain's end, ids and offsets out of range in such a row."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def edges(n, src, dst, w):
    return llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.asarray(w, np.int32))


def chains():
    out = []
    rng = np.random.default_rng(9)
    for n in (2, 63, 64, 65, 129, 1001, 8192):
        p = rng.permutation(n)
        out.append((edges(n, p[:-1], p[1:], rng.integers(0, 9, n - 1)), int(p[0])))
        out.append((edges(n, np.arange(n), rng.integers(0, n, n), rng.integers(0, 9, n)), n // 2))    # a loop with tails
        src = np.concatenate([p[:-1], [p[n // 2]]])                                                   # one vertex of two arcs
        out.append((edges(n, src, np.concatenate([p[1:], [p[0]]]), rng.integers(0, 9, n)), int(p[0])))
    return out


@pytest.mark.parametrize("shape", [dict(), dict(block=64), dict(block=512, chunk=4), dict(block=1024)], ids=str)
def test_chains(shape):
    gs = chains()
    b = llp.Batch([("sssp", g, s) for g, s in gs]).solve(**shape)
    assert not b.status.any().item()
    for (g, s), got in zip(gs, b.results()):
        assert np.array_equal(got, oracle.sssp(g.n, g.src, g.dst, g.w, s, bag=True)), (g.n, g.m)


def test_faults_on_a_chain():
    n = 200
    i = np.arange(n - 1)
    heavy = np.ones(n - 1)
    heavy[[50, 60]] = 2**30 + 5
    bad_id = np.arange(1, n)
    bad_id[100] = n
    negative = np.ones(n - 1)
    negative[120] = -1
    good = edges(n, i, i + 1, np.ones(n - 1))
    b = llp.Batch([("sssp", good, 0), ("sssp", edges(n, i, i + 1, heavy), 0), ("sssp", edges(n, i, bad_id, np.ones(n - 1)), 0),
                   ("sssp", edges(n, i, i + 1, negative), 0), ("sssp", good, 7)])
    with pytest.raises(llp.LLPError):
        b.solve(chunk=5)
    assert b.status.cpu().tolist() == [llp.OK, llp.E_OVERFLOW, llp.E_INPUT, llp.E_INPUT, llp.OK]
    r = b.results()
    assert np.array_equal(r[0], np.arange(n))
    assert np.array_equal(r[4][7:], np.arange(n - 7)) and (r[4][:7] == 2**31 - 1).all()
