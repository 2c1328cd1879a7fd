"""GPU parity of the grouped transitive closure at its edges: group and block
boundaries, rows longer than a wave walks lane by lane, deep chains in and
against id order, the 16-row groups of large n, and malformed inputs."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def closure(n, src, dst):
    g = llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.ones(len(src), np.int32))
    csr = llpgen.CSRGraph(g, weighted=False)
    return llp.transitive_closure(n, csr.out_ptr, csr.out_dst).cpu().numpy().view(np.uint32)


def expand(bits, n):
    return ((bits[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1).reshape(bits.shape[0], -1)[:, :n].astype(bool)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 128, 129, 160])
@pytest.mark.parametrize("deg", [1, 3])
def test_sizes(n, deg):
    g = llpgen.uniform_graph(n, deg * n, seed=n, cycle=False) if n > 1 else llpgen.EdgeList(
        1, np.zeros(1, np.int32), np.zeros(1, np.int32), np.zeros(1, np.int32))
    assert np.array_equal(closure(n, g.src, g.dst), oracle.transitive_closure(n, g.src, g.dst))


@pytest.mark.parametrize("deg", [63, 64, 65, 255, 256, 257, 700])
def test_long_rows(deg):
    """Hubs with deg arcs (duplicates and self-loops among them) beside short rows."""
    n = 300
    rng = np.random.default_rng(deg)
    src = np.concatenate([np.full(deg, 5), np.full(deg, 130), rng.integers(0, n, 100)])
    dst = rng.integers(0, n, src.size)
    assert np.array_equal(closure(n, src, dst), oracle.transitive_closure(n, src, dst))


@pytest.mark.parametrize("n", [200, 2111])
def test_chains(n):
    """i reaches exactly the later ones of its chain, whatever the order of the ids."""
    for p in (np.arange(n), np.arange(n)[::-1], np.random.default_rng(n).permutation(n)):
        got = expand(closure(n, p[:-1], p[1:]), n)
        pos = np.empty(n, np.int64)
        pos[p] = np.arange(n)
        assert np.array_equal(got, pos[:, None] < pos[None, :])


@pytest.mark.parametrize("n", [32768, 32769, 65535, 65536])
def test_largest(n):
    """Sampled rows against breadth-first reachability."""
    sp = pytest.importorskip("scipy.sparse")
    csg = pytest.importorskip("scipy.sparse.csgraph")
    g = llpgen.uniform_graph(n, n + n // 4, seed=n, cycle=False)
    got = closure(n, g.src, g.dst)
    A = sp.csr_matrix((np.ones(g.m, np.int8), (g.src, g.dst)), shape=(n, n))
    for u in [0, 15, 16, 31, 32, n - 17, n - 1] + [int(v) for v in llpgen.uniform_ints(25, 0, n - 1, seed=n)]:
        reach = np.zeros(n, bool)
        reach[csg.breadth_first_order(A, u, directed=True, return_predecessors=False)] = True
        reach[u] = bool(reach[g.src[g.dst == u]].any())
        assert np.array_equal(expand(got[u:u + 1], n)[0], reach), u


def test_malformed_rows_are_refused():
    """Ids and offsets out of range (checked by the kernel before use)."""
    n = 100
    for ptr, dst in [(np.arange(n + 1), np.full(n, n)), (np.arange(n + 1), np.full(n, -1)),
                     (np.concatenate([[5], np.arange(1, n + 1)]), np.zeros(n)),
                     (np.concatenate([np.arange(n), [n + 1]]), np.zeros(n))]:
        with pytest.raises(llp.LLPError) as e:
            llp.transitive_closure(n, ptr.astype(np.int32), dst.astype(np.int32))
        assert e.value.status == llp.E_INPUT
    # the same call with sound arrays works
    assert expand(closure(3, [0, 1], [1, 2]), 3).tolist() == [[0, 1, 1], [0, 0, 1], [0, 0, 0]]
