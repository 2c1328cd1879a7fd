"""GPU parity of the transitive closure where the rows per group change with n
(one group per CU) and where a wave's vertices have at most two arcs or more."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")

CUS = 256


def closure(n, src, dst):
    g = llpgen.EdgeList(n, np.asarray(src, np.int32), np.asarray(dst, np.int32), np.ones(len(src), np.int32))
    csr = llpgen.CSRGraph(g, weighted=False)
    return llp.transitive_closure(n, csr.out_ptr, csr.out_dst).cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("n,deg", [(k * CUS + d, deg) for k in (1, 2, 4) for d in (-1, 0, 1) for deg in (1, 2, 3)
                                   if k < 4 or deg == 3])
def test_random(n, deg):
    """Every vertex has deg arcs, the last deg + 9."""
    rng = np.random.default_rng(n + deg)
    src = np.concatenate([np.repeat(np.arange(n), deg), np.full(9, n - 1)])
    dst = rng.integers(0, n, src.size)
    assert np.array_equal(closure(n, src, dst), oracle.transitive_closure(n, src, dst))


@pytest.mark.parametrize("n", [300, 1000, 8 * CUS, 8 * CUS + 1, 16 * CUS, 16 * CUS + 1])
def test_chains_and_trees(n):
    """Paths whose rows are known: i reaches the later ones of its chain; a binary tree's vertex its subtree."""
    p = np.random.default_rng(n).permutation(n)
    bits = closure(n, p[:-1], p[1:])
    got = np.unpackbits(bits.view(np.uint8), axis=1, bitorder="little")[:, :n].astype(bool)
    pos = np.empty(n, np.int64)
    pos[p] = np.arange(n)
    assert np.array_equal(got, pos[:, None] < pos[None, :])
    i = np.arange(1, n)
    bits = closure(n, (i - 1) // 2, i)
    got = np.unpackbits(bits.view(np.uint8), axis=1, bitorder="little")[:, :n].astype(bool)
    want = np.zeros((n, n), bool)
    for v in range(n - 1, 0, -1):
        want[(v - 1) // 2] |= want[v]
        want[(v - 1) // 2, v] = True
    assert np.array_equal(got, want)


def test_malformed_in_a_short_row():
    n = 600
    for bad in (n, -1):
        dst = np.arange(1, n + 1)
        dst[-1] = 0
        dst[400] = bad
        with pytest.raises(llp.LLPError) as e:
            llp.transitive_closure(n, np.arange(n + 1, dtype=np.int32), dst.astype(np.int32))
        assert e.value.status == llp.E_INPUT
