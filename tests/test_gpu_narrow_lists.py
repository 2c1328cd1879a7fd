"""Lists with few entries in each segment, whose windows run over the ends of
segments: frontiers of 1 to 700 entries of one to a few hundred arcs, spread
over the segments by the round before, as graph rounds and as job levels."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def layers(widths, deg, seed):
    """Arcs from every vertex of a layer to deg random ones of the next, and one
    to each of those at least."""
    rng = np.random.default_rng(seed)
    base = np.concatenate([[0], np.cumsum(widths)])
    src, dst = [], []
    for k in range(len(widths) - 1):
        a, b = widths[k], widths[k + 1]
        s = np.concatenate([np.repeat(np.arange(a), deg), rng.integers(0, a, b)])
        t = np.concatenate([rng.integers(0, b, a * deg), np.arange(b)])
        src.append(base[k] + s)
        dst.append(base[k + 1] + t)
    return int(base[-1]), np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)


CASES = [([1, 63, 64, 65, 255, 257, 511, 513, 700, 3, 1], 2), ([1, 2, 300, 600, 600, 40, 600], 40),
         ([1, 30, 30, 30, 500, 500], 300), ([1, 700, 1, 700, 1], 1)]


@pytest.mark.parametrize("widths,deg", CASES)
@pytest.mark.parametrize("chunk", [0, 1, 2, 8])
def test_graph_rounds(widths, deg, chunk):
    n, src, dst = layers(widths, deg, 11)
    w = np.random.default_rng(5).integers(0, 100, src.size).astype(np.int32)
    dg = llp.DeviceGraph(llpgen.CSRGraph(llpgen.EdgeList(n, src, dst, w), weighted=True, out_weights=True))
    want = oracle.sssp(n, src, dst, w, 0, bag=True)
    for kw in (dict(sched=llp.SCHED_PLAIN), dict(sched=llp.SCHED_FIXED, flags=llp.PUSH),
               dict(sched=llp.SCHED_FIXED, flags=llp.PUSH, delta=50), dict(sched=llp.SCHED_FIXED, delta=50),
               dict(sched=llp.SCHED_HYBRID, max_rounds=n)):
        d = llp.sssp(dg, 0, chunk=chunk, **kw)
        torch.cuda.synchronize()
        assert np.array_equal(d.cpu().numpy(), want), kw


@pytest.mark.parametrize("widths,deg", CASES)
@pytest.mark.parametrize("chunk", [0, -1, 200])
def test_job_levels(widths, deg, chunk):
    n, src, dst = layers(widths, deg, 12)
    dur = np.random.default_rng(6).integers(1, 1000, n).astype(np.int32)
    order = np.argsort(dst, kind="stable")
    ptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n))]).astype(np.int32)
    idx = src[order]
    got = llp.jobs(ptr, idx, dur, *llpgen.job_succ(ptr, idx), chunk=chunk)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.jobs(ptr, idx, dur, bag=True))
