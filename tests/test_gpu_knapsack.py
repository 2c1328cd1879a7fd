"""GPU parity of the knapsack row sweep at the edges of its layout: cells per
thread just full and just over, rows that end inside a wave, weights at a
wave's first and last cell, item counts around the 64 loaded at a time, and
values around 2^31 - 1; and of the split into groups of items whose rows are
merged, against the oracle and against the same solve in a workspace too
small for the split."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def items_of(W, k, seed):
    """k items whose weights cover 0, W, the multiples of 64 and their neighbours, and a few above W."""
    wt = llpgen.uniform_ints(k, 0, W + 1, seed=seed).astype(np.int32)
    edge = [0, 1, W, W + 1, 63, 64, 65, 127, 128, 256, 512, 513]
    wt[: min(k, len(edge))] = edge[:k]
    return wt, llpgen.uniform_ints(k, 0, 1000, seed=seed, tag=0x61).astype(np.int32)


@pytest.mark.parametrize("items", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("block,W", [(64, 0), (64, 62), (64, 63), (64, 64), (64, 1023), (64, 1024), (64, 1300),
                                     (64, 2047), (512, 511), (512, 4095), (512, 4096), (512, 16383), (1024, 1022),
                                     (1024, 8191), (1024, 8192), (1024, 16383), (0, 640), (0, 6400)])
def test_knapsack_row_edges(block, W, items):
    wt, val = items_of(W, items, seed=1000 + W + items)
    want, want_row = oracle.knapsack(wt, val, W, row=True)
    best, row = llp.knapsack(wt, val, W, row=True, block=block)
    assert best == want
    assert np.array_equal(row.cpu().numpy(), want_row)


@pytest.mark.parametrize("k", [3, 40, 300])
def test_knapsack_values_at_the_int32_bound(k):
    """The total value just fits, then exceeds the bound by one; items that
    cannot be packed do not count; a negative weight is reported first."""
    wt = np.ones(k, np.int32)
    val = np.full(k, (2**31 - 1) // k, np.int32)
    val[k // 2] += (2**31 - 1) - int(val.astype(np.int64).sum())
    assert llp.knapsack(wt, val, k) == 2**31 - 1
    heavy = np.append(wt, k + 1).astype(np.int32), np.append(val, 5).astype(np.int32)
    assert llp.knapsack(*heavy, k) == 2**31 - 1
    val[k - 1] += 1
    with pytest.raises(llp.LLPError) as e:
        llp.knapsack(wt, val, k)
    assert e.value.status == llp.E_OVERFLOW
    wt[k - 1] = -1
    with pytest.raises(llp.LLPError) as e:
        llp.knapsack(wt, val, k)
    assert e.value.status == llp.E_INPUT


@pytest.mark.parametrize("items,W", [(33, 40), (100, 255), (257, 511), (257, 512), (300, 513), (1000, 767),
                                     (1000, 1024), (401, 4097), (999, 16383)])
def test_knapsack_split(items, W):
    wt, val = items_of(W, items, seed=77 + W)
    want, want_row = oracle.knapsack(wt, val, W, row=True)
    for ws in (None, torch.empty(256, dtype=torch.uint8, device="cuda")):
        best, row = llp.knapsack(wt, val, W, row=True, ws=ws)
        assert best == want
        assert np.array_equal(row.cpu().numpy(), want_row)


def test_knapsack_split_reused_workspace_and_errors():
    """Solves of other sizes in one workspace leave nothing behind; a bad item
    in the last group and an overflow that only the merges reach are seen."""
    W, k = 1500, 2000
    ws = llp.workspace(llp.KIND_KNAPSACK, 4000, 6400)
    for seed, (n, cap) in enumerate([(k, W), (4000, 6400), (700, 300), (k, W)]):
        wt, val = items_of(cap, n, seed=seed)
        best, row = llp.knapsack(wt, val, cap, row=True, ws=ws)
        want, want_row = oracle.knapsack(wt, val, cap, row=True)
        assert best == want and np.array_equal(row.cpu().numpy(), want_row)
    ones = np.ones(W, np.int32)
    val = np.full(W, (2**31 - 1) // W, np.int32)
    val[7] += (2**31 - 1) - int(val.astype(np.int64).sum())
    assert llp.knapsack(ones, val, W, ws=ws) == 2**31 - 1
    val[W - 1] += 1
    with pytest.raises(llp.LLPError) as e:
        llp.knapsack(ones, val, W, ws=ws)
    assert e.value.status == llp.E_OVERFLOW
    bad = ones.copy()
    bad[W - 1] = -1
    with pytest.raises(llp.LLPError) as e:
        llp.knapsack(bad, val, W, ws=ws)
    assert e.value.status == llp.E_INPUT
