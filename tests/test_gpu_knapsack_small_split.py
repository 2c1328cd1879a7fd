"""GPU parity of the knapsack split at its narrowest rows and fewest items."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


@pytest.mark.parametrize("items,W", [(110, 3), (150, 40)])
def test_small_split(items, W):
    wt = llpgen.uniform_ints(items, 0, max(1, W // 2), seed=items)
    val = llpgen.uniform_ints(items, 0, 1000, seed=items + 1)
    ws = llp.workspace(llp.KIND_KNAPSACK, items, W)
    assert ws.numel() > 256
    want, want_row = oracle.knapsack(wt, val, W, row=True)
    best, row = llp.knapsack(wt, val, W, row=True, ws=ws)
    assert best == want and np.array_equal(row.cpu().numpy(), want_row)
