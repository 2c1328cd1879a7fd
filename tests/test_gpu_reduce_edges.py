"""GPU parity of the reduction at its edges: empty, one word, an array whose
first word is off the 16-byte alignment, odd counts, tiles just full, and
repeated sums in one workspace that held other data."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


@pytest.mark.parametrize("n", [0, 1, 2, 3, 511, 512, 513, 2047, 2048, 2049, 100003, 1048575, 4194304, 4194305])
def test_alignment_and_counts(n):
    x = llpgen.u64_words(n + 3, seed=n + 1)
    t = torch.from_numpy(x.view(np.int64)).cuda()
    ws = torch.full((1 << 16,), 0x5A, dtype=torch.uint8, device="cuda")
    for off in (0, 1, 2, 3):
        want = oracle.reduce_sum(x[off:off + n])
        for _ in range(2):
            assert llp.reduce_sum(t[off:off + n], ws=ws) == want
            got = llp.reduce_sum_noalloc(t[off:off + n])
            assert int(got.cpu().numpy().view(np.uint64)[0]) == want
