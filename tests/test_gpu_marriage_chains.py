"""GPU parity of the single-workgroup stable-marriage chains where their forms
change: fewer men than a wave, lists just as long as the per-man table of 64
positions and longer, men rejected past the table (all men share one list),
and lists that run out."""
import numpy as np
import pytest

import llpgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
llp = pytest.importorskip("paper_2603_13147_amd")


def check(mpref, wrank):
    st = llp.Stats()
    wife, prop = llp.stable_marriage(mpref, wrank, stats=st)
    want_wife, want_prop = oracle.stable_marriage(mpref, wrank)[:2]
    assert np.array_equal(wife.cpu().numpy(), want_wife)
    assert np.array_equal(prop.cpu().numpy(), want_prop)
    assert st.advances == int(np.asarray(want_prop, np.int64).sum()) + len(want_prop)


@pytest.mark.parametrize("n", [3, 5, 6, 63, 64, 65, 70, 128, 129, 1023, 1025, 2049])
def test_random_lists(n):
    check(*llpgen.sm_prefs(n, seed=n))


@pytest.mark.parametrize("n", [64, 65, 127, 200, 333])
def test_one_list_for_all_men(n):
    """Man i ends i-th by rank: n (n + 1) / 2 proposals, most past the table;
    with the women's ranks reversed every chain displaces instead."""
    rng = np.random.default_rng(n)
    mpref = np.tile(rng.permutation(n).astype(np.int16), (n, 1))
    order = rng.permutation(n).astype(np.int16)
    check(mpref, np.tile(order, (n, 1)))
    check(mpref, np.tile(order[::-1].copy(), (n, 1)))
    check(mpref, llpgen.sm_prefs(n, seed=n + 1)[1])


@pytest.mark.parametrize("n", [2, 64, 100])
def test_exhausted_list(n):
    """All men name one woman throughout: all but one run out of list."""
    mpref = np.zeros((n, n), np.int16)
    with pytest.raises(llp.LLPError) as e:
        llp.stable_marriage(mpref, llpgen.sm_prefs(n, seed=1)[1])
    assert e.value.status == llp.E_INFEASIBLE
