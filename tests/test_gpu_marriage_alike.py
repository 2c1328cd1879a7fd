"""GPU parity of stable marriage where many displacement chains are under way
at once: lists and ranks alike, so that chains go on in several passes, by
threads and by waves, inside the table of 64 positions and past it."""
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


def alike(n, strength, rng):
    """Lists sorted by a common order plus noise, as positions -> persons."""
    return np.argsort(np.arange(n) / n * strength + rng.random((n, n)), axis=1).astype(np.int16)


@pytest.mark.parametrize("n", [129, 400, 1100, 1500])
def test_same_lists_and_ranks(n):
    rng = np.random.default_rng(n)
    lists = np.tile(rng.permutation(n).astype(np.int16), (n, 1))
    up = np.arange(n, dtype=np.int16)
    for ranks in (up, up[::-1], rng.permutation(n).astype(np.int16)):
        check(lists, np.tile(ranks, (n, 1)))


@pytest.mark.parametrize("n,strength", [(300, 4), (1000, 32), (1300, 1)])
def test_lists_and_ranks_alike(n, strength):
    rng = np.random.default_rng(n)
    lists = alike(n, strength, rng)
    check(lists, np.argsort(alike(n, strength, rng), axis=1).astype(np.int16))
    check(lists, llpgen.sm_prefs(n, seed=n)[1])


@pytest.mark.parametrize("n,women", [(300, 200), (1100, 3), (1100, 70)])
def test_many_exhausted_lists(n, women):
    """Only some of the women are named, over and over: the other men run out of list, however many."""
    mpref = np.tile(np.resize(np.arange(women, dtype=np.int16), n), (n, 1))
    for ranks in (np.arange(n), np.arange(n)[::-1]):
        with pytest.raises(llp.LLPError) as e:
            llp.stable_marriage(mpref, np.tile(ranks.astype(np.int16), (n, 1)))
        assert e.value.status == llp.E_INFEASIBLE
