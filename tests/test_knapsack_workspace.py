"""Workspace sizes of the knapsack (host side of libllp.so, no GPU)."""
import ctypes
import os

import pytest

from conftest import ROOT

LIB = os.path.join(ROOT, "paper_2603_13147_amd", "libllp.so")
KNAPSACK, HEADER = 5, 256

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libllp.so not built")


def size(items, W):
    lib = ctypes.CDLL(LIB)
    lib.llp_workspace_bytes.restype = ctypes.c_size_t
    lib.llp_workspace_bytes.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    return lib.llp_workspace_bytes(KNAPSACK, items, W, None)


@pytest.mark.parametrize("items,W", [(-1, 5), (5, -1), (1000, 16384), (1000, 10**5), (10**6, 2**31 - 1),
                                     (1000, 2**40), (2**31, 5000), (2**62, 100)])
def test_sizes_no_solve_accepts_ask_for_the_header(items, W):
    """So a binding that sizes first still gets the solver's argument error, not an allocation of gigabytes."""
    assert size(items, W) == HEADER


@pytest.mark.parametrize("items,W", [(110, 3), (150, 40), (100, 255), (257, 511), (257, 512), (300, 513), (1000, 767),
                                     (1000, 1024), (401, 4097), (999, 16383), (2000, 1500), (1500, 1500)])
def test_sizes_of_the_split_tests_split(items, W):
    """The GPU tests of the split have these sizes; a rule that kept them whole would empty those tests."""
    assert size(items, W) > HEADER


@pytest.mark.parametrize("items,W", [(0, 0), (1, 16383), (33, 40), (64, 256)])
def test_small_knapsacks_stay_whole(items, W):
    assert size(items, W) == HEADER
