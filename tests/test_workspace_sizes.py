"""Workspace sizes, asked on the host: a program may hold a workspace of the size
that an earlier version of the library asked for (the numbers below), so sorts
and builds ask for no more; and a workspace shorter than a call needs is refused
before anything is done."""
import ctypes

import pytest

import paper_2307_06345_amd as cs

lib = cs._lib

SORT = {0: 3173120, 1: 3177984, 1000: 3189760, 1 << 16: 4472576, (1 << 20) + 1: 24155136, 1 << 24: 338962944,
        (1 << 30) + 5: 21493737984}
BUILD = {(0, 1): 4221952, (1000, 1176): 4246784, (1 << 16, 10082): 6045696, (1 << 20, 162343): 33587968,
         (1 << 20, 1 << 20): 52018176, (1 << 24, 2582134): 474229504, (1500, 100000): 4755456}


@pytest.mark.parametrize("n", SORT)
def test_sorts_ask_for_no_more_than_they_did(n):
    assert lib.cstone_sort_workspace_bytes(n) <= SORT[n]


@pytest.mark.parametrize("n,cap", BUILD)
def test_builds_ask_for_no_more_than_they_did(n, cap):
    assert lib.cstone_build_workspace_bytes(n, cap) <= BUILD[n, cap]


@pytest.mark.parametrize("leaves", [1, 9])
def test_a_short_workspace_of_a_rebalance_is_refused(leaves):
    """Also where the direct tree would do with less than the rounds: whether they
    are needed shows only once the tree is known."""
    n, n_crit, cap = 1000, 64, 100000
    need = lib.cstone_rebalance_workspace_bytes(n, n_crit, cap)
    p = ctypes.c_void_p(1 << 40)  # never touched
    nl = ctypes.c_size_t(leaves)
    assert lib.cstone_rebalance(p, n, n_crit, p, ctypes.byref(nl), cap, None, 0, None, p, need - 1, None) == 1
