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


class _Short:
    """Stands for the allocator: nothing longer than `most` bytes is to be had."""

    def __init__(self, most):
        self.most, self.asked = most, []

    def __call__(self, nbytes, device):
        self.asked.append(nbytes)
        if nbytes > self.most:
            raise cs.torch.OutOfMemoryError("no memory")
        return nbytes


def test_a_shorter_workspace_where_memory_is_short(monkeypatch):
    for most, got in ((1000, 800), (500, 300)):
        short = _Short(most)
        monkeypatch.setattr(cs, "_workspace", short)
        assert cs._workspace_or(800, lambda: 300, "cpu") == got
    for nbytes, least in ((800, 600), (800, 800), (600, 900)):
        monkeypatch.setattr(cs, "_workspace", _Short(500))
        with pytest.raises(cs.torch.OutOfMemoryError):
            cs._workspace_or(nbytes, lambda: least, "cpu")


def test_the_least_sizes_are_those_of_before():
    """What the calls asked for when they went by rounds and shard by shard."""
    import numpy as np
    for G, before in ((1, 473180928), (2, 305285888), (8, 268500224)):
        off = np.linspace(0, 1 << 24, G + 1).astype(np.uint64)
        cap = 10 * (1 << 24) // 65 + 1024
        p = off.ctypes.data_as(ctypes.c_void_p)
        least = lib.cstone_build_sharded_least_workspace_bytes(p, G, cap)
        assert 0 < least <= before < lib.cstone_build_sharded_workspace_bytes(p, G, cap)
    assert lib.cstone_rebalance_least_workspace_bytes(1 << 24, 1000, 168628) <= 2845440
    assert lib.cstone_focus_rebalance_least_workspace_bytes(1500) <= 43008
