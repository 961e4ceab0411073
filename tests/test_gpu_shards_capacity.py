"""A sharded build whose tree exceeds the capacity, after the shards have come out
of one sort: the rounds that say how far it comes run on the parted shards, and
end as those of separately sorted shards do. Whole numbers: exact."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")

END = 1 << 63


@pytest.mark.parametrize("n,G", [(30000, 9), (70001, 64), (50000, 1)])
@pytest.mark.parametrize("short", [1, 3000])
def test_capacity_of_a_sharded_build(n, G, short):
    x, y, z = wl.uniform_cube(n, n + G)
    off = np.array([n * g // G for g in range(G + 1)], np.uint64)
    ref = oracle.build_tree(x, y, z, wl.UNIT_BOX, wl.HILBERT, 16)
    K0 = np.array([0, END], np.uint64)
    K, _, _, conv, hist = oracle.rebalance_iterate(ref["P"], K0, 16)
    assert conv
    cap = K.size - 1 - short
    print("[case] sharded capacity", n, G, cap, flush=True)
    d = [cs.from_numpy(a, "cuda") for a in (x, y, z)]
    P = torch.empty(n, dtype=torch.int64, device="cuda")
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    leaves = torch.empty(cap + 1, dtype=torch.int64, device="cuda")
    leaves[:2].copy_(cs.from_numpy(K0, "cuda"))
    p = off.ctypes.data_as(ctypes.c_void_p)
    ws = cs._workspace(cs._lib.cstone_build_sharded_workspace_bytes(p, G, cap), "cuda")
    nl, rounds = ctypes.c_size_t(1), ctypes.c_uint32(0)
    box = cs.Box.of(wl.UNIT_BOX)
    st = cs._lib.cstone_build_sharded(*(cs._ptr(t) for t in d), p, G, ctypes.byref(box), wl.HILBERT, 16, cs._ptr(P),
                                      cs._ptr(perm), cs._ptr(leaves), ctypes.byref(nl), cap, None, 0, ctypes.byref(rounds),
                                      cs._ptr(ws), ws.numel(), cs._stream())
    assert cs.STATUS[st] == "CAPACITY"
    arrays = [K0] + hist
    at = next(i for i, h in enumerate(arrays) if h.size - 1 > cap)
    assert nl.value == arrays[at].size - 1  # what the next round needed
    last = arrays[at - 1]
    assert np.array_equal(cs.to_numpy(leaves[: last.size]), last)
    hP, hperm = cs.to_numpy(P), cs.to_numpy(perm)
    for g in range(G):
        a, b = int(off[g]), int(off[g + 1])
        Pg, permg = oracle.sort(ref["keys"][a:b])
        assert np.array_equal(hP[a:b], Pg) and np.array_equal(hperm[a:b], permg), g
