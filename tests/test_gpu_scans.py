"""Leaf-count scans (by way of the domain partition, which searches them) and
node counts, against the oracle: leaf counts around a scan tile (2048) and
around the number of tiles whose sums are scanned (2048), more domains than
waves, and node keys in other orders than the tree's. All exact."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


@pytest.mark.parametrize("nl,R", [(1, 1), (1, 5), (63, 5), (64, 5), (65, 70001), (2047, 5), (2048, 1), (2049, 5), (4095, 7),
                                  (100001, 1000), (2048 * 2048 - 1, 5), (2048 * 2048, 5), (5000001, 64)])
def test_partition_at_the_scan_limits(nl, R):
    rng = np.random.default_rng(nl + R)
    N = rng.integers(0, 40, nl).astype(np.uint32)
    N[rng.random(nl) < 0.3] = 0
    print("[case] partition", nl, R, flush=True)
    assert np.array_equal(cs.to_numpy(cs.sfc_partition(cs.from_numpy(N, "cuda"), R)), oracle.sfc_partition(N, R))


@pytest.mark.parametrize("n,n_crit", [(100, 200), (3000, 16), (60000, 4)])
def test_node_counts_in_any_order(n, n_crit):
    s = wl.make_set("plummer", n, 8, 0, wl.HILBERT, n_crit)
    ref = oracle.build_tree(s.x, s.y, s.z, s.box, s.curve, n_crit)
    NK, rng = ref["NK"], np.random.default_rng(n)
    K, N = cs.from_numpy(ref["K"], "cuda"), cs.from_numpy(ref["counts"], "cuda")
    lvl = np.array([(int(k).bit_length() - 1) // 3 for k in NK])
    start = np.array([(int(k) - (1 << (3 * int(l)))) << (3 * (21 - int(l))) for k, l in zip(NK, lvl)], np.uint64)
    end = np.array([int(a) + (1 << (3 * (21 - int(l)))) for a, l in zip(start, lvl)], np.uint64)
    want = (np.searchsorted(ref["P"], end) - np.searchsorted(ref["P"], start)).astype(np.uint32)
    print("[case] node counts", n, n_crit, NK.size, flush=True)
    for order in (np.arange(NK.size), np.arange(NK.size)[::-1], rng.permutation(NK.size)):
        got = cs.octree_node_counts(K, N, cs.from_numpy(np.ascontiguousarray(NK[order]), "cuda"))
        assert np.array_equal(cs.to_numpy(got), want[order])
