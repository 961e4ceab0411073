"""Small sets of very small leaves, whose tiles' internal nodes several blocks
write, against the CPU oracle: N_crit on both sides of where that begins and
ends, one tile and many, chains of levels (every point twice), and a focused
tree. All outputs are integers and must match exactly."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


@pytest.mark.parametrize("n,n_crit", [(2, 1), (100, 1), (4096, 1), (5000, 1), (5000, 2), (9001, 4), (20000, 7), (20000, 8), (65536, 1),
                                      (262144, 1), (262145, 2), (700001, 1)])
@pytest.mark.parametrize("twice", [False, True])
def test_build_of_small_leaves(n, n_crit, twice):
    x, y, z = wl.uniform_cube(n, n + n_crit)
    if twice:
        x, y, z = (np.repeat(a[: (n + 1) // 2], 2)[:n].copy() for a in (x, y, z))
    print("[case] small leaves", n, n_crit, twice, flush=True)
    r = cs.build(*(cs.from_numpy(a, "cuda") for a in (x, y, z)), wl.UNIT_BOX, wl.HILBERT, n_crit)
    ref = oracle.build_tree(x, y, z, wl.UNIT_BOX, wl.HILBERT, n_crit)
    for name, got in (("K", r.leaves), ("counts", r.counts), ("NK", r.node_keys), ("CO", r.child), ("LO", r.level_offsets)):
        assert np.array_equal(cs.to_numpy(got), ref[name]), name


def test_focus_of_small_leaves():
    n = 9001
    P = np.sort(oracle.compute_keys(*wl.uniform_cube(n, 4), wl.UNIT_BOX, wl.HILBERT)[0])
    fa, fb = int(P[n // 3]), int(P[n // 2])
    print("[case] focus of small leaves", flush=True)
    dP = cs.from_numpy(P, "cuda")
    K, N, r = cs.focus_rebalance(dP, 1, cs.HILBERT, fa, fb, 0.5)
    K2, N2, r2 = cs.focus_rebalance(dP, 1, cs.HILBERT, fa, fb, 0.5, max_iters=21)  # by rounds
    assert np.array_equal(cs.to_numpy(K), cs.to_numpy(K2)) and np.array_equal(cs.to_numpy(N), cs.to_numpy(N2)) and r == r2
