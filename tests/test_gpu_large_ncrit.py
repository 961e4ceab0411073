"""Large N_crit, against the CPU oracle: the line up to which nodes are read off
bytes (128), the waves of the tree's first pass that look at a few keys only
(N_crit from 512, the particles of a wave, on), particle counts around N_crit and
the waves' and tiles' edges, batches in which such sets stand beside others, and
both sides of the lines between the direct tree and the rounds. All outputs are
integers and must match exactly."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


def eq(got, ref, what):
    a = cs.to_numpy(got)
    assert a.shape == ref.shape and np.array_equal(a, ref), what


def points(kind, n, seed):
    x, y, z = wl.uniform_cube(n, seed)
    if kind == "crowd":  # most in a small corner: long chains of levels, and empty space
        k = n * 3 // 4
        for a in (x, y, z):
            a[:k] = 0.3 + a[:k] * 1e-3
    return x, y, z


CASES = [("uniform", 30000, 127), ("uniform", 30000, 128), ("uniform", 30000, 129), ("crowd", 70001, 129),
         ("uniform", 511, 511), ("uniform", 513, 512), ("uniform", 1024, 512), ("uniform", 4096, 511), ("uniform", 4097, 513),
         ("uniform", 70001, 512), ("uniform", 70001, 1000), ("uniform", 300007, 4095), ("uniform", 300007, 30000),
         ("crowd", 5000, 512), ("crowd", 70001, 700), ("crowd", 300007, 600), ("crowd", 300007, 5000), ("crowd", 20000, 19999)]


@pytest.mark.parametrize("kind,n,n_crit", CASES)
def test_build_of_large_leaves(kind, n, n_crit):
    print("[case] large leaves", kind, n, n_crit, flush=True)
    x, y, z = points(kind, n, n + n_crit)
    r = cs.build(*(cs.from_numpy(a, "cuda") for a in (x, y, z)), wl.UNIT_BOX, wl.HILBERT, n_crit)
    ref = oracle.build_tree(x, y, z, wl.UNIT_BOX, wl.HILBERT, n_crit)
    for name, got in (("K", r.leaves), ("counts", r.counts), ("NK", r.node_keys), ("CO", r.child), ("LO", r.level_offsets)):
        eq(got, ref[name], name)


def test_batch_of_large_and_small_leaves():
    """A set that keeps no byte per particle must still end the one before it."""
    sets = []
    for i, (kind, n, c) in enumerate(CASES):
        sets.append(wl.ParticleSet(*points(kind, n, i), wl.UNIT_BOX, i % 2, c, kind))
        m = 3000 + 37 * i
        sets.append(wl.ParticleSet(*points("crowd", m, 50 + i), wl.UNIT_BOX, i % 2, (1, 16, 256)[i % 3], "crowd"))
    print("[case] batch of", len(sets), "sets", flush=True)
    cat = [cs.from_numpy(np.concatenate([getattr(s, a) for s in sets]), "cuda") for a in "xyz"]
    b = cs.Batch([(s.n, s.box, s.curve, s.n_crit) for s in sets])
    b.ws[:].fill_(0xa5)  # no byte of the workspace is zero by chance
    b.upload()
    b.build(*cat)
    res = b.set_results()
    for i, s in enumerate(sets):
        v = b.set_view(i, res[i])
        ref = oracle.build_tree(s.x, s.y, s.z, s.box, s.curve, s.n_crit)
        assert v["status"] == "OK"
        for name, key in (("leaves", "K"), ("counts", "counts"), ("node_keys", "NK"), ("child", "CO"), ("level_offsets", "LO")):
            eq(v[name], ref[key], f"set {i} {name}")


@pytest.mark.parametrize("n", [1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("n_crit", [16, 1000])
def test_rebalance_from_another_tree_on_both_sides_of_the_line(n, n_crit):
    P = np.sort(oracle.compute_keys(*points("crowd", n, 1), wl.UNIT_BOX, wl.HILBERT)[0])
    Q = np.sort(oracle.compute_keys(*points("uniform", n, 2), wl.UNIT_BOX, wl.HILBERT)[0])
    print("[case] rebalance", n, n_crit, flush=True)
    for K0 in (oracle.build_leaves(Q, n_crit), oracle.build_leaves(P, n_crit), oracle.build_leaves(P, 4 * n_crit)):
        K, N, rounds, conv, _ = oracle.rebalance_iterate(P, K0, n_crit)
        assert conv
        gK, gN, r = cs.rebalance(cs.from_numpy(P, "cuda"), n_crit, leaves=cs.from_numpy(K0, "cuda"))
        eq(gK, K, "K")
        eq(gN, N, "counts")
        assert r == rounds


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1])
def test_focus_from_another_tree_on_both_sides_of_the_line(n):
    """The same tree comes from the root, which is always direct, and its rounds
    are the same as those of a call that a limit on them sends to the rounds."""
    g = torch.Generator(device="cuda").manual_seed(n)
    P = torch.sort(torch.randint(0, 1 << 62, (n,), device="cuda", generator=g)).values
    fa, fb = int(P[n // 3]), int(P[n // 3 + n // 64])
    print("[case] focus", n, flush=True)
    K0 = cs.focus_rebalance(P, 64, cs.HILBERT, 0, fa, 0.5)[0]
    want = cs.focus_rebalance(P, 64, cs.HILBERT, fa, fb, 0.5)
    a = cs.focus_rebalance(P, 64, cs.HILBERT, fa, fb, 0.5, leaves=K0)
    b = cs.focus_rebalance(P, 64, cs.HILBERT, fa, fb, 0.5, leaves=K0, max_iters=21)
    for got in (a, b):
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert a[2] == b[2]


@pytest.mark.parametrize("n_crit", [100, 300])
def test_rebuild_on_both_sides_of_the_line(n_crit):
    """2^25 particles: a rebuild with a leaf per 32 particles or more is direct,
    one with fewer leaves goes by rounds; both must be the build from the root."""
    n = 1 << 25
    g = torch.Generator(device="cuda").manual_seed(n_crit)
    a = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    print("[case] rebuild", n, n_crit, flush=True)
    b = cs.Builder(n, n_crit, leaf_capacity=n // 3)
    b.build(*a, wl.UNIT_BOX, cs.HILBERT, 16 if n_crit == 100 else n_crit)  # (finer: a leaf per 4 to 8)
    first = b.n_leaves
    assert (first >= n // 32) == (n_crit == 100)
    K0 = b.leaves[: first + 1].clone()
    for t in a:
        t.mul_(0.999)
    r = b.build(*a, wl.UNIT_BOX, cs.HILBERT, n_crit)
    want = [t.clone() for t in (r.sorted_keys, r.perm, r.leaves, r.counts, r.node_keys, r.child, r.level_offsets)]
    b.leaves[: first + 1].copy_(K0)
    b.n_leaves = first
    r = b.build(*a, wl.UNIT_BOX, cs.HILBERT, n_crit, incremental=True)
    got = (r.sorted_keys, r.perm, r.leaves, r.counts, r.node_keys, r.child, r.level_offsets)
    for i, (x, y) in enumerate(zip(got, want)):
        assert torch.equal(x, y), i
    K, N, rounds = cs.rebalance(r.sorted_keys, n_crit, leaves=K0, capacity=b.capacity, max_iters=21)
    assert torch.equal(K, r.leaves) and torch.equal(N, r.counts) and rounds == r.rounds
