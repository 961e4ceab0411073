"""The tree written straight from the sorted keys, with its links, against the
CPU oracle: particle counts at the edges of its tiles (4096 particles; up to 64
tiles are summed without a scan), N_crit on both sides of the limits of its
searches, sets whose internal nodes outgrow a tile's slots (chains of one-child
nodes), duplicates that cannot split; and trees reached from another tree at
capacities around the longest array on the way. All outputs are integers and
must match exactly."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")

END = 1 << 63


def eq(a, b, what):
    a, b = np.asarray(cs.to_numpy(a)), np.asarray(b)
    assert a.shape == b.shape, (what, a.shape, b.shape)
    bad = np.nonzero(a != b)[0]
    assert bad.size == 0, f"{what}: {bad.size} mismatches, first at {bad[:5]}: {a[bad[:5]]} vs {b[bad[:5]]}"


def points(kind, n, seed):
    """Coordinates in the unit box."""
    if kind == "uniform":
        return wl.uniform_cube(n, seed)
    if kind == "pairs":  # every point twice: a chain of one-child nodes down to level 21 for every pair
        x, y, z = wl.uniform_cube((n + 1) // 2, seed)
        return tuple(np.repeat(a, 2)[:n].copy() for a in (x, y, z))
    if kind == "heaps":  # a few points with hundreds of particles each among others
        x, y, z = wl.uniform_cube(n, seed)
        i = np.random.default_rng(seed).integers(0, 9, n)
        return tuple(np.where(i < 5, a[i], a) for a in (x, y, z))
    raise ValueError(kind)


CASES = [("uniform", 4095, 64), ("uniform", 4096, 1), ("uniform", 4097, 2), ("uniform", 8193, 255),
         ("uniform", 30000, 256), ("uniform", 30000, 257), ("uniform", 20000, 4095), ("uniform", 20000, 19999),
         ("uniform", 300, 300), ("uniform", 64 * 4096, 64), ("uniform", 64 * 4096 + 1, 8), ("uniform", 700001, 16),
         ("pairs", 4096, 1), ("pairs", 20001, 1), ("heaps", 20000, 1), ("heaps", 50001, 64), ("heaps", 300007, 16)]


@pytest.mark.parametrize("kind,n,n_crit", CASES)
@pytest.mark.parametrize("curve", [wl.MORTON, wl.HILBERT])
def test_build_at_the_tree_pass_limits(kind, n, n_crit, curve):
    print("[case] tree", kind, n, n_crit, curve, flush=True)
    x, y, z = points(kind, n, n + n_crit)
    r = cs.build(*(cs.from_numpy(a, "cuda") for a in (x, y, z)), wl.UNIT_BOX, curve, n_crit)
    ref = oracle.build_tree(x, y, z, wl.UNIT_BOX, curve, n_crit)
    for name, got in (("K", r.leaves), ("counts", r.counts), ("NK", r.node_keys), ("CO", r.child),
                      ("LO", r.level_offsets)):
        eq(got, ref[name], name)
    depth = int(np.nonzero(np.diff(ref["LO"].astype(np.int64)))[0].max())
    assert r.rounds == depth + 1  # every level is a round, and one round sees no change


def test_batch_of_the_tree_pass_limits():
    sets = [wl.ParticleSet(*points(kind, n, n + c), wl.UNIT_BOX, i % 2, c, kind)
            for i, (kind, n, c) in enumerate(CASES)] + [wl.make_set("uniform", 0, 3, 0, wl.MORTON, 5000)]
    print("[case] batch of", len(sets), "sets", flush=True)
    cat = [cs.from_numpy(np.concatenate([getattr(s, a) for s in sets]), "cuda") for a in "xyz"]
    b = cs.Batch([(s.n, s.box, s.curve, s.n_crit) for s in sets])
    for rounds in (22, 5):  # 5: cut at level 5, as five literal rounds from the root leave the array
        b.set_rounds(rounds)
        b.build(*cat)
        res = b.set_results()
        for i, s in enumerate(sets):
            v = b.set_view(i, res[i])
            P = np.sort(oracle.compute_keys(s.x, s.y, s.z, s.box, s.curve)[0])
            K, N, r, conv, _ = oracle.rebalance_iterate(P, np.array([0, END], np.uint64), s.n_crit, rounds)
            assert v["status"] == ("OK" if conv else "NOT_CONVERGED") and v["rounds"] == r, (i, v["status"], v["rounds"], r)
            eq(v["leaves"], K, f"set {i} K")
            eq(v["counts"], N, f"set {i} counts")
            for name, got, want in zip(("NK", "CO", "LO"), (v["node_keys"], v["child"], v["level_offsets"]),
                                       oracle.link_octree(K)):
                eq(got, want, f"set {i} {name}")


@pytest.mark.parametrize("coarse,fine", [(64, 4), (4, 64), (16, 16)])
def test_rebalance_from_another_tree_at_tight_capacities(coarse, fine):
    """The start tree is finer in one half of the curve and coarser in the
    other, so the rounds split and merge at once; the capacity runs around the
    longest array on the way, and the outcome is that of the literal rounds."""
    n = 40000
    P = np.sort(oracle.compute_keys(*points("uniform", n, 5), wl.UNIT_BOX, wl.HILBERT)[0])
    Q = np.sort(oracle.compute_keys(*points("heaps", n, 6), wl.UNIT_BOX, wl.HILBERT)[0])
    half = END // 2
    a, b = oracle.build_leaves(Q, coarse), oracle.build_leaves(Q, fine)
    K0 = np.concatenate([a[a < half], b[b >= half]]).astype(np.uint64)
    K, N, rounds, conv, hist = oracle.rebalance_iterate(P, K0, 16)
    assert conv
    longest = max(h.size - 1 for h in hist)
    caps = {c for c in (longest + 5000, longest, longest - 1, K.size - 1) if c >= K0.size - 1} | {K0.size - 1}
    for cap in sorted(caps):  # (a capacity below the start array is refused)
        print("[case] from another tree", coarse, fine, "capacity", cap, flush=True)
        first_over = next((h.size - 1 for h in hist if h.size - 1 > cap), None)
        if first_over is None:
            gK, gN, r = cs.rebalance(cs.from_numpy(P, "cuda"), 16, leaves=cs.from_numpy(K0, "cuda"), capacity=cap)
            eq(gK, K, "K")
            eq(gN, N, "counts")
            assert r == rounds
        else:
            with pytest.raises(cs.CstoneError) as e:
                cs.rebalance(cs.from_numpy(P, "cuda"), 16, leaves=cs.from_numpy(K0, "cuda"), capacity=cap)
            assert e.value.name == "CAPACITY" and e.value.n_leaves == first_over
            last = [K0] + hist
            at = next(i for i, h in enumerate(last) if h.size - 1 > cap) - 1
            eq(e.value.buffer[: last[at].size], last[at], "last array that fitted")


@pytest.mark.parametrize("n", [50001, (1 << 20) + 3])
def test_rebuild_of_heaps_from_the_tree_before(n):
    """Particles heaped on a few points: buckets that the sort leaves to its
    low passes, which the build runs (with the tree) once it has seen them. The
    tree before must still be there to start from."""
    H, c = wl.HILBERT, 16
    print("[case] rebuild of heaps", n, flush=True)
    b = cs.Builder(n, c, leaf_capacity=n + 64)
    first = points("uniform", n, 1)
    b.build(*(cs.from_numpy(a, "cuda") for a in first), wl.UNIT_BOX, H, c)
    K0 = oracle.build_leaves(np.sort(oracle.compute_keys(*first, wl.UNIT_BOX, H)[0]), c)
    x, y, z = points("heaps", n, 2)
    ref = oracle.build_tree(x, y, z, wl.UNIT_BOX, H, c)
    _, _, rounds, _, _ = oracle.rebalance_iterate(ref["P"], K0, c)
    for timed in (False, True):
        b.n_leaves = K0.size - 1
        b.leaves[: K0.size].copy_(cs.from_numpy(K0, "cuda"))
        r = b.build(*(cs.from_numpy(a, "cuda") for a in (x, y, z)), wl.UNIT_BOX, H, c, incremental=True, timed=timed)
        for name, got in (("P", r.sorted_keys), ("perm", r.perm), ("K", r.leaves), ("counts", r.counts),
                          ("NK", r.node_keys), ("CO", r.child), ("LO", r.level_offsets)):
            eq(got, ref[name], name)
        assert r.rounds == rounds
