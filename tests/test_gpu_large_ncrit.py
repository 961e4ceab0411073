"""Large N_crit, against the CPU oracle: the waves of the tree's first pass that
look at a few keys only (N_crit from 512, the particles of a wave, on), particle
counts around N_crit and the waves' and tiles' edges, batches in which such sets
stand beside others. All outputs are integers and must match exactly."""
import numpy as np
import pytest

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


CASES = [("uniform", 511, 511), ("uniform", 513, 512), ("uniform", 1024, 512), ("uniform", 4096, 511), ("uniform", 4097, 513),
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
