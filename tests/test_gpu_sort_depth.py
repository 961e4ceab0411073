"""The sort's extra digit for crowded keys, against the oracle's stable sort:
buckets of one 36-bit prefix on both sides of the bucket kernel's limits (after
the extra digit they are its buckets), key counts on both sides of the least
that is sampled, and crowded keys given in sorted and in scattered order (the
sample must not depend on it)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


def crowded(n, bits, lo, hi, rng):
    """n keys in buckets of lo .. hi keys that share their top `bits` bits, the
    buckets in 200 clusters (so that 27-bit prefixes are crowded too); half of
    the low bits repeat."""
    sizes = rng.integers(lo, hi + 1, n // lo + 2)
    core = rng.choice(1 << 27, 200, replace=False).astype(np.uint64) << np.uint64(36)
    pre = core[rng.integers(0, 200, sizes.size)]
    if bits > 27:
        pre |= rng.integers(0, 1 << (bits - 27), sizes.size, dtype=np.uint64) << np.uint64(63 - bits)
    low = rng.integers(0, 1 << (63 - bits), n, dtype=np.uint64)
    low[::2] &= np.uint64(~np.uint64(0xFFFF))
    return np.repeat(pre, sizes)[:n] | low


@pytest.mark.parametrize("order", ["scattered", "sorted"])
@pytest.mark.parametrize("n,bits,lo,hi", [((1 << 20) - 1, 27, 1500, 2000), (1 << 20, 36, 40, 300),
                                          ((1 << 20) + 1, 36, 1900, 2100), (1100001, 36, 150, 170),
                                          (1 << 21, 36, 2500, 9000), (1300003, 45, 1, 3), (1200000, 63, 200, 5000)])
def test_sort_of_crowded_keys(n, bits, lo, hi, order):
    rng = np.random.default_rng(n + bits)
    keys = crowded(n, bits, lo, hi, rng)
    keys = np.sort(keys) if order == "sorted" else keys[rng.permutation(n)]
    print("[case] crowded sort", n, bits, lo, hi, order, flush=True)
    P, perm = cs.sort(cs.from_numpy(keys, "cuda"))
    rP, rperm = oracle.sort(keys)
    assert np.array_equal(cs.to_numpy(P), rP)
    assert np.array_equal(cs.to_numpy(perm), rperm)
    for shape in (2, 3, 4):
        cs.tune_set(cs.TUNE_SORT, n, shape)
        try:
            P2, perm2 = cs.sort(cs.from_numpy(keys, "cuda"))
        finally:
            cs.tune_set(cs.TUNE_SORT, n, -1)
        assert torch.equal(P, P2) and torch.equal(perm, perm2), shape


@pytest.mark.parametrize("n", [1 << 20, 1400001])
def test_build_of_a_crowded_set(n):
    """The build's own route: its key kernel counts the extra digit too."""
    rng = np.random.default_rng(n)
    x, y, z = (0.4 + 1e-3 * rng.standard_normal(n) for _ in range(3))
    x[: n // 10], y[: n // 10], z[: n // 10] = (rng.random(n // 10) for _ in range(3))
    box = ((0.0, 0.0, 0.0), (1.0, 1.0, 1.0))
    print("[case] crowded build", n, flush=True)
    r = cs.build(*(cs.from_numpy(a, "cuda") for a in (x, y, z)), box, cs.HILBERT, 16)
    ref = oracle.build_tree(x, y, z, box, cs.HILBERT, 16)
    for name, got in (("P", r.sorted_keys), ("perm", r.perm), ("K", r.leaves), ("counts", r.counts), ("NK", r.node_keys),
                      ("CO", r.child), ("LO", r.level_offsets)):
        assert np.array_equal(cs.to_numpy(got), ref[name]), name


def test_sort_of_crowded_keys_beyond_2_30():
    """The extra digit with 64-bit look-back words, whose rows its pass and the
    next one share; checked by what fixes a stable sort."""
    from tests import device_checks as dc
    n = (1 << 30) + 777
    g = torch.Generator(device="cuda").manual_seed(31)
    print("[case] crowded sort", n, flush=True)
    core = torch.randint(0, 1 << 27, (n // 1000,), device="cuda", generator=g) << 36
    keys = core[torch.randint(0, core.numel(), (n,), device="cuda", generator=g)]
    keys |= torch.randint(0, 1 << 36, (n,), device="cuda", generator=g)
    keys[:: 5] &= ~0xFFFFFF  # ties
    P, perm = cs.sort(keys)
    dc.check_sorted_perm(P, perm, n, keys)
