"""The sort's tile shapes by size, against the oracle's stable sort: key counts
on both sides of the lines between the shapes, and around the tiles of the
smaller two (2048 and 4096 keys)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")

SIZES = [1, 63, 2047, 2048, 2049, 4097, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 4095, (1 << 20) - 1, 1 << 20,
         (1 << 20) + 1]


@pytest.mark.parametrize("n", SIZES)
def test_sort_beside_the_lines(n):
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    keys[::3] = keys[: keys[::3].size]  # ties, whose order has to be kept
    keys[1::5] &= np.uint64((1 << 37) - 1)  # one crowded level-9 octant
    print("[case] sort shape", n, flush=True)
    P, perm = cs.sort(cs.from_numpy(keys, "cuda"))
    rP, rperm = oracle.sort(keys)
    assert np.array_equal(cs.to_numpy(P), rP)
    assert np.array_equal(cs.to_numpy(perm), rperm)


@pytest.mark.parametrize("shape", [9, 10])
@pytest.mark.parametrize("n", [100003, (1 << 21) + 77])
def test_small_shapes_by_table(n, shape):
    """The small shapes where the table names them, also beyond their lines."""
    rng = np.random.default_rng(n + shape)
    keys = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    print("[case] sort shape by table", n, shape, flush=True)
    rP, rperm = oracle.sort(keys)
    cs.tune_set(cs.TUNE_SORT, n, shape)
    try:
        P, perm = cs.sort(cs.from_numpy(keys, "cuda"))
    finally:
        cs.tune_set(cs.TUNE_SORT, n, -1)
    assert np.array_equal(cs.to_numpy(P), rP)
    assert np.array_equal(cs.to_numpy(perm), rperm)


@pytest.mark.parametrize("n", [(3 << 19) - 1, 3 << 19, (3 << 19) + 1])
@pytest.mark.parametrize("kind", ["uniform", "crowded"])
def test_sort_beside_the_upper_line(n, kind):
    """The line between the middle and the largest shape, with and without the extra digit."""
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    if kind == "crowded":
        core = rng.choice(1 << 27, n // 200, replace=False).astype(np.uint64) << np.uint64(36)
        keys = core[rng.integers(0, core.size, n)] | (keys & np.uint64((1 << 36) - 1))
    print("[case] sort shape, upper line", n, kind, flush=True)
    P, perm = cs.sort(cs.from_numpy(keys, "cuda"))
    rP, rperm = oracle.sort(keys)
    assert np.array_equal(cs.to_numpy(P), rP)
    assert np.array_equal(cs.to_numpy(perm), rperm)
