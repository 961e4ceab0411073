"""The look-back's fallback in the pass for the sort's extra digit, and in the pass
that reads its output: with no patience every wait goes to it, and crowded keys
are still sorted exactly."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


def test_fallback_of_the_extra_digit():
    n = (1 << 20) + 1
    rng = np.random.default_rng(8)
    core = rng.choice(1 << 27, n // 300, replace=False).astype(np.uint64) << np.uint64(36)
    keys = core[rng.integers(0, core.size, n)] | rng.integers(0, 1 << 36, n, dtype=np.uint64)
    keys[::7] = keys[3]  # ties
    rP, rperm = oracle.sort(keys)
    d = cs.from_numpy(keys, "cuda")
    splits = [v for v, s in enumerate(cs.sort_variant_splits()) if s]
    try:
        cs.set_lookback_patience(0)
        for v in [-1] + splits:
            print("[case] fallback of the extra digit, shape", v, flush=True)
            cs.tune_set(cs.TUNE_SORT, n, v)
            P, perm = cs.sort(d)
            assert np.array_equal(cs.to_numpy(P), rP) and np.array_equal(cs.to_numpy(perm), rperm), v
    finally:
        cs.set_lookback_patience(256)
        cs.tune_set(cs.TUNE_SORT, n, -1)
