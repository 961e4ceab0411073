"""Domain bounds on both sides of the line between a wave and a thread per bound,
against their definition. Whole numbers: exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


@pytest.mark.parametrize("ranks", [1, 2, (1 << 14) - 1, 1 << 14, (1 << 14) + 1, 70001])
@pytest.mark.parametrize("nl", [1, 8, 50002])
def test_bounds(nl, ranks):
    rng = np.random.default_rng(nl + ranks)
    counts = rng.integers(0, 30, nl).astype(np.uint32)
    print("[case] bounds", nl, ranks, flush=True)
    got = cs.to_numpy(cs.sfc_partition(cs.from_numpy(counts, "cuda"), ranks))
    S = np.concatenate([[0], np.cumsum(counts.astype(np.uint64))])
    # the first i with S[i] * ranks >= r * S[nl], and nl for the last
    want = np.searchsorted(S * np.uint64(ranks), np.arange(ranks, dtype=np.uint64) * S[-1], side="left")
    assert np.array_equal(got, np.concatenate([want, [nl]]))
