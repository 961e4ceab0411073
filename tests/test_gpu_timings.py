"""Stage times of builds whose sort has buckets left after the host's look: the
low passes' time is theirs, and the tree before them is not the sort's."""
import pytest
import torch

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


def test_low_passes_after_the_look_are_timed():
    n = 1 << 24
    g = torch.Generator(device="cuda").manual_seed(1)
    a = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    heap = torch.randint(0, 9, (n,), device="cuda", generator=g)
    heaped = [torch.where(heap < 5, t[heap], t) for t in a]  # 5 points with a million particles and a half each
    b = cs.Builder(n, 64, leaf_capacity=n)
    box = ((0.0,) * 3, (1.0,) * 3)
    print("[case] timed builds", n, flush=True)
    plain, heaps = [], []
    for _ in range(5):
        plain.append(b.build(*a, box, cs.HILBERT, 64, timed=True))
        heaps.append(b.build(*heaped, box, cs.HILBERT, 64, timed=True))
    low = min(r.sort_pass_ms[3] for r in heaps)
    # five launches over 9 million listed keys, 24 B a key and pass: over 0.15 ms at 6 TB/s
    assert low > 0.15 and min(r.sort_pass_ms[3] for r in plain) < 0.05
    # the sort is its set-up launch and its passes: 0.06 ms is four times what the set-up takes
    assert min(r.stage_ms[1] - sum(r.sort_pass_ms) for r in heaps) < 0.06
    # both trees are in the rebalance stage: more than the one of a plain build takes
    assert min(r.stage_ms[2] for r in heaps) > 0.0
