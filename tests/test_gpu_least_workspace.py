"""Calls that may have less workspace than they ask for: the same results. Whole
numbers: exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")

BOX = ((0.0,) * 3, (1.0,) * 3)


def same(a, b):
    for x, y in zip(a, b):
        assert torch.equal(x, y) if torch.is_tensor(x) else x == y


def test_results_with_the_least_workspace(monkeypatch):
    n = 100003
    g = torch.Generator(device="cuda").manual_seed(1)
    a = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    P = torch.sort(cs.compute_keys(*a, BOX, cs.HILBERT)).values
    fa, fb = int(P[n // 2]), int(P[n // 2 + 5000])
    off = np.linspace(0, n, 6).astype(np.uint64)
    calls = [("cstone_rebalance", lambda: cs.rebalance(P, 256, capacity=5000)),
             ("cstone_focus_rebalance", lambda: cs.focus_rebalance(P, 256, cs.HILBERT, fa, fb, 0.5, capacity=5000)),
             ("cstone_build_sharded", lambda: cs.build_sharded(*a, off, BOX, cs.HILBERT, 256, capacity=5000))]
    real = cs._workspace
    for name, call in calls:
        print("[case]", name, flush=True)
        want = call()
        asked = []

        def short(nbytes, device):
            asked.append(nbytes)
            if len(asked) == 1:
                raise torch.OutOfMemoryError("no memory")
            return real(nbytes, device)

        monkeypatch.setattr(cs, "_workspace", short)
        same(call(), want)
        monkeypatch.setattr(cs, "_workspace", real)
        assert len(asked) == 2 and asked[1] < asked[0]
