"""The MAC of more nodes than its launch has threads, against the same nodes in
parts that it has. Bytes: exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")


def test_mac_of_many_nodes():
    n = 1 << 21
    g = torch.Generator(device="cuda").manual_seed(3)
    a = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    r = cs.build(*a, ((0.0,) * 3, (1.0,) * 3), cs.HILBERT, 8)
    nk = r.node_keys
    assert nk.numel() > 1024 * 256
    print("[case] MAC of", nk.numel(), "nodes", flush=True)
    fa, fb = 1 << 61, (1 << 61) + (1 << 55) + 12345
    whole = cs.focus_mac(nk, cs.HILBERT, fa, fb, 0.5)
    parts = [cs.focus_mac(nk[i: i + 100003], cs.HILBERT, fa, fb, 0.5) for i in range(0, nk.numel(), 100003)]
    assert torch.equal(whole, torch.cat(parts))
    assert 0 < int(whole.sum()) < nk.numel()
