"""The gather of three coordinate arrays by way of packed records, bit for bit
against indexing: particle counts around the least that is packed (2^21) and
the tiles (1024 and 2048), permutations that scatter, that do not, and on both sides of
the line between, sources at odd addresses, and the calls that stay with the
separate passes (selections, results over sources). Copies: no tolerance."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

cs = pytest.importorskip("paper_2307_06345_amd")

M = 1 << 21


def perm_of(kind, n, rng):
    p = np.arange(n)
    if kind == "random":
        return rng.permutation(n)
    if kind == "reversed":
        return p[::-1]
    if kind == "near":  # shuffled within 64
        return np.concatenate([b + rng.permutation(min(64, n - b)) for b in range(0, n, 64)])
    k = {"fifth": n // 5, "third": n // 3}[kind]  # the first k at random, the rest in order
    return np.concatenate([rng.permutation(k), p[k:]])


def same(out, src, idx):
    for o, s in zip(out, src):
        assert torch.equal(o.view(torch.int64), s.view(torch.int64)[idx])


@pytest.mark.parametrize("kind", ["random", "reversed", "near", "fifth", "third"])
@pytest.mark.parametrize("n", [M - 1, M, M + 1, M + 1023, M + 1025])
def test_packed_gather(n, kind):
    rng = np.random.default_rng(n)
    idx = torch.from_numpy(np.ascontiguousarray(perm_of(kind, n, rng))).cuda()
    g = torch.Generator(device="cuda").manual_seed(n)
    bits = [torch.randint(-(1 << 62), 1 << 62, (n + 1,), device="cuda", generator=g) for _ in range(3)]  # any bits, NaN too
    src = [b.view(torch.float64)[k % 2: n + k % 2] for k, b in enumerate(bits)]  # one at an odd multiple of 8 B
    print("[case] packed gather", n, kind, flush=True)
    out = cs.gather_xyz(*src, idx.to(torch.int32))
    same(out, src, idx)


def test_packed_gather_elsewhere():
    n = M + 77
    g = torch.Generator(device="cuda").manual_seed(1)
    src = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    idx = torch.randperm(n, device="cuda", generator=g)
    perm = idx.to(torch.int32)
    same(cs.gather_xyz(*src, perm[:M]), src, idx[:M])  # a selection
    want = [s[idx] for s in src]
    work = [s.clone() for s in src]
    spare = torch.empty_like(src[0])
    cs.gather_xyz(*work, perm, out=(spare, work[0], work[1]))  # each pass over the array before it
    for o, w in zip((spare, work[0], work[1]), want):
        assert torch.equal(o, w)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    out = cs.gather_xyz(*src, perm, stream=s)
    torch.cuda.current_stream().wait_stream(s)
    same(out, src, idx)


def test_packed_gather_in_a_graph():
    """The choice between records and arrays is made on the device, replay by replay."""
    n = M + 5
    g = torch.Generator(device="cuda").manual_seed(2)
    src = [torch.rand(n, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    perm = torch.arange(n, dtype=torch.int32, device="cuda")
    out = [torch.empty_like(s) for s in src]
    cs.gather_xyz(*src, perm, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cs.gather_xyz(*src, perm, out=out)
    for k in range(4):
        idx = torch.randperm(n, device="cuda", generator=g) if k % 2 == 0 else torch.arange(n, device="cuda")
        perm.copy_(idx.to(torch.int32))
        for s in src:
            s.mul_(1.25)
        graph.replay()
        torch.cuda.synchronize()
        same(out, src, idx)
