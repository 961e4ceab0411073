"""Which sorts take the extra digit, by the rule's own functions compiled for the
host: the sampled places lie in the keys, and the sample sees a cluster's crowded
prefixes in whatever order the keys come, while uniform keys, pairs and heaps of
equal keys (which the digit does not part) go without."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_06345_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>
#include "depth.hpp"

int main(int argc, char** argv) {  // a file of keys: prints whether they take the digit
    for (uint64_t n : {1ull << 20, (1ull << 20) + 1, 1ull << 24, (1ull << 32) - 1})
        for (uint32_t i = 0; i < cs::kDeepSample; ++i)
            if (cs::depth_place(i, n) >= n) return 2;
    FILE* f = std::fopen(argv[1], "rb");
    const uint64_t n = std::strtoull(argv[2], nullptr, 10);
    std::vector<uint64_t> keys(n);
    if (std::fread(keys.data(), 8, n, f) != n) return 2;
    std::map<uint64_t, uint64_t> first;  // prefix: word, with its count
    uint64_t pairs = 0, with_first = 0, together = 0;
    for (uint32_t i = 0; i < cs::kDeepSample; ++i) {
        const uint64_t w = cs::depth_word(keys[cs::depth_place(i, n)]);
        if ((w & cs::kDepthCount) || w == 0) return 2;
        auto [it, fresh] = first.try_emplace(w >> 32, w | 1);
        if (fresh) continue;
        if (!cs::depth_one_prefix(it->second, w)) return 2;
        pairs += it->second & cs::kDepthCount;
        ++with_first;
        together += cs::depth_one_digit(it->second, w);
        if ((it->second & cs::kDepthCount) < cs::kDepthCount) ++it->second;
    }
    std::printf("%d", int(cs::depth_pays(pairs, with_first, together, n)));
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("depth")
    (d / "depth.cpp").write_text(PROGRAM)
    exe = str(d / "depth")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", exe, str(d / "depth.cpp")], check=True)

    def takes(keys):
        keys.astype(np.uint64).tofile(str(d / "keys"))
        r = subprocess.run([exe, str(d / "keys"), str(keys.size)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        return r.stdout == "1"

    return takes


def random_keys(n, rng):
    return rng.integers(0, 1 << 63, n, dtype=np.uint64)


@pytest.mark.parametrize("order", ["scattered", "sorted"])
@pytest.mark.parametrize("n", [1 << 20, (1 << 22) + 5])
def test_crowded_prefixes_take_the_digit(program, n, order):
    rng = np.random.default_rng(n)
    core = rng.choice(1 << 27, n // 300, replace=False).astype(np.uint64) << np.uint64(36)  # 300 keys a prefix
    keys = core[rng.integers(0, core.size, n)] | rng.integers(0, 1 << 36, n, dtype=np.uint64)
    assert program(np.sort(keys) if order == "sorted" else keys)


@pytest.mark.parametrize("order", ["scattered", "sorted"])
@pytest.mark.parametrize("kind", ["uniform", "pairs", "equal", "heaps", "few"])
def test_keys_that_the_digit_does_not_part_go_without(program, kind, order):
    n = (1 << 20) + 77
    rng = np.random.default_rng(5)
    keys = random_keys(n, rng)
    if kind == "pairs":
        keys = np.repeat(keys, 2)[:n]
    elif kind == "equal":
        keys[:] = keys[0]
    elif kind == "heaps":  # a third on five places
        keys[: n // 3] = keys[rng.integers(0, 5, n // 3)]
        keys = keys[rng.permutation(n)]
    elif kind == "few":
        keys = keys[rng.integers(0, 1000, n)]
    assert not program(np.sort(keys) if order == "sorted" else keys)


def test_heaps_among_crowded_prefixes_take_the_digit(program):
    n = 1 << 21
    rng = np.random.default_rng(6)
    core = rng.choice(1 << 27, n // 2000, replace=False).astype(np.uint64) << np.uint64(36)
    keys = core[rng.integers(0, core.size, n)] | rng.integers(0, 1 << 36, n, dtype=np.uint64)
    keys[: n // 10] = keys[0]
    assert program(keys[rng.permutation(n)])
