"""The index arithmetic with which a rebuild compares its new array with the one
before, compiled for the host: for every pair of positions that two searches in
an old array can give, in order or not (the keys of a tree of unsorted particles
come in any order), every key that is looked at lies among those that were read,
and those inside the old array."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_06345_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "overlap.hpp"

struct Staged {  // the keys a tile has read: an index past them ends the program
    const std::vector<uint64_t>& a;
    uint32_t first, held;
    uint64_t operator[](uint32_t i) const {
        if (i >= held || first + i >= a.size()) {
            std::printf("index %u of %u from %u\n", i, held, first);
            std::exit(1);
        }
        return a[first + i];
    }
};

int main() {
    unsigned long long looked = 0;
    for (uint32_t nl = 2; nl <= 40; ++nl) {
        std::vector<uint64_t> old(nl + 1);  // closing key included
        for (uint32_t i = 0; i <= nl; ++i) old[i] = 10 * i;
        for (uint32_t p0 = 0; p0 <= nl; ++p0)
            for (uint32_t p1 = 0; p1 <= nl; ++p1) {
                const cs::OldKeys o = cs::old_keys(p0, p1);
                if (!(o.first < o.last && o.last <= nl)) return std::printf("keys %u .. %u of %u\n", o.first, o.last, nl), 1;
                if (p1 > p0 && (o.first != (p0 ? p0 - 1 : 0) || o.last != p1)) return std::puts("trees are compared as before"), 1;
                const Staged b{old, o.first, o.last - o.first + 1};
                for (uint64_t k = 0; k <= 10 * nl + 10; k += 5) {
                    const uint32_t p = cs::at_or_before(b, 0u, o.last - o.first, k);
                    looked += b[p + 1] - b[p];
                }
                for (uint32_t i = p0; i < p1; ++i) looked += b[i - o.first + 1] - b[i - o.first];
            }
    }
    return looked ? 0 : 1;
}
"""


def test_a_rebuild_looks_at_keys_it_has_read(tmp_path):
    src = tmp_path / "overlap.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "overlap")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", exe, str(src)], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
