"""The whole-tensor pruner's order, from the header that its kernels are built with: which elements reach a key, against the keys."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_18513_amd", "csrc")

SOURCE = r"""
#include "key_order.hpp"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace slimfit;

template <int BITS, bool MAG> long check(const std::vector<uint32_t> &elements, const std::vector<uint32_t> &edges)
{
    long wrong = 0, looked = 0;
    for (uint32_t lo : edges) {
        if (!reach_exists<BITS, MAG>(lo)) continue;
        const Reach r = reach_of<BITS, MAG>(lo);
        for (uint32_t b : elements) {
            ++looked;
            wrong += reaches<BITS, MAG>(b, r) != (key_of<BITS, MAG>(b) >= lo);
            if (!MAG && reach_is_positive<BITS>(lo)) wrong += reaches_positive<BITS>(b, lo) != (key_of<BITS, MAG>(b) >= lo);
        }
    }
    return looked ? wrong : -1;
}

int main()
{
    std::vector<uint32_t> all16, edges16, some32, edges32;
    for (uint32_t b = 0; b < 65536u; ++b) all16.push_back(b);
    for (uint32_t bin = 0; bin < 4096u; ++bin) {
        edges16.push_back(bin << 4);
        edges32.push_back(bin << 20);
    }
    uint64_t state = 88172645463325252ull;
    for (int i = 0; i < 20000; ++i) {
        state ^= state << 13; state ^= state >> 7; state ^= state << 17;
        some32.push_back((uint32_t)(state >> 16));
    }
    // both sides of every edge's own number, zeros, infinities and NaN of both signs
    for (uint32_t b : all16)
        for (uint32_t low : {0u, 1u, 0xFFFFu}) some32.push_back(b << 16 | low);
    printf("%ld %ld %ld %ld\n", check<16, true>(all16, edges16), check<16, false>(all16, edges16), check<32, true>(some32, edges32),
           check<32, false>(some32, edges32));
    // numbers in order have keys in order; -0 that of +0; NaN outside the infinities
    const uint32_t order[] = {0xFFC00000u, 0xFF800001u, 0xFF800000u, 0xC0000000u, 0xBF800000u, 0x80000001u, 0x00000000u, 0x00000001u, 0x3F800000u, 0x40000000u,
                              0x7F800000u, 0x7F800001u, 0x7FC00000u};
    for (int i = 1; i < 13; ++i)
        if (!(key_of<32, false>(order[i - 1]) < key_of<32, false>(order[i])) || !(key_of<16, true>(0x3F80u) < key_of<16, true>(0xC000u))) return 1;
    if (key_of<32, false>(0x80000000u) != key_of<32, false>(0u) || key_of<16, false>(0x8000u) != key_of<16, false>(0u)) return 1;
    return key_of<32, true>(0x80000000u) != key_of<32, true>(0u);
}
"""


@pytest.mark.parametrize("options", [["-O1"], ["-O3"]])
def test_what_reaches_an_edge_has_its_key(tmp_path, options):
    """Every bf16 element against every bin's lower edge, both orders; fp32 at random and around every edge."""
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", *options, "-I", CSRC, str(src), "-o", str(exe)], check=True)
    ran = subprocess.run([str(exe)], capture_output=True, text=True)
    assert ran.returncode == 0 and ran.stdout.split() == ["0"] * 4, ran.stdout
