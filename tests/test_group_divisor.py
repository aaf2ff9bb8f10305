"""The product that stands for the division by the group size in the decompressor, on the host, against the
division, for every group size the calls take."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2206_11357_amd", "csrc")

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include "gact_device.h"
int main() {
    for (int G = 32; G <= 1024; G += 32) {
        gact::Geometry geo{};
        geo.lpg = G / 32;
        gact::group_divisor(&geo);
        const uint64_t d = (uint64_t)G / 16, end = (uint64_t)gact::kMagicElems / 16;
        const auto bad = [&](uint64_t i) {
            if (i >= end) return false;
            return (((i * geo.group_magic) >> 32) >> geo.group_shift) != i / d;
        };
        // each group's first and last place on both ends of the range and at steps across it
        for (uint64_t g = 0; g * d < end; g += (g < 200000 || (end / d - g) < 200000) ? 1 : 997)
            if (bad(g * d) || bad(g * d + d - 1)) { std::printf("G %d, group %llu\n", G, (unsigned long long)g); return 1; }
        if (bad(end - 1)) { std::printf("G %d, end\n", G); return 1; }
    }
    return 0;
}
"""


def test_the_product_is_the_quotient_over_its_whole_range(tmp_path):
    src, exe = tmp_path / "divisor.cpp", tmp_path / "divisor"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout
