"""The layout of the adaptive solver's scratch: pieces of any size are aligned for
every vector width, do not overlap and end inside the counted size."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_19075_amd", "csrc")
DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "carve.h"

struct alignas(16) Pair { double x, y; };
struct Block120 { char c[120]; };

// the mixture one batch of networks takes: odd counts of doubles, a block that is
// no multiple of 16 bytes, then maps read as 16-byte pairs
static size_t lay(nd::Carve c, char* base, int seed) {
    size_t end = 0, k = (size_t)seed;
    auto piece = [&](auto* q, size_t n) {
        k = k * 6364136223846793005ull + 1442695040888963407ull;
        if (!base) return;
        const size_t b = (size_t)((char*)q - base);
        if (b % 128 || b < end) { std::printf("piece at %zu, previous end %zu\n", b, end); std::exit(1); }
        end = b + n * sizeof(*q);
    };
    for (int b = 0; b < 5; ++b) {
        const size_t n = 1 + (k >> 33) % 999;
        piece(c.take<double>(9 * n), 9 * n);
        piece(c.take<Block120>(1), 1);
        piece(c.take<Pair>(n), n);
        piece(c.take<double>(0), 0);
        piece(c.take<int32_t>(n), n);
    }
    if (base && end > c.bytes()) { std::printf("end %zu beyond %zu\n", end, c.bytes()); std::exit(1); }
    return c.bytes();
}

int main() {
    for (int seed = 0; seed < 200; ++seed) {
        const size_t bytes = lay(nd::Carve(), nullptr, seed);
        char* buf = (char*)std::aligned_alloc(256, (bytes + 255) / 256 * 256);
        if (lay(nd::Carve(buf), buf, seed) != bytes) { std::printf("sizes differ\n"); return 1; }
        std::free(buf);
    }
    std::printf("layout ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_pieces_are_aligned_and_disjoint(tmp_path):
    src, exe = tmp_path / "carve.cpp", str(tmp_path / "carve")
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "layout ok" in r.stdout, r.stdout
