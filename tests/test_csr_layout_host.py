"""Host layout of CSR in-edges for the gather kernel: against its definition, edge by
edge, for rows in any order, empty rows, rows longer than a chunk and sizes around
the limits of row tiles, of the sort's passes and of packing."""
import os
import subprocess

import pytest

from paper_2410_19075_amd import build as nd_build

CSRC = nd_build.CSRC
DRIVER = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <random>
#include "csr_layout.h"
using namespace nd;
#define CHECK(c) do { if (!(c)) { std::printf("n %lld: line %d: %s\n", (long long)n, __LINE__, #c); return false; } } while (0)

// degree(i) edges in row i, ascending sources unless `shuffled`; hub: its degree
template <class KT, class F>
static bool check(int64_t n, F degree, bool shuffled) {
    std::mt19937_64 g(n);
    std::vector<int64_t> rp(n + 1, 0);
    std::vector<int32_t> col;
    std::vector<double> w;
    for (int64_t i = 0; i < n; ++i) {
        std::vector<int32_t> r(degree(i));
        for (auto& v : r) v = (int32_t)(g() % n);
        if (!shuffled) std::sort(r.begin(), r.end());
        for (int32_t v : r) col.push_back(v), w.push_back((double)(g() >> 11) * 0x1p-53);
        rp[i + 1] = (int64_t)col.size();
    }
    const CsrLayout<KT> L = csr_layout<KT>(n, rp.data(), col.data(), w.data());
    const int64_t rows = csr_rows(n);
    const bool packed = csr_packed(n);
    int64_t end = 0, widest = 1;
    for (int b = 0; b < kCsrSourceBlocks; ++b) {
        const int64_t lo = csr_block_begin(b, n), hi = csr_block_begin(b + 1, n);
        const int64_t* p = L.bptr.data() + (size_t)b * (n + 1);
        CHECK(p[0] == end);
        end = p[n];
        for (int64_t r0 = 0; r0 < n; r0 += rows) {
            const int64_t r1 = std::min(r0 + rows, n);
            // the tile's edges of the block in row order
            std::vector<int32_t> rc;
            std::vector<double> rw;
            for (int64_t i = r0; i < r1; ++i) {
                for (int64_t e = rp[i]; e < rp[i + 1]; ++e)
                    if (col[e] >= lo && col[e] < hi) rc.push_back(col[e]), rw.push_back(w[e]);
                CHECK(p[i + 1] - p[r0] == (int64_t)rc.size());
            }
            widest = std::max<int64_t>(widest, (int64_t)rc.size());
            for (size_t c0 = 0; c0 < rc.size(); c0 += kCsrChunk) {
                const size_t m = std::min<size_t>(kCsrChunk, rc.size() - c0);
                std::vector<char> seen(m, 0);
                for (size_t q = 0; q < m; ++q) {
                    const uint32_t v = L.col[p[r0] + c0 + q];
                    const size_t slot = packed ? v & (kCsrChunk - 1) : q;
                    CHECK(slot < m && !seen[slot]);
                    seen[slot] = 1;
                    const int64_t src = packed ? (v >> kCsrSlotBits) + lo : v;
                    CHECK(src == rc[c0 + slot]);
                    CHECK(L.w[p[r0] + c0 + q] == (KT)rw[c0 + slot]);
                    if (packed && q) {  // ascending sources, equal ones in row order
                        CHECK(L.col[p[r0] + c0 + q] > L.col[p[r0] + c0 + q - 1]);
                    }
                }
            }
        }
    }
    CHECK(end == (int64_t)col.size());
    CHECK(L.edges == std::min<int64_t>(kCsrChunk, widest));
    return true;
}

int main() {
    bool ok = true;
    for (int64_t n : {1, 3, 8, 255, 256, 257, 1000, 4096, 8200, 65535, 65536, 66001})
        for (bool shuffled : {false, true}) {
            ok = ok && check<double>(n, [](int64_t i) { return i % 5 == 0 ? 0 : 1 + i % 13; }, shuffled);
            ok = ok && check<float>(n, [](int64_t) { return 3; }, shuffled);
        }
    for (bool shuffled : {false, true}) {
        // dense tiles (one counting pass), a row with several chunks, no edges at all
        ok = ok && check<double>(2000, [](int64_t) { return 90; }, shuffled);
        ok = ok && check<float>(30000, [](int64_t i) { return i == 700 ? 150000 : 2; }, shuffled);
        ok = ok && check<double>(500, [](int64_t) { return 0; }, shuffled);
    }
    // the largest packed size and the first that keeps plain sources
    ok = ok && check<float>(int64_t(1) << 22, [](int64_t i) { return i % 4 == 0; }, false);
    ok = ok && check<float>((int64_t(1) << 22) + 1, [](int64_t i) { return i % 4 == 0; }, true);
    std::printf(ok ? "layout ok\n" : "layout wrong\n");
    return ok ? 0 : 1;
}
"""


@pytest.mark.skipif(not os.path.exists(nd_build.HIPCC), reason="hipcc not available")
def test_layout_against_its_definition(tmp_path):
    src, exe = tmp_path / "layout.hip", str(tmp_path / "layout")
    src.write_text(DRIVER)
    r = subprocess.run([nd_build.HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-I" + CSRC,
                        "-I" + os.path.join(nd_build.ROOT, "include"), str(src), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "layout ok" in r.stdout, r.stdout
