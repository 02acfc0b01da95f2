"""How a level of the discrepancy tail is dealt to workgroups (csrc/skim_tail.h), on
the CPU: every step of every tile of every pair, and every tile of an odd last
row, belongs to exactly one workgroup, so no two write the same outputs; the
parts and arrival counters stay within their buffers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include "skim_tail.h"
#include <cstdio>
#include <vector>
using namespace skim;
static int check(uint32_t rows, uint64_t cells) {
    const TailLevel L = tail_level(rows, cells);
    const uint32_t T = tail_tiles(cells);
    std::vector<std::vector<uint8_t>> seen(L.pairs * T);  // by step
    for (uint64_t p = 0; p < L.pairs; ++p)
        for (uint32_t t = 0; t < T; ++t) seen[p * T + t].assign(16 * t + 16, 0);
    std::vector<uint8_t> copied(T, 0);
    for (uint64_t i = 0; i < L.items; ++i) {
        const TailItem w = tail_item(L, i);
        if (w.pair >= L.pairs) {
            if (w.pair != L.pairs || w.tile >= T || copied[w.tile]++) return 1;
            continue;
        }
        if (w.nparts > 1 && (i - w.part >= kTailPartials || i >= kTailPartials ||
                             w.pair * T + w.tile >= kTailSplit)) return 2;
        for (int64_t t : {(int64_t)w.tile, (int64_t)w.more}) {  // (a second one only of whole tiles)
            if (t < 0) continue;
            if (t >= T) return 3;
            auto &s = seen[w.pair * T + t];
            const uint64_t d0 = (uint64_t)w.part * L.part;
            if (d0 >= s.size()) return 4;
            for (uint64_t d = d0; d < d0 + L.part && d < s.size(); ++d)
                if (s[d]++) return 5;  // a step done twice
        }
    }
    for (auto &s : seen)
        for (uint8_t x : s)
            if (!x) return 6;
    if (rows % 2)
        for (uint8_t x : copied)
            if (!x) return 7;
    return 0;
}
int main() {
    const uint32_t rows[] = {2, 3, 4, 5, 7, 50, 200, 341, 342, 511, 512, 513, 1023, 1024, 1025, 2047, 3001};
    const uint64_t cells[] = {2, 11, 255, 256, 257, 300, 512, 513, 768, 769, 1001, 4097, 9000, 65537};
    int bad = 0;
    for (uint32_t r : rows)
        for (uint64_t c : cells) {
            if ((double)r * (c / 256 + 1) * (c / 16 + 1) > 4e8) continue;
            const int e = check(r, c);
            if (e) std::printf("rows %u cells %llu: %d\n", r, (unsigned long long)c, e), bad = 1;
        }
    if (!bad) std::puts("every step once");
    return bad;
}
"""


def test_every_step_belongs_to_one_workgroup(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are not available")
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(CHECK)
    r = subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "paper_1408_6282_amd", "csrc"), str(src), "-o",
                        str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
