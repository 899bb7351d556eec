"""The eight-bit codes of gaps in time (compiled for the host from the kernels'
header, no GPU, under UndefinedBehaviorSanitizer): a code's floor is a lower
bound of every gap that has it, codes grow with the gap, and the gap 0 of an
edge given twice has a code like any other."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "tm_primitives.h"

int main() {
    uint32_t last = 0;
    for (int bit = 0; bit < 64; ++bit)
        for (u64 part = 0; part < 8; ++part) {
            const u64 gap = ((u64)1 << bit) + (bit >= 3 ? part << (bit - 3) : 0);
            const uint32_t c = gap_code(gap);
            if (c < last || c >= kGapNone || (u64)gap_floor(c) > gap) {
                std::printf("gap %llu: code %u, floor %lld\n", (unsigned long long)gap, c, (long long)gap_floor(c));
                return 1;
            }
            last = c;
        }
    // a floor is at least half of each of its gaps, up to the span of times a graph may have
    for (int bit = 0; bit < 62; ++bit)
        if ((u64)gap_floor(gap_code(((u64)2 << bit) - 1)) <= ((u64)1 << bit) - 1) return 2;
    if (gap_code(0) != gap_code(1) || gap_floor(kGapNone) < (int64_t)1 << 62) return 3;
    std::printf("gap codes ok\n");
    return 0;
}
"""


def test_gap_codes(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    src, exe = tmp_path / "gaps.hip", tmp_path / "gaps"
    src.write_text(SOURCE)
    r = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-Xarch_host",
                        "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all",
                        "-I" + os.path.join(ROOT, "paper_2507_20441_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "gap codes ok" in r.stdout, r.stdout + r.stderr
