"""The radix sort's scratch size (compiled for the host from the kernels'
header, no GPU): a block sized for some number of keys serves every smaller
number too -- callers size it for their largest chunk -- also across the count
where the sort's tiles change size."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "tm_primitives.h"

constexpr int64_t kAt[] = {1, 1023, 1024, 1025, kSortSmall - 1, kSortSmall, kSortSmall + 1, 2 * kSortSmall,
                           4 * kSortSmall - 1, 4 * kSortSmall, 4 * kSortSmall + 1, (int64_t)1 << 28,
                           ((int64_t)1 << 31) - 1};
constexpr size_t words(int64_t n) { return (size_t)sort_tiles(n) * kSortDigits * sizeof(u64); }

constexpr bool holds() {
    for (int64_t large : kAt)
        for (int64_t small : kAt)
            if (small <= large &&
                (sort_status_bytes(large) < words(small) || sort_scratch_bytes(large) < sort_scratch_bytes(small)))
                return false;
    return true;
}
static_assert(holds(), "a sort of fewer keys needs more scratch than one of more keys");
static_assert(sort_status_bytes(0) == 0, "no keys, no status words");
"""


def test_scratch_of_many_keys_serves_fewer(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    src = tmp_path / "scratch.hip"
    src.write_text(SOURCE)
    r = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-fsyntax-only", "-std=c++17",
                        "-I" + os.path.join(ROOT, "paper_2507_20441_amd", "csrc"), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
