"""The rule that decides whether a wave's rectangle fits its LDS tile, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1908_02681_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

SOURCE = r"""
#include <cstdio>
#include "rz_internal.h"
int main()
{
    unsigned area, words, sh;
    while (std::scanf("%u %u %u", &area, &words, &sh) == 3)
        std::printf("%d\n", (int)rz::tile_fits(area, words, sh));
}
"""


def test_tile_rule_holds_for_every_area(tmp_path):
    """Areas on both sides of the tile's limit, and those of large screens (up to
    32768 x 32768) whose size in bytes passes 2^32, against 64-bit arithmetic."""
    if not shutil.which(CLANG):
        pytest.skip("clang not available")
    src, exe = tmp_path / "fits.cpp", tmp_path / "fits"
    src.write_text(SOURCE)
    subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROOT}/include", f"-I{CSRC}",
                    "-I/opt/rocm/include", str(src), "-o", str(exe)], check=True)
    areas = {1, 2, 3, 1 << 30}
    for near in [128, 256, 384, 512, 768, 1024] + [1 << k for k in range(20, 31)]:
        areas |= {near + d for d in (-1, 0, 1, 255, 256, 257, 383, 384, 385, 768, 769, 1024, 1025)}
    areas = sorted(a for a in areas if 1 <= a <= 1 << 30)
    rows = [(a, w, sh) for a in areas for w in (256, 768, 1024, 2048) for sh in (3, 4)]
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d" % r for r in rows),
                         capture_output=True, text=True, check=True).stdout.split()
    want = [str(int((a << sh) <= 8 * w)) for a, w, sh in rows]
    bad = [r for r, g, e in zip(rows, out, want) if g != e]
    assert len(out) == len(rows) and not bad, bad[:8]
