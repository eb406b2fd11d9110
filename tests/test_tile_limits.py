"""Limits that the host side of the library sets for the kernels, on the CPU: the rule that
decides whether a wave's rectangle fits its LDS tile, and the depths of a view that need
no clamp."""
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


RANGES = r"""
#include <cstdio>
#include <cstring>
#include "rz.h"
#include "rz_internal.h"
namespace rz {
int make_proj(const rz_view *v, const rz_depth_map *dm, Proj *P);
}
int main()
{
    int kind;
    double near_, far_, scale;
    while (std::scanf("%d %lf %lf %lf", &kind, &near_, &far_, &scale) == 4) {
        rz_view v;
        rz_depth_map dm;
        std::memset(&v, 0, sizeof v);
        std::memset(&dm, 0, sizeof dm);
        v.near_ = near_, v.far_ = far_, v.width = 64, v.height = 48;
        dm.kind = kind, dm.scale = scale;
        rz::Proj P;
        const int rc = rz::make_proj(&v, &dm, &P);
        std::printf("%d %.17g %.17g\n", rc, P.dlo[0], P.dhi[0]);
    }
}
"""


def test_depths_without_a_clamp(tmp_path):
    """Nearly all of [near, far) needs no clamp to the depth map's last value, whatever
    the map, far at 10^30 with the float encodings included."""
    from paper_1908_02681_amd import build
    if not shutil.which(CLANG) or not os.path.exists(build.LIB):
        pytest.skip("clang or the built library not available")
    src, exe = tmp_path / "ranges.cpp", tmp_path / "ranges"
    src.write_text(RANGES)
    subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROOT}/include", f"-I{CSRC}",
                    "-I/opt/rocm/include", str(src), build.LIB, "-L/opt/rocm/lib", "-lamdhip64",
                    f"-Wl,-rpath,{os.path.dirname(build.LIB)}", "-Wl,-rpath,/opt/rocm/lib",
                    "-o", str(exe)], check=True)
    rows = [(kind, near, far, 0.0) for kind in (0, 3, 4)
            for near, far in ((0.5, 4000.0), (1e-3, 1e9), (3300.0, 4700.0), (0.1, 1e13), (0.1, 1e30))]
    rows += [(1, 0.5, 4000.0, 1000.0), (1, 1.0, 2.0, 2.0 ** 38)]
    out = subprocess.run([str(exe)], input="\n".join("%d %r %r %r" % r for r in rows),
                         capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(rows)
    for (kind, near, far, scale), line in zip(rows, out):
        rc, lo, hi = line.split()
        assert rc == "0", (kind, near, far, scale)
        assert float(lo) == near and far - (far - near) * 2.0 ** -19 <= float(hi) <= far, (kind, far, line)
