"""The work split of the wide softmax, compiled for the host without HIP: it follows from the shape alone.

The order in which the column norms are added is that of the blocks, so a grid that depended on the device would
change their last bits from one device to another.
"""
import os
import shutil
import subprocess

import pytest

from paper_2211_12858_amd import build as sb_build

PROGRAM = """
#include <cstdio>
#include "sb_grad_plan.h"
int main() {
  long long n; int d, parts;
  while (std::scanf("%lld %d %d", &n, &d, &parts) == 3) {
    const sb::WidePlan p = sb::wide_plan(n, d, parts);
    std::printf("%d %d %d %d\\n", p.rows, p.waves, p.tiles, p.grid);
  }
}
"""


def test_wide_plan(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ is not available")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I" + os.path.abspath(sb_build.CSRC), str(src), "-o", str(exe)], check=True)
    shapes = [(n, d) for n in (1, 31, 33, 64, 255, 257, 20_001, 65_536, 300_007, 2_000_000, 2**31 - 1)
              for d in (105, 128, 129, 256, 257, 511, 512, 513, 576, 577, 640, 641, 1023, 1024)]
    text = "\n".join("%d %d %d" % (n, d, min((n + 255) // 256, 1536)) for n, d in shapes)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
    assert len(out.splitlines()) == len(shapes)
    for (n, d), line in zip(shapes, out.splitlines()):
        rows, waves, tiles, grid = map(int, line.split())
        cols = 32 * (64 // rows)
        assert rows == (64 if d <= 512 else 32) and waves <= 16
        assert (waves - 1) * cols < d <= waves * cols, "a wave without columns, or columns without a wave"
        assert tiles == -(-n // rows)
        parts = min(-(-n // 256), 1536)
        per = -(-tiles // grid)
        assert 1 <= grid <= min(parts, tiles), "more blocks than norm partials or tiles"
        assert (grid - 1) * per < tiles, "a block without tiles"
        # all that fit at once, so that the tiles per block are the fewest
        most = min(256 * (16 // waves), parts, tiles)
        assert per == -(-tiles // most)
