"""The cut of a cell grid into bricks is plain arithmetic: for grids up to the most cells a system may
have (2^28), long thin ones among them, the bricks of a grid cover it once, stay within their
largest edge and within the replica's capacity.  Compiled for the host from the library's header."""
import os
import subprocess

import pytest

from paper_1507_07068_amd import build

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstdlib>
#include "md_bricks.hpp"
// n gx gy gz per case: "ok" or what is wrong
int main() {
  long long n;
  int gd[3];
  while (std::scanf("%lld %d %d %d", &n, gd, gd + 1, gd + 2) == 4) {
    const long long cap = md::brick_capacity(n, gd);
    int bn[3];
    const int per[3] = {1, 1, 1};
    md::choose_bricks(n, cap, gd, bn);
    const int bq[3] = {gd[0] / bn[0], gd[1] / bn[1], gd[2] / bn[2]};
    const char* bad = nullptr;
    if ((long long)bn[0] * bn[1] * bn[2] > cap) bad = "capacity";
    int next[3] = {0, 0, 0};
    for (int a = 0; a < 3 && !bad; ++a) {
      const long long step = a == 0 ? 1 : a == 1 ? bn[0] : (long long)bn[0] * bn[1];
      for (int i = 0; i < bn[a] && !bad; ++i) {
        const md::BrickHdr b = md::brick_geom(gd, bn, bq, per, 0, (int)(i * step));
        const int first = a == 0 ? b.x0 : a == 1 ? b.y0 : b.z0;
        const int cells = a == 0 ? b.x1 - b.x0 + 1 : a == 1 ? b.nry - 2 : b.nrows / b.nry - 2;
        if (first != next[a]) bad = "first cell";
        else if (cells < 1 || cells > md::BRICK_MAX) bad = "edge";
        else if (b.xa < 0 || b.xb >= gd[0] || b.xa > b.x0 || b.xb < b.x1) bad = "window";
        next[a] = first + cells;
      }
      if (!bad && next[a] != gd[a]) bad = "end";
    }
    std::printf("%lld %d %d %d: %s\n", n, gd[0], gd[1], gd[2], bad ? bad : "ok");
  }
}
"""

GRIDS = [(2000, 6, 6, 6), (300, 13, 5, 11), (8_000_000, 137, 137, 70), (216_000, 41, 41, 23), (5, 1, 1, 1),
         # dilute and dense axes past 113,500 cells (6-cell bricks) and 46,341 (1-cell bricks)
         (3000, 120_000, 3, 3), (3000, 3, 120_000, 3), (3000, 3, 3, 120_000), (50_000_000, 50_000, 3, 3),
         (1000, 1 << 20, 16, 16), (100, 1 << 28, 1, 1), (60_000_000, 1, 1, 1 << 20), (120_000_000, 645, 645, 645)]


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    d = tmp_path_factory.mktemp("brick_cut")
    src, exe = d / "cut.hip", d / "cut"
    src.write_text(PROGRAM)
    r = subprocess.run([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", build.CSRC, "-I",
                        os.path.join(build.ROOT, "include"), str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, g)) for g in GRIDS), capture_output=True,
                         text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    return dict(line.split(": ") for line in out.stdout.strip().splitlines())


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_bricks_cover_the_grid(cut, grid):
    assert cut[" ".join(map(str, grid))] == "ok"
