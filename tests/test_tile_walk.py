"""Every tile of a product is taken by exactly one workgroup: the walk of
csrc/tile_walk.h, compiled for the host and composed as the product kernel does (whole
tiles, in ranges or in rounds, then the parts of a last round), over many numbers of
tiles and slices."""
import os
import subprocess

import pytest

from paper_2602_02549_amd.build import CSRC, hipcc

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "tile_walk.h"
using namespace oz2;

static bool covers(int tx, int ty, int nz, bool rounds, bool cut) {
  const int tiles = tx * ty * nz, parts = cut ? tail_parts(tiles) : 0;
  const int full = parts ? tiles / kCus * kCus : tiles, group = rounds ? 16 : 8;
  const int grid = full + (tiles - full) * parts;
  std::vector<int> seen((size_t)tiles * 4, 0);
  for (int bid = 0; bid < grid; ++bid) {
    TilePos t;
    int first = 0, count = 4;
    if (bid >= full) {
      const int place = xcd_place(bid - full, grid - full);
      t = tile_at(full + place / parts, tx, ty, group);
      count = 4 / parts;
      first = place % parts * count;
    } else {
      t = tile_at(rounds ? round_place(bid, full) : xcd_place(bid, full), tx, ty, group);
    }
    if (t.z < 0 || t.z >= nz || t.tx < 0 || t.tx >= tx || t.ty < 0 || t.ty >= ty) return false;
    for (int q = first; q < first + count; ++q)
      ++seen[(((size_t)t.z * tx + t.tx) * ty + t.ty) * 4 + q];
  }
  for (int s : seen)
    if (s != 1) return false;
  return true;
}

int main() {
  long checked = 0;
  for (int tx = 1; tx <= 40; tx += tx < 20 ? 1 : 4)
    for (int ty = 1; ty <= 40; ty += ty < 20 ? 1 : 4)
      for (int nz : {1, 2, 3, 7, 14, 16, 17, 22, 25, 33, 49})
        for (int mode = 0; mode < 4; ++mode, ++checked)
          if (!covers(tx, ty, nz, mode & 1, mode & 2)) {
            std::printf("%d x %d x %d mode %d\n", tx, ty, nz, mode);
            return 1;
          }
  std::printf("checked %ld\n", checked);
}
"""


def test_every_tile_once(tmp_path):
    try:
        cc = hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    p = subprocess.run([cc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, env=dict(os.environ))
    assert out.returncode == 0, out.stdout
    assert out.stdout.startswith("checked")
