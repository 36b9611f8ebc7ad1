"""Blocks of a launch -> tiles of its problems (csrc/tile_map.h), compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "tile_map.h"
int main() {                                  // per launch: number of problems, their tile counts -> "problem tile xcd" per working block
  int n;
  while (std::scanf("%d", &n) == 1) {
    struct { int n; struct { int tiles, tile_start; } p[64]; } a;
    a.n = n;
    int rows = 0;
    for (int i = 0; i < n; ++i) {
      if (std::scanf("%d", &a.p[i].tiles) != 1) return 1;
      a.p[i].tile_start = rows;
      rows += sna::tile_rows(a.p[i].tiles);
    }
    const int blocks = sna::launch_blocks(a);
    if (blocks > rows * sna::kXcds) return 2;
    bool ended[sna::kXcds] = {};
    for (int b = 0; b < blocks; ++b) {
      const sna::TilePlace at = sna::place_of_block(a, b);
      if (n == 1 && at.tile != sna::tile_of_block(a.p[0].tiles, a.p[0].tile_start, b)) return 3;
      if (at.tile < 0) ended[b % sna::kXcds] = true;
      else if (ended[b % sna::kXcds]) return 4;         // a block without a tile ahead of one with
      else std::printf("%d %d %d\n", at.problem, at.tile, b % sna::kXcds);
    }
    std::printf("end\n");
  }
}
"""


@pytest.mark.parametrize("launches", [[[t] for t in list(range(1, 42)) + [255, 256, 257, 9408, 200000]],
                                      [[1] * 16, [7, 8, 9], [84, 84, 84], [3, 1568, 1, 17, 64, 5, 2, 31], list(range(1, 33))]])
def test_every_tile_once_and_evenly_over_xcds(tmp_path, launches):
    (tmp_path / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2312_16733_amd", "csrc"),
                    str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver")], check=True)
    text = "\n".join(f"{len(l)} " + " ".join(map(str, l)) for l in launches) + "\n"
    out = subprocess.run([str(tmp_path / "driver")], input=text, capture_output=True, text=True, check=True).stdout.split("end\n")
    assert len(out) == len(launches) + 1
    for tiles, lines in zip(launches, out):
        got = [tuple(map(int, l.split())) for l in lines.split("\n") if l]
        assert sorted((g, t) for g, t, _ in got) == [(g, t) for g, n in enumerate(tiles) for t in range(n)]
        for g, n in enumerate(tiles):
            per = [[t for p, t, x in got if p == g and x == xcd] for xcd in range(8)]
            assert max(map(len, per)) - min(map(len, per)) <= 1
            assert all(p == list(range(p[0], p[0] + len(p))) for p in per if p)         # consecutive tiles share an XCD
