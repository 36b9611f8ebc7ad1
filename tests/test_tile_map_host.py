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
    int tiles[64], start[64], rows = 0;
    for (int i = 0; i < n; ++i) {
      if (std::scanf("%d", &tiles[i]) != 1) return 1;
      start[i] = rows;
      rows += sna::tile_rows(tiles[i]);
    }
    for (int b = 0; b < rows * sna::kXcds; ++b) {
      int g = 0;
      for (int i = 1; i < n; ++i)
        if ((b >> 3) >= start[i]) g = i;      // the kernels' find_problem
      const int t = sna::tile_of_block(tiles[g], start[g], b);
      if (t >= 0) std::printf("%d %d %d\n", g, t, b % sna::kXcds);
    }
    std::printf("end\n");
  }
}
"""


@pytest.mark.parametrize("launches", [[[t] for t in list(range(1, 42)) + [255, 256, 257, 9408, 200000]],
                                      [[1] * 16, [7, 8, 9], [3, 1568, 1, 17, 64, 5, 2, 31], list(range(1, 33))]])
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
