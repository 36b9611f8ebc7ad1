"""The tile choice of a launch (csrc/tile_choice.h, plain host code) against its formula written out problem by problem
and variant by variant, and the host time it takes: it is asked for every layer slot of a launch list built anew."""
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "tile_choice.h"
#include <chrono>
#include <cstdio>
#include <vector>
using namespace sna;
int main() {
  int nv = 0, v, bm, bn, steps;
  if (scanf("%d", &nv) != 1) return 1;
  std::vector<TileShape> shapes(64, TileShape{32, 32, 0});
  for (int i = 0; i < nv; ++i) {
    if (scanf("%d %d %d %d", &v, &bm, &bn, &steps) != 4) return 1;
    shapes[v] = {bm, bn, steps};
  }
  for (const TileCost& c : kTileCosts) printf("%d %.9g %.9g %.9g %.9g %.9g\n", c.variant, c.launch, c.block, c.step, c.step_taps, c.walk);
  int n, mode;
  while (scanf("%d %d", &n, &mode) == 2) {
    std::vector<TileWork> ws(n);
    for (TileWork& w : ws)
      if (scanf("%d %d %d %d", &w.M, &w.K, &w.kt, &w.taps) != 4) return 1;
    const TileChoice c = pick_tile(ws.data(), ws.size(), mode, shapes.data());
    double best = 1e9;
    volatile int sink = 0;
    for (int t = 0; t < 20; ++t) {
      const auto t0 = std::chrono::steady_clock::now();
      for (int k = 0; k < 10; ++k) sink = sink + pick_tile(ws.data(), ws.size(), mode, shapes.data()).variant;
      const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() / 10 * 1e6;
      if (us < best) best = us;
    }
    printf("%d %d %.4f\n", c.variant, (int)c.split, best);
  }
}
"""
# variant -> (tile rows, tile columns, most K steps one block walks)
SHAPES = {28: (32, 32, 128), 29: (64, 64, 128), 30: (128, 96, 128), 4: (64, 64, 1 << 30), 27: (64, 64, 1 << 30),
          25: (64, 128, 1 << 30), 1: (128, 64, 1 << 30), 2: (128, 96, 1 << 30), 8: (64, 128, 1 << 30),
          9: (128, 64, 1 << 30), 11: (128, 128, 1 << 30), 22: (128, 128, 1 << 30), 12: (128, 32, 1 << 30),
          24: (128, 96, 1 << 30)}


def chunk_steps(kt):
    n = 1 if kt <= 24 else (2 if kt <= 64 else 4)
    return -(-kt // n)


def expected_us(cost, problems, split):
    """The formula of tile_choice.h for one variant and one layout; None where a block would walk too many steps."""
    variant, launch, block, step, step_taps, walk = cost
    bm, bn, max_steps = SHAPES[variant]
    blocks = work = sums_mb = 0.0
    for m, k, kt, taps in problems:
        per = chunk_steps(kt)
        parts = -(-kt // per) if split else 1
        steps = per if parts > 1 else kt
        if steps > max_steps:
            return None
        if parts > 1:
            sums_mb += 4e-6 * parts * m * k
        b = -(-m // bm) * -(-k // bn) * parts
        blocks += b
        work += b * steps * ((step_taps if taps > 1 else step) + (walk if parts == 1 and per < kt else 0.0))
    per_cu = blocks / 256
    if per_cu < 4:
        per_cu = float(np.ceil(per_cu))
    return launch + per_cu * (block + work / blocks) + (1.9 + 1.6 * sums_mb if sums_mb > 0 else 0.0)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_choice")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O3", "-std=c++17", "-I", os.path.join(ROOT, "paper_2312_16733_amd", "csrc"),
                    str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)

    def ask(launches):
        text = [str(len(SHAPES))] + [f"{v} {bm} {bn} {st}" for v, (bm, bn, st) in SHAPES.items()]
        for mode, problems in launches:
            text.append(f"{len(problems)} {mode}")
            text += [" ".join(map(str, p)) for p in problems]
        out = subprocess.run([str(d / "driver")], input="\n".join(text) + "\n", capture_output=True, text=True, check=True).stdout
        lines = [l.split() for l in out.strip().split("\n")]
        costs = [(int(l[0]),) + tuple(float(x) for x in l[1:]) for l in lines if len(l) == 6]
        return costs, [(int(l[0]), int(l[1]), float(l[2])) for l in lines if len(l) == 3]
    return ask


def random_launch(rng, n):
    problems = []
    for _ in range(n):
        taps = rng.choice([1, 9])
        c = 8 * rng.randrange(1, 1100 if rng.random() < 0.2 else 260)
        m = rng.randrange(1, 200000 if rng.random() < 0.3 else 4000)
        problems.append((m, 8 * rng.randrange(1, 260), -(-taps * c // 64), taps))
    return problems


def test_choice_is_the_formulas_minimum(driver):
    rng = random.Random(11)
    launches = [(rng.randrange(4), random_launch(rng, rng.choice([1, 1, 2, 5, 16, 32]))) for _ in range(400)]
    costs, got = driver(launches)
    assert sorted(c[0] for c in costs) == sorted(SHAPES) and len(got) == len(launches)
    for (mode, problems), (variant, split, _) in zip(launches, got):
        layouts = [0] if mode == 1 else ([1] if mode >= 2 else [0, 1])
        times = {(c[0], s): expected_us(c, problems, s) for c in costs for s in layouts}
        least = min(t for t in times.values() if t is not None)
        assert split in layouts and times[(variant, split)] is not None
        assert times[(variant, split)] <= least * (1 + 1e-6), (mode, problems)      # fp32 constants; equal times are ties
        if mode == 0 and all(chunk_steps(p[2]) == p[2] for p in problems):
            assert split == 0                                                       # nothing to spread


def test_choice_for_a_mixed_launch_takes_little_host_time(driver):
    """Some fifty slots a list, two launches of host work each already: a choice must not cost more than a launch's
    submission (2.4 us).  Walking fourteen variants twice over sixteen descriptors took 4 to 8."""
    _, got = driver([(0, [(3136 + i, 720 - 8 * i, -(-9 * (90 - i) // 8), 9) for i in range(16)])])
    assert got[0][2] < 2.4, got


TUNE_DRIVER = r"""
#include "tile_choice.h"
#include <cstdio>
int main() {                                  // variants, the variant without an entry; per variant: launches, number of sums, the sums
  int nv, without;
  while (scanf("%d %d", &nv, &without) == 2) {
    std::vector<sna::TuneSample> s(nv);
    for (auto& v : s) {
      int n;
      if (scanf("%d %d", &v.launches, &n) != 2) return 1;
      v.ms.resize(n);
      for (double& t : v.ms)
        if (scanf("%lf", &t) != 1) return 1;
    }
    printf("%d\n", sna::measured_variant(s, without));
  }
}
"""


def test_tuner_compares_variants_over_the_same_launches(tmp_path):
    """A shape that two launches of a forward share, one of which only some variants can run: a variant's sum over one
    launch is no better for being smaller."""
    (tmp_path / "d.cpp").write_text(TUNE_DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2312_16733_amd", "csrc"), str(tmp_path / "d.cpp"),
                    "-o", str(tmp_path / "d")], check=True)
    calls = [  # (variant without an entry, [(launches, sums)]) -> variant
        ((0, [(2, [10, 11, 12]), (1, [5, 5, 5]), (2, [9, 9, 9])]), 2),            # variant 1 ran on one launch only
        ((0, [(2, [10, 11, 12]), (1, [5, 5, 5]), (2, [11, 10.9, 10.9])]), 0),     # and 0.9 % are noise
        ((1, [(2, [10, 10, 10]), (1, [5, 5, 5]), (2, [9, 9, 9])]), 2),            # the one without an entry ran on one only
        ((1, [(1, [10, 10, 10]), (1, [9, 9, 50]), (0, [])]), 1),                  # medians; nothing measured for variant 2
        ((2, [(1, [10, 10, 10]), (1, [9, 9, 9]), (0, [])]), 1),
        ((2, [(0, []), (0, []), (0, [])]), 2),
    ]
    text = "\n".join(f"{len(v)} {w} " + " ".join(f"{n} {len(t)} " + " ".join(map(str, t)) for n, t in v) for (w, v), _ in calls)
    out = subprocess.run([str(tmp_path / "d")], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert [int(o) for o in out] == [want for _, want in calls]
