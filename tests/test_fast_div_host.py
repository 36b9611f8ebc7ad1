"""Division by a known number (csrc/fast_div.h), compiled for the host, against the / operator."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include <random>
#include "fast_div.h"
static long bad = 0, n = 0;
static void check(int64_t x, int64_t d) {
  if (d < 1 || d > INT32_MAX || x < 0 || x > INT32_MAX) return;
  ++n;
  if (sna::FastDiv::by((int)d).div((int)x) != (int)(x / d)) {
    if (!bad++) std::printf("%ld / %ld\n", (long)x, (long)d);
  }
}
int main() {
  for (int64_t d = 1; d <= 2048; ++d)                            // every small divisor around its multiples at both ends
    for (int64_t k : {int64_t(0), int64_t(1), int64_t(2), INT32_MAX / d - 1, INT32_MAX / d})
      for (int e = -1; e <= 1; ++e) check(k * d + e, d);
  for (int p = 0; p < 31; ++p)                                   // divisors around the powers of two
    for (int64_t d = (1ll << p) - 2; d <= (1ll << p) + 2; ++d)
      for (int q = 0; q <= 31; ++q)
        for (int e = -2; e <= 2; ++e) {
          check((1ll << q) + e, d);
          if (d > 0) check((1ll << q) / d * d + e, d);
        }
  std::mt19937_64 rng(1);
  for (int i = 0; i < 2000000; ++i) {
    const int64_t d = (rng() >> (33 + rng() % 31)) + 1;
    check(rng() >> 33, d);
    check((rng() >> 33) / d * d - 1, d);                         // the last of a quotient
  }
  std::printf("%ld wrong of %ld\n", bad, n);
  return bad != 0 || n < 4000000;
}
"""


def test_every_quotient_is_the_operators(tmp_path):
    (tmp_path / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2312_16733_amd", "csrc"), str(tmp_path / "d.cpp"),
                    "-o", str(tmp_path / "d")], check=True)
    r = subprocess.run([str(tmp_path / "d")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
