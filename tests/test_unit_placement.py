"""The rule that places query tiles on workgroups (place() of csrc/amskv_internal.hpp, the same code the kernels run) built for the CPU:
every tile of every (b,h) exactly once; whole (b,h) per XCD up to the last multiple of eight, and beyond it while no XCD has more than a
given number of tiles; else XCDs with equal numbers of them; and the form without left-over units where there are none."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "amskv_internal.hpp"
using namespace amskv;
static void check(bool ok, const char* what, int n, int t) {
  if (!ok) { std::printf("%s: %d units, %d tiles\n", what, n, t); std::exit(1); }
}
int main() {
  const int tiles[] = {1, 2, 3, 5, 7, 8, 9, 13, 32, 79};
  for (int most : {0, 8, 24, 32})
  for (int n = 1; n <= 130; ++n)
    for (int t : tiles) {
      const bool few = (n + 7) / 8 * t <= most, even = n % 8 == 0 || t == 1;
      const int whole = whole_units(n, t, most);
      check((whole < n) == !(few || even) && whole % 8 == 0, "the rule", n, t);
      std::vector<int> seen(n * t, 0), per_xcd(8, 0);
      for (unsigned id = 0; id < placed_grid(n, t, whole); ++id) {
        const Place p = whole < n ? place<true>(id, n, t, whole) : place<false>(id, n, t, whole);
        check(p.bh >= 0 && p.tile >= 0 && p.tile < t, "in range", n, t);
        if (p.bh >= n) continue;
        ++seen[p.bh * t + p.tile];
        ++per_xcd[id & 7];
        check((p.bh >= (n & ~7) && !few) || (p.bh & 7) == (int)(id & 7), "whole units on one XCD", n, t);
        if (whole >= n) {
          const Place q = place<true>(id, n, t, whole);
          check(q.bh == p.bh && q.tile == p.tile, "both forms agree", n, t);
        }
      }
      for (int x : seen) check(x == 1, "every tile once", n, t);
      int lo = n * t, hi = 0;
      for (int x : per_xcd) lo = x < lo ? x : lo, hi = x > hi ? x : hi;
      check(hi - lo <= (few ? t : 1), "equal shares", n, t);
    }
  std::puts("all placed");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_tile_once_and_xcds_even(tmp_path):
    src, exe = str(tmp_path / "placement.cpp"), str(tmp_path / "placement")
    with open(src, "w") as f:
        f.write(PROGRAM)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2511_16047_amd", "csrc"),
                        src, "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert b.returncode == 0, b.stdout[-4000:]
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0 and "all placed" in r.stdout, r.stdout[-4000:]
