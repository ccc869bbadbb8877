"""The workgroup mapping of the (point, slot) launches (csrc/xcd_map.h) on the host: every item has exactly one
block, and a launch of points_per_launch points stays below the 2^32 threads of a grid dimension."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_22718_amd", "csrc")

PROGRAM = r"""
#include "xcd_map.h"
#include <stdio.h>
#include <vector>
int main() {
  for (int points = 1; points <= 140; ++points)
    for (int slots : {1, 2, 3, 7, 8, 12, 103}) {
      std::vector<int> seen((size_t)points * slots, 0);
      const unsigned n = xcd_blocks(points, slots);
      for (unsigned j = 0; j < n; ++j) {
        int p = -1, s = -1;
        xcd_item((int)j, points, slots, &p, &s);
        if (p < 0 || s < 0 || s >= slots) { printf("item (%d, %d) of %d x %d\n", p, s, points, slots); return 1; }
        if (p < points) seen[(size_t)p * slots + s]++;
      }
      for (int v : seen)
        if (v != 1) { printf("an item with %d blocks: %d x %d\n", v, points, slots); return 1; }
    }
  for (int threads : {256, 512, 1024})
    for (int slots = 1; slots <= 1000000; slots += 1 + slots / 50) {
      const int most = points_per_launch(slots, threads);
      if (most < 1) return 1;
      const size_t all = (size_t)1 << 32;
      for (int d : {0, 1, 5, 8, 9}) {
        const int points = most - d;
        if (points >= 1 && (size_t)xcd_blocks(points, slots) * threads >= all) { printf("%d x %d of %d threads\n", points, slots, threads); return 1; }
      }
      // and not needlessly small: 16 more points would not fit
      if (most < 0x7ffffff8 && ((size_t)most + 16) * slots * threads < all) { printf("only %d x %d\n", most, slots); return 1; }
    }
  printf("ok\n");
  return 0;
}
"""


def test_every_item_once_and_launches_below_the_grid_limit(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src = tmp_path / "map.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "map"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
