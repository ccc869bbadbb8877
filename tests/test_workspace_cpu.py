"""Chunk sizes of a plan's workspace for the memory that is free (csrc/workspace.h), on the host: the full sizes
where there is plenty, never less than the plan needs, the optional part within half of what is free, and more
memory never gives smaller chunks."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_22718_amd", "csrc")

PROGRAM = r"""
#include "workspace.h"
#include <stdio.h>
#include <stdlib.h>
int main() {
  srand(7);
  for (int trial = 0; trial < 20000; ++trial) {
    workspace_request r{};
    r.vbuf_point = 256 + (size_t)rand() % 60000000;
    r.base = 1 + rand() % 40;
    r.adjoint = r.base + rand() % 100;
    if (rand() % 2) {
      r.growth_point = 1000 + (size_t)rand() % 40000000;
      r.growth = 1 + rand() % 200;
    }
    const size_t need = r.base * r.vbuf_point;
    workspace_points last{0, 0, 0};
    for (size_t f = 0; f <= (size_t)96 << 30; f = f ? f + f / 3 + 1 : 1 << 20) {
      const workspace_points w = workspace_fit(r, f);
      if (w.adjoint < r.base || w.adjoint > r.adjoint) { printf("adjoint %d\n", w.adjoint); return 1; }
      if (r.growth ? w.growth < 1 || w.growth > r.growth : w.growth != 0) { printf("growth %d\n", w.growth); return 1; }
      if (w.vbuf < w.adjoint || w.vbuf < w.growth || w.vbuf < r.base) { printf("rows %d\n", w.vbuf); return 1; }
      if (w.vbuf > w.adjoint && w.vbuf > w.growth) { printf("spare rows %d\n", w.vbuf); return 1; }
      const size_t bytes = w.vbuf * r.vbuf_point + w.growth * r.growth_point;
      const bool least = w.vbuf == r.base && w.growth <= 1;
      if (!least && bytes > f / 2) { printf("%zu of %zu free\n", bytes, f); return 1; }
      if (w.growth < last.growth) { printf("growth %d after %d\n", w.growth, last.growth); return 1; }
      last = w;
      const int big = r.growth > r.adjoint ? r.growth : r.adjoint;
      if (f / 2 >= big * r.vbuf_point + r.growth * r.growth_point && (w.adjoint != r.adjoint || w.growth != r.growth)) {
        printf("not full\n");
        return 1;
      }
    }
    const workspace_points z = workspace_fit(r, 0);
    if (z.vbuf * r.vbuf_point != need || z.growth != (r.growth ? 1 : 0)) { printf("nothing free\n"); return 1; }
  }
  printf("ok\n");
  return 0;
}
"""


def test_chunks_for_the_free_memory(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src = tmp_path / "fit.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "fit"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
