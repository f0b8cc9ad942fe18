"""The loss head's work items (paper_2608_00029_amd/csrc/lmhead_sched.h) cover
every logit exactly once, for grids with and without a last partial round, and
an item cut from a tile is at most one per work group."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include <vector>
#include "lmhead_sched.h"
using namespace cattn;
int main() {
  int bad = 0;
  for (int per : {1, 5, 32})
    for (int n_vt : {1, 3, 8, 9, 40, 73})
      for (int n_mt : {1, 2, 5, 12}) {
        const int V = n_vt * 4, M = n_mt * 4;  // in units of 64 rows
        std::vector<int> seen(V * M, 0);
        for (int x = 0; x < kXcdGroup; ++x) {
          const int tiles = lmh_xcd_tiles(x, n_vt, n_mt), items = lmh_xcd_items(tiles, per);
          if (items - tiles / per * per > per) ++bad;
          for (int i = 0; i < items; ++i) {
            const LmhItem t = lmh_xcd_item(x, i, n_vt, n_mt, per);
            if (t.v_ext % 128 || t.m_ext % 64 || t.v0 % 128 || t.m0 % 64) ++bad;
            if (i < tiles / per * per && (t.v_ext != kLmhTileV || t.m_ext != kLmhTileM)) ++bad;
            for (int v = t.v0 / 64; v < (t.v0 + t.v_ext) / 64; ++v)
              for (int m = t.m0 / 64; m < (t.m0 + t.m_ext) / 64; ++m)
                if (v >= V || m >= M || ++seen[v * M + m] > 1) ++bad;
          }
        }
        for (int s : seen) bad += s != 1;
      }
  printf("bad=%d\n", bad);
  return bad != 0;
}
"""


def test_items_cover_every_logit_once(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "items.cpp", str(tmp_path / "items")
    src.write_text(CHECK)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2608_00029_amd", "csrc"), str(src),
                    "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and "bad=0" in out.stdout, out.stdout
