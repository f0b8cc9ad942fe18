"""grouped_rank (paper_2608_00029_amd/csrc/attn_sched.h) visits every (head,
rank) once, group by group of heads and rank by rank inside a group."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include <vector>
#include "attn_sched.h"
using namespace cattn;
int main() {
  int bad = 0;
  for (int BH : {1, 7, 64, 65, 192, 400})
    for (int nt : {1, 3, 8})
      for (int hg : {1, 8, 64, 1000}) {
        std::vector<int> seen(BH * nt, 0);
        int last_group = 0, last_rank = 0;
        for (int b = 0; b < BH * nt; ++b) {
          const HeadRank r = grouped_rank(b, BH, nt, hg);
          if (r.bh < 0 || r.bh >= BH || r.rank < 0 || r.rank >= nt) { ++bad; continue; }
          ++seen[r.bh * nt + r.rank];
          const int g = r.bh / hg;
          if (g < last_group || (g == last_group && r.rank < last_rank)) ++bad;
          last_group = g;
          last_rank = r.rank;
        }
        for (int s : seen) bad += s != 1;
      }
  printf("bad=%d\n", bad);
  return bad != 0;
}
"""


def test_grouped_rank_is_an_ordered_permutation(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "groups.cpp", str(tmp_path / "groups")
    src.write_text(CHECK)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2608_00029_amd", "csrc"), str(src),
                    "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and "bad=0" in out.stdout, out.stdout
