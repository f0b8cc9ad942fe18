"""grouped_rank (paper_2608_00029_amd/csrc/attn_sched.h) visits every (head,
rank) once, group by group of heads and rank by rank inside a group; work_order
picks it on the sides of its limits (256 CUs) where it measured faster."""

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
// heads per group: as few groups of at most 64 as it takes, of even size, a multiple of 8
static int even(int BH) {
  int n = 1;
  while (n * 64 < BH) ++n;
  int hg = 8;
  while (n * hg < BH) hg += 8;
  return hg;
}
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
  // pass, D, causal, heads, S, tiles, resident per CU: whether heads are grouped
  struct { Pass pass; int D; bool causal; int BH, S, nt, per_cu; bool grouped; } rules[] = {
      {Pass::kFwd, 128, true, 256, 1024, 8, 3, true},   {Pass::kFwd, 128, true, 191, 1024, 8, 3, false},
      {Pass::kFwd, 128, true, 256, 1025, 9, 3, false},  {Pass::kFwd, 64, true, 256, 512, 4, 4, false},
      {Pass::kFwd, 64, true, 257, 512, 4, 4, true},     {Pass::kFwd, 64, true, 1135, 24, 1, 4, false},
      {Pass::kDq, 128, true, 210, 384, 3, 2, false},    {Pass::kDq, 128, true, 300, 384, 3, 2, true},
      {Pass::kDq, 128, false, 340, 160, 2, 2, false},   {Pass::kDq, 128, false, 340, 192, 2, 2, true},
      {Pass::kDq, 128, false, 513, 160, 2, 2, true},    {Pass::kDq, 128, false, 250, 300, 3, 2, false},
      {Pass::kDkdv, 64, true, 340, 258, 3, 3, false},   {Pass::kDkdv, 128, true, 210, 300, 3, 2, false},
      {Pass::kDkdv, 128, true, 208, 392, 4, 2, false},  {Pass::kDkdv, 128, true, 300, 300, 3, 2, true},
      {Pass::kDq, 128, true, 323, 186, 2, 2, true},     {Pass::kDq, 64, false, 513, 256, 2, 4, true},
      {Pass::kDkdv, 128, true, 323, 186, 2, 2, false},  {Pass::kDkdv, 128, true, 513, 186, 2, 2, true},
      {Pass::kDkdv, 128, true, 323, 300, 3, 2, true},    {Pass::kDkdv, 64, true, 768, 160, 2, 3, false},
      {Pass::kDkdv, 64, true, 942, 140, 2, 3, false},   {Pass::kDkdv, 64, false, 400, 256, 2, 3, true},
      {Pass::kDkdv, 128, false, 400, 1024, 8, 2, false}};
  for (auto& r : rules)
    for (int otherwise : {0, 256})
      if (work_order(r.pass, r.D, r.causal, r.BH, r.S, r.nt, r.per_cu, 256, otherwise) !=
          (r.grouped ? -even(r.BH) : otherwise))
        ++bad;
  if (even(192) != 64 || even(208) != 56 || even(257) != 56 || even(330) != 56 || even(513) != 64) ++bad;
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
