"""The loss head's work items (paper_2608_00029_amd/csrc/lmhead_sched.h) cover
every logit exactly once, for grids with and without a last partial round, and
an item cut from a tile is at most one per work group.  The built kernel holds
the stores per tile that its waits count on."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_00029_amd.binding import library_path
from test_residency import _code_objects

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


def test_stores_per_tile(tmp_path):
    """While a tile's stores drain, a wave waits for its oldest copies by letting
    4 + 34 younger operations be in flight: with fewer than 34 stores in the
    built kernel it would read a chunk that has not landed."""
    objdump = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
    if objdump is None:
        pytest.skip("llvm-objdump not found")
    with open(library_path(), "rb") as f:
        blob = f.read()
    found = 0
    for i, elf in enumerate(_code_objects(blob)):
        if b"lmhead_logits_stats_kernel" not in elf:
            continue
        path = tmp_path / f"{i}.elf"
        path.write_bytes(elf)
        text = subprocess.run([objdump, "-d", str(path)], capture_output=True, text=True, check=True).stdout
        body = re.search(r"<\S*lmhead_logits_stats_kernel\S*>:\n(.*?)(\n\n|\Z)", text, re.S)[1]
        assert len(re.findall(r"\bglobal_store_dwordx4\b", body)) == 32
        assert len(re.findall(r"\bglobal_store_dwordx2\b", body)) == 2
        assert not re.search(r"\b(scratch|buffer|flat)_", body)
        found += 1
    assert found == 1
