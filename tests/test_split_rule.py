"""The rule that splits a bf16 work group's other axis into parts (split_parts in
paper_2608_00029_amd/csrc/attn_sched.h), compiled with the host C++ compiler:
it takes the form that measured faster on either side of each of its limits (256
CUs), never gives a part no tile to run, and knows only 1, 2 and 4 parts."""

import os
import shutil
import subprocess

import pytest

from test_gpu_noclamp import CASES as NOCLAMP_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "attn_sched.h"
int main() {
  int pass, D, causal, BH, S;
  while (std::scanf("%d %d %d %d %d", &pass, &D, &causal, &BH, &S) == 5)
    std::printf("%d\n", cattn::split_parts((cattn::Pass)pass, D, causal != 0, BH, S, 256));
}
"""
FWD, DQ, DKDV = 0, 1, 2

# (D, causal, BH, S): parts of the forward, dQ, dK/dV that measured fastest (within 3%)
MEASURED = {
    # one or two tiles: nothing to share, however small the grid
    (64, True, 512, 32): (1, 1, 1), (64, False, 64, 64): (1, 1, 1), (128, True, 128, 64): (1, 1, 1),
    (128, True, 256, 25): (1, 1, 1),
    # short sequences: four parts only while each CU has one work group of 32 rows
    (64, True, 64, 128): (4, 4, 4), (64, True, 128, 128): (2, 2, 2), (128, True, 64, 128): (4, 4, 4),
    (128, True, 128, 128): (2, 2, 2), (64, True, 192, 100): (1, 1, 1), (128, True, 256, 100): (2, 1, 1),
    # two work groups of 32 rows per CU
    (64, False, 64, 256): (2, 2, 2), (64, True, 32, 512): (4, 4, 4), (64, False, 32, 512): (4, 2, 2),
    (64, False, 16, 1024): (4, 4, 4), (64, True, 32, 384): (4, 2, 4), (64, False, 56, 288): (2, 2, 2),
    (64, True, 89, 224): (2, 1, 2), (64, True, 84, 224): (2, 1, 2), (64, True, 105, 154): (1, 1, 2),
    (64, True, 133, 154): (1, 1, 1), (64, False, 64, 261): (2, 1, 2), (64, False, 149, 187): (2, 1, 2),
    (64, False, 57, 272): (2, 1, 2), (64, True, 36, 1142): (2, 2, 2), (64, False, 72, 371): (2, 1, 2), (64, False, 81, 352): (2, 1, 1), (64, True, 48, 384): (2, 2, 2), (64, True, 68, 450): (2, 1, 2),
    (64, True, 40, 777): (2, 2, 2), (64, True, 49, 650): (2, 2, 2),
    # long causal sequences: more parts, on larger grids
    (64, True, 6, 4096): (4, 4, 4), (64, True, 12, 2048): (4, 4, 4), (64, False, 12, 2048): (2, 2, 2),
    (64, True, 12, 4096): (2, 2, 2), (64, True, 24, 2048): (2, 2, 2), (64, True, 40, 1024): (2, 2, 2),
    (64, True, 14, 4096): (2, 2, 2), (64, True, 18, 4096): (2, 1, 1), (64, False, 28, 2048): (1, 1, 1),
    (64, False, 40, 1568): (2, 1, 1), (64, True, 22, 2264): (2, 2, 2), (64, True, 18, 2855): (2, 2, 2),
    (64, True, 31, 1659): (2, 1, 2),
    (64, True, 56, 1024): (2, 1, 1),
    # head dimension 128
    (128, True, 152, 160): (2, 1, 1),
    (128, True, 16, 2048): (2, 2, 2), (128, False, 16, 2040): (2, 2, 2), (128, False, 96, 256): (1, 1, 1),
    (128, False, 20, 2048): (1, 1, 1),
    # the headline and the long-context training shapes
    (64, True, 96, 1024): (1, 1, 1), (128, True, 32, 4096): (1, 1, 1),
}


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("split")
    src, exe = d / "split.cpp", str(d / "split")
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2608_00029_amd", "csrc"), str(src),
                    "-o", exe], check=True)

    def ask(shapes):
        text = "".join("%d %d %d %d %d\n" % s for s in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        assert len(out) == len(shapes)
        return [int(x) for x in out]

    return ask


def test_measured_limits(parts):
    shapes = [(p, D, int(c), BH, S) for D, c, BH, S in MEASURED for p in (FWD, DQ, DKDV)]
    want = [w for row in MEASURED.values() for w in row]
    wrong = [(s, g, w) for s, g, w in zip(shapes, parts(shapes), want) if g != w]
    assert not wrong, wrong


def test_noclamp_cases_reach_every_form(parts):
    """The comparison with the unclamped build runs every number of parts at both
    head dimensions, with whole and with ragged tiles, in all three kernels."""
    shapes = [(p, D, 1, B * H, S) for B, H, S, D, _ in NOCLAMP_CASES for p in (FWD, DQ, DKDV)]
    got = parts(shapes)
    assert all(len(set(got[i:i + 3])) == 1 for i in range(0, len(got), 3))
    reached = {(D, n, S % 32 == 0) for (_, D, _, _, S), n in zip(shapes, got)}
    assert reached == {(D, n, whole) for D in (64, 128) for n in (1, 2, 4) for whole in (True, False)}


def test_range(parts):
    shapes = [(p, D, c, BH, S) for p in (FWD, DQ, DKDV) for D in (64, 128) for c in (0, 1)
              for BH in (1, 7, 64, 200, 3000, 2000000) for S in (1, 31, 32, 33, 64, 65, 96, 97, 128, 500, 2048, 8192)]
    for (_, D, _, BH, S), n in zip(shapes, parts(shapes)):
        nt = (S + 31) // 32
        assert n in (1, 2, 4)
        assert n <= nt + 1  # no more than one part of a sequence's last tiles goes without
        assert n == 1 or nt >= 3
        if n == 4:  # a CU's share of 32-row work groups stays small
            assert BH * nt <= (3 if D == 64 else 1) * 256
