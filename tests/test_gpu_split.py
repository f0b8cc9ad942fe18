"""The bf16 attention kernels on either side of the rules that split a work
group's other axis into two or four parts, with parts that have one tile more
than others, parts without a tile, and ragged ends, and grids taken in groups of heads: every output of sampled
heads against the float64 oracle, with the tolerances and per-element bounds of
the parity tests."""

import pytest
import torch

from paper_2608_00029_amd.workloads import make_inputs
from parity_util import say
from test_gpu_parity import compare_all, gpu_fwd_bwd

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, S, D, causal
    (2, 16, 512, 64, True),    # 512 work groups in four parts (the most)
    (2, 12, 700, 64, True),    # 528: two parts, ragged
    (3, 3, 1057, 64, False),   # four parts, 34 tiles: uneven; last tile of one row
    (8, 10, 500, 64, False),   # forward in two parts, backward unsplit
    (8, 13, 480, 64, True),    # 832 work groups in two parts: unsplit
    (1, 8, 1000, 128, True),   # 256 in four parts (the most at D = 128), ragged
    (1, 9, 1000, 128, True),   # 288: two parts
    (2, 32, 500, 128, False),  # 512 in two parts (the most)
    (2, 33, 500, 128, True),   # unsplit, ragged
    (4, 12, 1000, 64, True),   # forward and dK/dV in two parts, dQ unsplit
    (2, 8, 1536, 64, True),    # four parts at three work groups per CU
    (16, 20, 60, 64, True),    # two tiles: unsplit, ragged
    (3, 40, 100, 128, False),  # four tiles, two parts, last tile of four rows
    (13, 16, 650, 64, True),   # 208 heads: three groups of 64 and one of 16, all kernels
    (12, 16, 300, 128, False),  # 192 heads, three tiles in little more than a round: over all heads
    (13, 16, 520, 128, True),  # 208 heads in groups at D = 128, all kernels
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_split_rules(cuda, case):
    B, H, S, D, causal = case
    q, k, v, do = make_inputs(B, H, S, D, "bf16", seed=40 + S + H)
    say(f"split {case}")
    scale = D ** -0.5
    got = gpu_fwd_bwd(q, k, v, do, scale, causal)
    for t in got:  # every element of every head written (the buffers started as NaN)
        assert torch.isfinite(t.float()).all()
    heads = sorted({(0, 0), (0, H - 1), (B - 1, 0), (B - 1, H - 1)})
    sel = lambda t: torch.stack([t[b, h] for b, h in heads])[None]  # noqa: E731
    compare_all("bf16", tuple(sel(t) for t in got), *(sel(t) for t in (q, k, v, do)), scale, causal)
