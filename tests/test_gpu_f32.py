"""The float32 kernels at the edges of their work split, against the float64
oracle: work groups of one row group in four parts and of two in two (short
sequences on large grids), parts with no tile, with one more tile than others,
and a last tile of one row, in both storage orders.  Tolerance: the float32
acceptance bar (max abs 1e-5)."""

import pytest
import torch

import oracle.attn_oracle as orc
from paper_2608_00029_amd import attn_bwd, attn_fwd
from paper_2608_00029_amd.workloads import make_inputs
from parity_util import check_tensor, say

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # B, H, S, D, causal, layout
    (64, 8, 33, 64, True, "bhsd"),     # two row groups, the second of one row
    (64, 8, 64, 128, False, "bshd"),   # two row groups, one tile per part
    (32, 16, 97, 64, False, "bshd"),   # two row groups, parts of two tiles; the last work group half empty
    (16, 16, 256, 128, True, "bhsd"),  # two row groups, the longest sequence
    (16, 16, 257, 64, True, "bhsd"),   # one row group, just past it
    (1, 3, 161, 128, True, "bshd"),    # one row group, six tiles over four parts, last tile of one row
    (1, 1, 96, 64, False, "bhsd"),     # one row group, a part without a tile
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_work_split_edges(cuda, case):
    B, H, S, D, causal, layout = case
    q, k, v, do = make_inputs(B, H, S, D, "f32", seed=60 + S + D)
    say(f"f32 split {case}")
    perm = (lambda t: t) if layout == "bhsd" else (lambda t: t.transpose(1, 2).contiguous())
    qd, kd, vd, dod = (perm(t.to(DEV)) for t in (q, k, v, do))
    o, dq, dk, dv = (torch.full_like(qd, float("nan")) for _ in range(4))
    lse = torch.full((B, H, S), float("nan"), dtype=torch.float32, device=DEV)
    scale = D ** -0.5
    attn_fwd(qd, kd, vd, scale, causal, o=o, lse=lse, layout=layout)
    attn_bwd(qd, kd, vd, o, dod, lse, scale, causal, dq=dq, dk=dk, dv=dv, layout=layout)
    torch.cuda.synchronize()
    for t in (o, lse, dq, dk, dv):
        assert torch.isfinite(t).all()
    heads = sorted({(0, 0), (0, H - 1), (B - 1, 0), (B - 1, H - 1), (B // 2, H // 2)})
    sel = lambda t: torch.stack([t[b, h] for b, h in heads])[None]  # noqa: E731
    qs, ks, vs, dos = (sel(t) for t in (q, k, v, do))
    ro, rlse = orc.attn_fwd(qs, ks, vs, scale, causal)
    rdq, rdk, rdv = orc.attn_bwd(qs, ks, vs, dos, scale, causal)
    for n, g, r in (("o", o, ro), ("dq", dq, rdq), ("dk", dk, rdk), ("dv", dv, rdv)):
        check_tensor(n, "f32", sel(perm(g).cpu()), r)
    check_tensor("lse", "f32", sel(lse.cpu()), rlse)
