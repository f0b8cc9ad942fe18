"""The loss head at the edges of its copy ring and of the merge: work groups
that walk several tiles with only two chunks of K per tile (stores of one tile
in flight over all chunks of the next), waves past the end of a ragged last
tile among them, tiles cut into parts for the last round, work groups with more
items than they look up at once, and rows of more and of exactly as many
partials as the merge holds in registers.  Every output of sampled rows against the float64 oracle,
with the bounds of the loss-head tests; every logit finite."""

import numpy as np
import pytest
import torch

from paper_2608_00029_amd.workloads import make_lmhead_inputs
from parity_util import say
from test_gpu_lmhead import DEV, check_rows, run

pytestmark = pytest.mark.gpu

CASES = [
    # M, N, K
    (1152, 18560, 64),    # 73 x 5 tiles, the last of each axis half empty
    (2048, 18432, 64),    # 72 x 8 tiles: two or three per work group
    (1152, 18560, 192),   # six chunks per tile
    (128, 65536, 64),     # 1024 partials per row
    (128, 65664, 128),    # 1026
    (384, 9088, 128),     # 36 x 2 tiles, all cut: parts past both ends
    (1024, 17536, 64),    # 69 x 4 tiles: whole ones, then cut ones, on the chiplets with nine
    (32512, 33024, 64),   # 129 x 127 tiles: up to 68 items a work group (64 looked up at once), the last cut
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_ring_and_merge_edges(case):
    M, N, K = case
    x, w, y = make_lmhead_inputs(M, N, K, 0.3, seed=17 + M + N + K)
    say(f"lmhead edges M{M} N{N} K{K}")
    z, lse, rl, loss, part = run(x, w, y)
    assert torch.isfinite(z).all() and torch.isfinite(part).all()
    g = np.random.default_rng(3)
    rows = np.unique(np.concatenate([[0, 127, M - 128, M - 1], g.choice(M, 20, replace=False)]))
    ri = torch.as_tensor(rows)
    rep = check_rows(rows, x, w, y, z[ri.to(DEV)].cpu(), lse.cpu()[ri], rl.cpu()[ri], part[ri.to(DEV)].cpu(), N)
    l64 = rl.cpu().double().mean().item()
    assert abs(loss.item() - l64) <= 1e-6 * abs(l64) + 1e-7
    print("  " + rep, flush=True)
