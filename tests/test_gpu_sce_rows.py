"""Cross-entropy forward on either side of the rule that gives a few long rows
16 waves each, against the float64 oracle with the tolerances of the
memory-bound operator tests; and rows with vocabulary entries masked by -inf,
where a lane may meet no finite logit at first, or at all."""

import numpy as np
import pytest
import torch

import oracle.memops_oracle as mo
from paper_2608_00029_amd import binding as b
from paper_2608_00029_amd.workloads import make_sce_inputs
from parity_util import say
from test_gpu_memops import _check_sce_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,V", [(1, 16384), (256, 16384), (257, 16384), (256, 16380), (3, 50304), (2, 16388),
                                    (1, 12288), (1, 12292), (256, 12288), (256, 12292), (257, 12292)])
def test_sce_row_rule(cuda, rows, V):
    z, t = make_sce_inputs(rows, V, seed=rows + V, sigma=3.0)
    say(f"sce rows={rows} V={V}")
    zd, td = z.to(cuda), t.to(cuda)
    scale = 1.0 / rows
    lse, rl, loss = b.sce_fwd(zd, td)
    dz = b.sce_bwd(zd, td, lse, scale)
    _check_sce_rows(z, t, lse, rl, dz, np.arange(rows), scale)
    assert abs(loss.item() - rl.cpu().double().mean().item()) <= 1e-6 * abs(loss.item()) + 1e-7


# Ranges masked with -inf, in entries: the first four-entry pieces of every lane
# past the first 256 (one load of each with 16 waves), of every lane, all but
# 12 entries, a stride that leaves one entry in four.
MASKS = {
    "1024:4096": [slice(1024, 4096)],
    "0:4096": [slice(0, 4096)],
    "all but 12": [slice(0, 7000), slice(7012, None)],
    "three of four": [slice(0, None, 4), slice(1, None, 4), slice(2, None, 4)],
}


@pytest.mark.parametrize("rows,V", [(2, 16384), (3, 50304), (300, 16384), (2, 8192)])
@pytest.mark.parametrize("mask", MASKS)
def test_sce_masked_entries(cuda, rows, V, mask):
    z, t = make_sce_inputs(rows, V, seed=rows + V, sigma=3.0)
    say(f"sce rows={rows} V={V} -inf at {mask}")
    e = 1e-5 + 6e-7 * z.abs().amax(dim=1).double().numpy()
    for sl in MASKS[mask]:
        z[:, sl] = float("-inf")
    finite = torch.nonzero(torch.isfinite(z[0]))[:, 0]
    t = finite[t.long() % len(finite)].to(torch.int32)
    zd, td = z.to(cuda), t.to(cuda)
    scale = 1.0 / rows
    lse, rl, loss = b.sce_fwd(zd, td)
    dz = b.sce_bwd(zd, td, lse, scale)
    rlse, rrl, rloss = mo.sce_fwd(z, t)
    assert np.all(np.abs(lse.cpu().double().numpy() - rlse) <= e)
    assert np.all(np.abs(rl.cpu().double().numpy() - rrl) <= e)
    assert abs(loss.item() - rloss) <= e.max()
    p = np.exp(z.double().numpy() - rlse[:, None])
    assert np.all(np.abs(dz.cpu().double().numpy() - mo.sce_bwd(z, t, scale)) <= scale * (p * (2 * e[:, None] + 1e-6) + 2e-7))
