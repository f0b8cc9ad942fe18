"""Cross-entropy forward on either side of the rule that gives a few long rows
16 waves each, against the float64 oracle with the tolerances of the
memory-bound operator tests."""

import numpy as np
import pytest

from paper_2608_00029_amd import binding as b
from paper_2608_00029_amd.workloads import make_sce_inputs
from parity_util import say
from test_gpu_memops import _check_sce_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,V", [(1, 16384), (256, 16384), (257, 16384), (256, 16380), (3, 50304), (2, 16388)])
def test_sce_row_rule(cuda, rows, V):
    z, t = make_sce_inputs(rows, V, seed=rows + V, sigma=3.0)
    say(f"sce rows={rows} V={V}")
    zd, td = z.to(cuda), t.to(cuda)
    scale = 1.0 / rows
    lse, rl, loss = b.sce_fwd(zd, td)
    dz = b.sce_bwd(zd, td, lse, scale)
    _check_sce_rows(z, t, lse, rl, dz, np.arange(rows), scale)
    assert abs(loss.item() - rl.cpu().double().mean().item()) <= 1e-6 * abs(loss.item()) + 1e-7
