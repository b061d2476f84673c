"""Steps that replay a captured graph after the kernel form has changed: the
graph of one form must not run for another.  Bitwise against plain launches of
the same sequence."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import NU, T_CFG, ZETA, say

pytestmark = pytest.mark.gpu

FORMS = [B.FR_FORM_POINT, B.FR_FORM_HALO, B.FR_FORM_POINT, B.FR_FORM_LINES, B.FR_FORM_AUTO, B.FR_FORM_POINT]


@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
@pytest.mark.parametrize("dual", [False, True])
def test_form_changes_between_replays(prec, dual):
    import torch
    p, n = 3, (4, 5, 3)
    say("graph forms prec=%d dual=%d" % (prec, dual))
    plans = [B.Plan(p, n, ZETA, NU, T_CFG, None, prec, B.FR_FUSED) for _ in range(2)]
    states = [torch.from_numpy(inputs.tgv(p, n, noise=1e-2, seed=21)).to("cuda") for _ in plans]
    past = states[0].clone()
    for graph, pl in enumerate(plans):
        pl.set(B.FR_OPT_GRAPH, graph)
    for i, form in enumerate(FORMS):
        for pl, U in zip(plans, states):
            pl.set(B.FR_OPT_FORM, form)
            if dual:
                B.fr_dual_step(pl.handle, U, past, None, 1e-2, 1e-3, 1e-30, 5, check_every=2,
                               raise_on_error=False)
            else:
                B.fr_rk_step(pl.handle, U, 5e-3, 4)
            (U * 1.0001).sum().item()     # other work in between
        assert torch.equal(*states), (i, form)
    assert bool(torch.isfinite(states[0]).all())
    for pl in plans:
        pl.close()
