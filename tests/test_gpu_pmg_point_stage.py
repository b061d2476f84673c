"""P-multigrid cycles whose coarse levels apply the BDF term and the fixed defect in
the point form's stage epilogue (a general Jacobian): bitwise against the separate
stage kernel.
Fewer elements than FR_FORM_AUTO's line tasks take, so that both run the point
form's residual."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import NU, T_CFG, ZETA, say

pytestmark = pytest.mark.gpu

SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])


@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
def test_cycles_bitwise_against_separate_stages(p, prec):
    import torch
    n = (4, 3, 3) if p < 5 else (3, 2, 2)
    say("pmg point stage p=%d prec=%d" % (p, prec))
    Un = torch.from_numpy(inputs.tgv(p, n, noise=1e-3, seed=p)).to("cuda")
    Unm1 = torch.from_numpy(inputs.tgv(p, n, noise=1e-3, seed=p + 10)).to("cuda")
    outs = []
    for fuse in (1, 0):
        plan = B.Plan(p, n, ZETA, NU, T_CFG, SKEW, prec)
        plan.set(B.FR_OPT_FUSE_STAGE, fuse)
        mg = B.Pmg(plan)
        U = Un.clone()
        rc, cycles, res = mg.dual_step(U, Un, Unm1, 1e-2, 1e-4, 1e-30, 2, raise_on_error=False)
        torch.cuda.synchronize()
        outs.append((U, rc, cycles, res))
        mg.close()
        plan.close()
    (Ua, ra, ca, sa), (Ub, rb, cb, sb) = outs
    assert (ra, ca) == (rb, cb) and ca == 2 and abs(sa - sb) <= 1e-12 * abs(sb)
    assert torch.equal(Ua, Ub) and not torch.equal(Ua, Un)
