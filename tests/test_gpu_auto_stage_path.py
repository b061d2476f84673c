"""FR_FORM_AUTO's stage path on both sides of its size rule: what
FR_INFO_STAGE_PATH reports, and RK4 steps with the bits of the form it names."""
import pytest

from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import NU, T_CFG, ZETA, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,prec,path", [(4, (10, 8, 10), B.FR_F64, B.FR_STAGE_POINT),
                                           (4, (89, 3, 3), B.FR_F64, B.FR_STAGE_HALO),
                                           (4, (11, 10, 10), B.FR_F64, B.FR_STAGE_HALO),
                                           (5, (4, 2, 2), B.FR_F32, B.FR_STAGE_POINT),
                                           (5, (17, 1, 1), B.FR_F32, B.FR_STAGE_HALO),
                                           (4, (4, 2, 2), B.FR_F32, B.FR_STAGE_HALO)])
def test_automatic_stage_path(p, n, prec, path):
    import torch
    say("auto stage path p=%d n=%s prec=%d" % (p, n, prec))
    U0 = torch.from_numpy(inputs.tgv(p, n, noise=1e-3, seed=31)).to("cuda")
    out = []
    for form in (B.FR_FORM_AUTO, B.FR_FORM_HALO if path == B.FR_STAGE_HALO else B.FR_FORM_POINT):
        plan = B.Plan(p, n, ZETA, NU, T_CFG, None, prec)
        plan.set(B.FR_OPT_FORM, form)
        assert B.fr_plan_get_int(plan.handle, B.FR_INFO_STAGE_PATH) == path
        U = U0.clone()
        B.fr_rk_step(plan.handle, U, 1e-4, 2)
        torch.cuda.synchronize()
        out.append(U)
        plan.close()
    assert torch.equal(*out) and not torch.equal(out[0], U0)
