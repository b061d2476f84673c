"""Time steps whose stage arrays have an odd number of values (even order, odd
number of elements): every array of the scratch starts on a boundary that the
kernels' 16-byte accesses need.  Against the oracle, in both precisions, on every
stage path, with diagonal and general Jacobians."""
import numpy as np
import pytest

import oracle
from paper_2107_14027_amd import binding as B
from gpu_util import T_CFG, ZETA, rel, say

pytestmark = pytest.mark.gpu

NU_V = 0.05
SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])


def state(p, n, seed):
    U = 0.3 * np.random.default_rng(seed).standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    U[:, :4] += np.array([1.0, 0.4, -0.3, 0.2])[None, :, None]
    return U


# the last two: larger than AUTO's line-task threshold, one of them with no epilogue (p = 6)
CASES = [(2, (3, 1, 5), None), (2, (13, 9, 7), None), (4, (3, 3, 1), None), (6, (1, 3, 1), None),
         (2, (3, 3, 1), SKEW), (4, (1, 3, 3), SKEW), (4, (5, 5, 3), SKEW), (6, (11, 13, 7), SKEW)]


@pytest.mark.parametrize("fuse,form", [(1, B.FR_FORM_AUTO), (1, B.FR_FORM_POINT), (1, B.FR_FORM_HALO),
                                       (0, B.FR_FORM_AUTO)])
@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
@pytest.mark.parametrize("p,n,jac", CASES)
def test_steps_against_oracle(p, n, jac, prec, fuse, form):
    import torch
    if jac is not None and form == B.FR_FORM_HALO:
        pytest.skip("the halo form needs a diagonal Jacobian")
    J = np.diag([0.30, 0.25, 0.35]) if jac is None else jac
    U0, dt = state(p, n, 70 + p), 2e-4
    assert U0.size % 2 == 1
    say("odd lattice p=%d n=%s skew=%s prec=%d fuse=%d form=%d" % (p, n, jac is not None, prec, fuse, form))
    plan = B.Plan(p, n, ZETA, NU_V, T_CFG, J, prec)
    plan.set(B.FR_OPT_FUSE_STAGE, fuse)
    plan.set(B.FR_OPT_FORM, form)
    U = torch.from_numpy(U0.copy()).to("cuda")
    B.fr_rk_step(plan.handle, U, dt, 1)
    V = U.clone()
    rc, it, res = B.fr_dual_step(plan.handle, V, U, None, 1e-2, dt, 1e-30, 2, raise_on_error=False)
    Ug, Vg = U.cpu().numpy(), V.cpu().numpy()
    plan.close()
    f64 = prec == B.FR_F64
    Uo = oracle.rk4(p, n, U0, ZETA, NU_V, T_CFG, dt, 1, J)
    assert rel(Ug, Uo) <= (1e-12 if f64 else 1e-5)
    assert rel(Ug - U0, Uo - U0) <= (1e-10 if f64 else 1e-4)
    Vo, ito, reso, _ = oracle.dual_step(p, n, Ug, Ug, None, ZETA, NU_V, T_CFG, 1e-2, dt, 1e-30, 2, 1, J)
    assert rc == B.FR_ENOCONV and it == ito == 2
    assert abs(res - reso) <= (1e-9 if f64 else 1e-4) * reso
    assert rel(Vg - Ug, Vo - Ug) <= (1e-9 if f64 else 1e-4)
