"""ACM-HD on diagonal Jacobians with two negative entries (det J > 0, the unit
normal of those faces points against its axis) and with three different positive
ones, against the oracle: the residual in every variant and form, in both
precisions, and RK4 and dual steps through every stage path."""
import numpy as np
import pytest

import oracle
from paper_2107_14027_amd import binding as B
from gpu_util import T_CFG, TOL, ZETA, check_groups, gpu_residual, rel, say

pytestmark = pytest.mark.gpu

NU_V = 0.05     # large enough for the viscous part of a face's flux to count
SIGNS = [(-1, -1, 1), (1, -1, -1), (-1, 1, -1), (1, 1, 1)]
LATTICES = {1: (4, 3, 5), 2: (3, 2, 4), 3: (2, 3, 2), 4: (3, 1, 2), 5: (2, 2, 1), 6: (1, 2, 2)}


def jacobian(signs):
    return np.diag(np.array(signs) * [0.30, 0.25, 0.35])


def state(p, n, seed, prec=B.FR_F64):
    U = 0.3 * np.random.default_rng(seed).standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    U[:, :4] += np.array([1.0, 0.4, -0.3, 0.2])[None, :, None]
    return U if prec == B.FR_F64 else U.astype(np.float32).astype(np.float64)


RUNS = ([(prec, B.FR_FUSED, f) for prec in (B.FR_F64, B.FR_F32)
         for f in (B.FR_FORM_AUTO, B.FR_FORM_POINT, B.FR_FORM_LINES, B.FR_FORM_HALO)] +
        [(B.FR_F64, B.FR_UNFUSED, B.FR_FORM_AUTO), (B.FR_F32, B.FR_MFMA, B.FR_FORM_AUTO)])


@pytest.mark.parametrize("prec,variant,form", RUNS)
@pytest.mark.parametrize("signs", SIGNS)
@pytest.mark.parametrize("p", range(1, 7))
def test_residual(p, signs, prec, variant, form):
    n, J = LATTICES[p], jacobian(signs)
    U = state(p, n, 90 + p, prec)
    what = "signed p=%d signs=%s prec=%d variant=%d form=%d" % (p, signs, prec, variant, form)
    say(what)
    R = gpu_residual(p, n, U, nu=NU_V, jac=J, precision=prec, variant=variant, form=form)
    Ro = oracle.residual(p, n, U, ZETA, NU_V, T_CFG, J)
    assert rel(R, Ro) <= TOL[prec]
    check_groups(R, Ro, prec, U, what=what)


@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
def test_residual_on_bricks(prec):
    """A lattice whose workgroups hold several elements."""
    p, n, J = 2, (13, 9, 8), jacobian(SIGNS[0])
    U = state(p, n, 99, prec)
    say("signed bricks prec=%d" % prec)
    R = gpu_residual(p, n, U, nu=NU_V, jac=J, precision=prec)
    assert rel(R, oracle.residual(p, n, U, ZETA, NU_V, T_CFG, J)) <= TOL[prec]


@pytest.mark.parametrize("fuse,form", [(1, B.FR_FORM_AUTO), (1, B.FR_FORM_POINT), (1, B.FR_FORM_HALO),
                                       (0, B.FR_FORM_AUTO)])
@pytest.mark.parametrize("signs", SIGNS[:2])
@pytest.mark.parametrize("p", [2, 3, 6])
def test_time_steps(p, signs, fuse, form):
    import torch
    n, J = LATTICES[p], jacobian(signs)
    U0 = state(p, n, 95 + p)
    say("signed steps p=%d signs=%s fuse=%d form=%d" % (p, signs, fuse, form))
    plan = B.Plan(p, n, ZETA, NU_V, T_CFG, J)
    plan.set(B.FR_OPT_FUSE_STAGE, fuse)
    plan.set(B.FR_OPT_FORM, form)
    U = torch.from_numpy(U0.copy()).to("cuda")
    B.fr_rk_step(plan.handle, U, 1e-3, 3)
    V = U.clone()
    rc, it, res = B.fr_dual_step(plan.handle, V, U, None, 1e-2, 1e-3, 1e-30, 3, raise_on_error=False)
    Ug, Vg = U.cpu().numpy(), V.cpu().numpy()
    plan.close()
    Uo = oracle.rk4(p, n, U0, ZETA, NU_V, T_CFG, 1e-3, 3, J)
    assert rel(Ug, Uo) <= 1e-12 and rel(Ug - U0, Uo - U0) <= 1e-10
    Vo, ito, reso, _ = oracle.dual_step(p, n, Ug, Ug, None, ZETA, NU_V, T_CFG, 1e-2, 1e-3, 1e-30, 3, 1, J)
    assert rc == B.FR_ENOCONV and it == ito == 3 and abs(res - reso) <= 1e-9 * reso
    assert rel(Vg, Vo) <= 1e-12 and rel(Vg - Ug, Vo - Ug) <= 1e-9
