"""The one-kernel residual of the standard ACM system (diagonal Jacobian, beta =
1/2, 16-byte aligned states) against the four-kernel path, which the same call
takes for a state that is only 8-byte aligned: lattices whose workgroups hold
several elements, full and ragged bricks, one-element directions, and beta,
tau and Jacobians on both sides of the rule."""
import numpy as np
import pytest

from oracle import acm_ldg
from paper_2107_14027_amd import binding as B
from gpu_util import NU, T_CFG, ZETA, rel, say

pytestmark = pytest.mark.gpu
CASES = [(1, (33, 18, 15)), (1, (3, 1, 2)), (2, (31, 13, 11)), (3, (15, 14, 11)), (3, (1, 1, 1)),
         (4, (13, 11, 9)), (5, (7, 9, 9)), (6, (1, 7, 5))]


def state(p, n, seed):
    rng = np.random.default_rng(seed)
    U = 0.3 * rng.standard_normal((n[0] * n[1] * n[2], 4, (p + 1) ** 3))
    return U + np.array([1.0, 0.4, -0.3, 0.2])[None, :, None]


def residual(p, n, U, beta, tau, jac, shift):
    """The GPU residual with U and R shift doubles past a 16-byte boundary."""
    import torch
    plan = B.Plan(p, n, ZETA, NU, T_CFG, jac)
    acm = B.Acm(plan, beta, tau)
    u, r = (torch.zeros(U.size + shift, dtype=torch.float64, device="cuda")[shift:] for _ in range(2))
    u.copy_(torch.from_numpy(U.ravel()))
    acm.residual(u, r)
    out = r.cpu().numpy().reshape(U.shape)
    acm.close()
    plan.close()
    return out


@pytest.mark.parametrize("p,n", CASES)
@pytest.mark.parametrize("tau", [0.1, 0.0])
def test_lines_against_four_kernels(p, n, tau):
    U = state(p, n, 40 + p)
    say("acm lines p=%d n=%s tau=%g" % (p, n, tau))
    a, b = (residual(p, n, U, 0.5, tau, None, shift) for shift in (0, 1))
    assert rel(a, b) <= 1e-12
    assert np.max(np.abs(a - b)) <= 5e-12 * np.max(np.abs(b))
    if len(U) <= 40:
        assert rel(a, acm_ldg.residual(p, n, U, ZETA, NU, 0.5, tau)) <= 1e-12


@pytest.mark.parametrize("beta,skew", [(0.5, True), (-0.5, False), (0.0, False)])
def test_other_settings_keep_the_four_kernels(beta, skew):
    p, n = 2, (4, 3, 3)
    jac = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]]) if skew else None
    U = state(p, n, 9)
    say("acm beta=%g skew=%s" % (beta, skew))
    a, b = (residual(p, n, U, beta, 0.1, jac, shift) for shift in (0, 1))
    assert np.array_equal(a, b)
    assert rel(a, acm_ldg.residual(p, n, U, ZETA, NU, beta, 0.1, jac)) <= 1e-12
