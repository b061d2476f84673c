"""The one-kernel residuals whose metric mixes the directions.  Linear hexahedra:
against the three-kernel path, which the same call takes for a state that is only
8-byte aligned.  A general constant Jacobian: AUTO against the point form, on both
sides of AUTO's size rule.  Lattices whose workgroups hold several elements, full
and ragged bricks, one-element directions and more elements than one brick a
compute unit."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import NU, T_CFG, TOL, ZETA, check_groups, gpu_residual, rel, say

pytestmark = pytest.mark.gpu

CASES = [(1, (33, 18, 15)), (1, (2, 1, 3)), (2, (31, 13, 11)), (3, (15, 14, 11)), (3, (1, 1, 1)),
         (4, (13, 11, 9)), (4, (1, 5, 2)), (5, (7, 9, 9)), (6, (1, 7, 5))]


def residual(p, n, C, U, shift):
    """The GPU residual with U and R shift doubles past a 16-byte boundary."""
    import torch
    plan = B.Plan(p, n, ZETA, 0.05, T_CFG)
    lh = B.LinearHex(plan)
    u, r = (torch.zeros(U.size + shift, dtype=torch.float64, device="cuda")[shift:] for _ in range(2))
    u.copy_(torch.from_numpy(U.ravel()))
    lh.residual(torch.from_numpy(np.ascontiguousarray(C)).to("cuda"), u, r)
    out = r.cpu().numpy().reshape(U.shape)
    lh.close()
    plan.close()
    return out


@pytest.mark.parametrize("p,n", CASES)
def test_one_kernel_against_three(p, n):
    U = 0.5 * np.random.default_rng(60 + p).standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    C = inputs.linear_hex_corners(n, amp=0.15, seed=p, smooth=0.1)
    say("metric lines p=%d n=%s" % (p, n))
    a, b = (residual(p, n, C, U, shift) for shift in (0, 1))
    # both sum the same terms in another order: some hundred roundings of the
    # largest residual, as in the comparison with the oracle
    assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])


@pytest.mark.parametrize("p,n", [(1, (17, 9, 14)), (2, (31, 13, 11)), (2, (4, 4, 4)), (3, (15, 14, 11)),
                                 (3, (1, 64, 1)), (3, (9, 7, 1)), (4, (13, 11, 9)), (5, (10, 11, 10)),
                                 (6, (10, 10, 10)), (6, (9, 3, 37))])
@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
def test_general_jacobian_against_point_form(p, n, prec):
    U = 0.3 * np.random.default_rng(80 + p).standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    say("skew lines p=%d n=%s prec=%d" % (p, n, prec))
    a, b = (gpu_residual(p, n, U, precision=prec, jac=SKEW, form=f) for f in (B.FR_FORM_AUTO, B.FR_FORM_POINT))
    assert rel(a, b) <= TOL[prec], rel(a, b)
    check_groups(a, b, prec, U, what="skew lines p=%d n=%s" % (p, n))


def test_general_jacobian_without_allocation():
    """The allocation-free call runs the same kernel, within its old limit."""
    import torch
    for n, ok in (((9, 8, 7), True), ((32, 32, 32), False)):
        plan = B.Plan(3, n, ZETA, NU, T_CFG, SKEW)
        U = torch.randn(plan.state_len, dtype=torch.float64, device="cuda")
        R, Rn = torch.empty_like(U), torch.empty_like(U)
        B.fr_residual(plan.handle, U, R)
        if ok:
            B.fr_residual_noalloc(plan.handle, U, Rn)
            assert torch.equal(R, Rn)
        else:
            with pytest.raises(B.FrError) as ei:
                B.fr_residual_noalloc(plan.handle, U, Rn)
            assert ei.value.code == B.FR_EINVAL
        torch.cuda.synchronize()
        plan.close()
