"""The one-kernel residual on linear hexahedra against the three-kernel path,
which the same call takes for a state that is only 8-byte aligned: lattices whose
workgroups hold several elements, full and ragged bricks, one-element directions
and more elements than one brick a compute unit."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import T_CFG, ZETA, say

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
