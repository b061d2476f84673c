"""FR_OPT_BLOCK sets the elements per workgroup of the point form's kernel; a
general Jacobian under FR_FORM_AUTO keeps that kernel when it is set."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from gpu_util import gpu_residual, say

pytestmark = pytest.mark.gpu

SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])


@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
@pytest.mark.parametrize("p,n", [(2, (7, 5, 4)), (4, (5, 6, 4)), (6, (10, 10, 10))])
def test_block_is_honoured_with_a_general_jacobian(p, n, prec):
    U = 0.3 * np.random.default_rng(p).standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    say("block p=%d n=%s prec=%d" % (p, n, prec))
    most = B.fr_launch_shape(p, prec, B.FR_K_FUSED)[0]
    for block in {1, most}:
        a, b = (gpu_residual(p, n, U, jac=SKEW, precision=prec, block=block, form=f)
                for f in (B.FR_FORM_AUTO, B.FR_FORM_POINT))
        assert np.array_equal(a, b), block
