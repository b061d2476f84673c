"""Device memory that a plan takes: what its calls need, and nothing left after
it is destroyed."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from gpu_util import NU, T_CFG, ZETA, say

pytestmark = pytest.mark.gpu

SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])
P, N = 3, (24, 24, 24)
TRACES = 6 * 24 ** 3 * 112 * 8      # bytes of one face-trace array in FP64 (93 MB)


def free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def state():
    import torch
    return 1e-2 * torch.randn(24 ** 3 * 13 * 64, dtype=torch.float64, device="cuda")


def test_destroy_gives_everything_back():
    """Steps of a general Jacobian use two face-trace arrays."""
    say("plan memory after destroy")
    U = state()
    free_after = []
    for _ in range(3):      # the first time pays for what the library itself keeps
        plan = B.Plan(P, N, ZETA, NU, T_CFG, SKEW)
        start = free()
        B.fr_rk_step(plan.handle, U, 1e-6, 1)
        assert start - free() >= 2 * TRACES
        plan.close()
        free_after.append(free())
    assert free_after[0] - free_after[2] < TRACES // 2


@pytest.mark.parametrize("form,arrays", [(B.FR_FORM_AUTO, 0), (B.FR_FORM_POINT, 1)])
def test_residual_of_a_general_jacobian_takes_what_it_reads(form, arrays):
    """The automatic form's one kernel has no face traces in memory."""
    import torch
    say("residual memory form=%d" % form)
    U = state()
    R = torch.empty_like(U)
    for _ in range(2):      # the first time pays for what the library itself keeps
        plan = B.Plan(P, N, ZETA, NU, T_CFG, SKEW)
        plan.set(B.FR_OPT_FORM, form)
        start = free()
        B.fr_residual(plan.handle, U, R)
        used = start - free()
        plan.close()
    assert arrays * TRACES <= used < arrays * TRACES + TRACES // 2
