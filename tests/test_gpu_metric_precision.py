"""Rounding of the one-kernel residual of a general Jacobian (FR_FORM_AUTO): in
single precision, against the oracle in double, its root mean square error per
variable group is no larger than the point form's.  Over some 10^5 values per group
that error is known to about 0.3 %; 1 % is allowed."""
import numpy as np
import pytest

import oracle
from paper_2107_14027_amd import binding as B
from gpu_util import GROUPS, T_CFG, ZETA, gpu_residual, say

pytestmark = pytest.mark.gpu

SKEW = np.array([[0.30, 0.09, -0.06], [0.03, 0.27, 0.075], [-0.045, 0.06, 0.33]])


@pytest.mark.parametrize("p,n", [(2, (21, 18, 19)), (3, (17, 15, 16)), (5, (11, 10, 12))])
def test_error_is_not_larger_than_the_point_forms(p, n):
    ne, m = n[0] * n[1] * n[2], p + 1
    # a smooth field with the velocity gradients as auxiliary variables, and some noise
    rng = np.random.default_rng(p)
    xi = np.polynomial.legendre.leggauss(m)[0]
    th = [2 * np.pi / k * ((xi + 1) / 2 + np.arange(k)[:, None]) for k in n]
    grid = [th[0][None, None, :, None, None, :], th[1][None, :, None, None, :, None], th[2][:, None, None, :, None, None]]
    to_x = np.diag([np.pi / k for k in n]) @ np.linalg.inv(SKEW)
    U = np.zeros((n[2], n[1], n[0], 13, m, m, m))
    for f in range(4):
        for _ in range(4):
            k = rng.integers(-4, 5, size=3)
            amp, ph = rng.normal() / 2, rng.uniform(0, 2 * np.pi)
            arg = k[0] * grid[0] + k[1] * grid[1] + k[2] * grid[2] + ph
            U[:, :, :, f] += amp * np.sin(arg)
            if f:
                for j, kj in enumerate(k @ to_x):
                    U[:, :, :, 4 + 3 * (f - 1) + j] += amp * kj * np.cos(arg)
    U = (U + 1e-3 * rng.standard_normal(U.shape)).reshape(ne, 13, m ** 3)
    U = U.astype(np.float32).astype(np.float64)
    Ro = oracle.residual(p, n, U, ZETA, 1.0 / 1600.0, T_CFG, SKEW)
    err = {}
    for form in (B.FR_FORM_AUTO, B.FR_FORM_POINT):
        R = gpu_residual(p, n, U, jac=SKEW, precision=B.FR_F32, form=form)
        err[form] = [float(np.linalg.norm((R - Ro)[:, sl])) for _, sl in GROUPS]
    say("metric precision p=%d:" % p, " ".join("%s %.3f" % (g[0], a / b) for g, a, b in
                                              zip(GROUPS, err[B.FR_FORM_AUTO], err[B.FR_FORM_POINT])))
    for a, b in zip(err[B.FR_FORM_AUTO], err[B.FR_FORM_POINT]):
        assert a <= 1.01 * b
