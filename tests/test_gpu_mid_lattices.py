"""Lattices with one to two bricks of elements for each compute unit, which get
smaller bricks: the residual of diagonal and general Jacobians on sampled elements
(the ends of the lattice among them) against the oracle, in both precisions."""
import numpy as np
import pytest

import oracle
from paper_2107_14027_amd import binding as B
from gpu_util import T_CFG, TOL, ZETA, gpu_residual, rel, say

pytestmark = pytest.mark.gpu

NU_V = 0.05
SKEW = np.array([[0.30, 0.05, -0.02], [0.01, 0.25, 0.04], [-0.03, 0.02, 0.35]])
# double: 257 to 512 bricks; single precision: 513 to 1024
CASES = [(1, (13, 13, 13), B.FR_F64), (1, (17, 17, 17), B.FR_F64), (1, (1, 61, 79), B.FR_F64),
         (2, (12, 12, 12), B.FR_F64), (2, (14, 13, 14), B.FR_F64), (3, (11, 11, 11), B.FR_F64),
         (3, (97, 1, 13), B.FR_F64), (4, (9, 9, 9), B.FR_F64),
         (1, (17, 18, 19), B.FR_F32), (2, (16, 16, 16), B.FR_F32), (3, (14, 13, 14), B.FR_F32)]


@pytest.mark.parametrize("jac", ["diagonal", "general"])
@pytest.mark.parametrize("p,n,prec", CASES)
def test_residual(p, n, prec, jac):
    ne = n[0] * n[1] * n[2]
    U = 0.3 * np.random.default_rng(ne).standard_normal((ne, 13, (p + 1) ** 3))
    if prec == B.FR_F32:
        U = U.astype(np.float32).astype(np.float64)
    J = SKEW if jac == "general" else np.diag([0.30, 0.25, 0.35])
    say("mid lattices p=%d n=%s prec=%d %s" % (p, n, prec, jac))
    R = gpu_residual(p, n, U, nu=NU_V, jac=J, precision=prec)
    assert np.all(np.isfinite(R))
    sel = np.unique(np.concatenate([np.arange(20), np.arange(ne - 20, ne),
                                    np.random.default_rng(p).integers(0, ne, 200)])).astype(np.int64)
    Ro = oracle.residual_elems(p, n, U, sel, ZETA, NU_V, T_CFG, J)
    assert rel(R.reshape(ne, -1)[sel], np.asarray(Ro).reshape(len(sel), -1)) <= TOL[prec]
