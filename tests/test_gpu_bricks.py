"""The line forms on lattices large enough for their workgroups to hold several
elements (smaller ones get one element each): bricks whose inner faces come
from the tile, bricks that stick out of the lattice, odd elements (whose blocks
start 8, 4 or 12 bytes after a 16-byte boundary), lattices of one element in a
direction, and a last group of workgroups that is not full."""
import numpy as np
import pytest

import oracle
from paper_2107_14027_amd import binding as B
from gpu_util import NU, T_CFG, TOL, ZETA, gpu_residual, rel, say

pytestmark = pytest.mark.gpu
PREC = [B.FR_F64, B.FR_F32]
# full and ragged bricks per order; at least 256 E (512 E in single precision) elements
CASES = [(1, (33, 18, 15)), (1, (1, 97, 89)), (2, (31, 13, 11)), (3, (15, 14, 11)), (3, (2, 1, 1031)),
         (4, (13, 11, 9)), (4, (1031, 1, 1)), (5, (7, 9, 9)), (6, (9, 7, 5))]


def rand_U(p, n, seed):
    rng = np.random.default_rng(seed)
    U = 0.3 * rng.standard_normal((n[0] * n[1] * n[2], 13, (p + 1) ** 3))
    U[:, :4] += np.array([1.0, 0.4, -0.3, 0.2])[None, :, None]
    return U


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("p,n", CASES)
def test_residual_on_bricks(prec, p, n):
    """Halo form against the oracle on sampled elements (the ends of the lattice
    among them) and bitwise against the line form everywhere."""
    U = rand_U(p, n, seed=700 + p)
    if prec == B.FR_F32:
        U = U.astype(np.float32).astype(np.float64)
    say("bricks p=%d n=%s prec=%d" % (p, n, prec))
    R = gpu_residual(p, n, U, precision=prec, form=B.FR_FORM_HALO)
    L = gpu_residual(p, n, U, precision=prec, form=B.FR_FORM_LINES)
    assert np.array_equal(R, L)
    ne = len(U)
    sel = np.unique(np.concatenate([np.arange(min(ne, 20)), np.arange(ne - 20, ne),
                                    np.random.default_rng(p).integers(0, ne, 60)])).astype(np.int64)
    Ro = oracle.residual_elems(p, n, U, sel, ZETA, NU, T_CFG)
    assert rel(R.reshape(ne, -1)[sel], np.asarray(Ro).reshape(len(sel), -1)) <= TOL[prec]


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("p,n", CASES)
def test_stage_update_on_bricks(prec, p, n):
    """RK4 and dual time stepping with the halo form's stage epilogue bitwise
    against its residual and the separate stage kernel."""
    import torch
    say("bricks stage p=%d n=%s prec=%d" % (p, n, prec))
    U0 = torch.tensor(1e-1 * rand_U(p, n, seed=800 + p), device="cuda")
    outs = []
    for fuse in (1, 0):
        pl = B.Plan(p, n, ZETA, NU, T_CFG, None, prec, B.FR_FUSED)
        pl.set(B.FR_OPT_FUSE_STAGE, fuse)
        pl.set(B.FR_OPT_FORM, B.FR_FORM_HALO)
        V = U0.clone()
        B.fr_rk_step(pl.handle, V, 1e-5, 2)
        W = V.clone()
        rc, it, res = B.fr_dual_step(pl.handle, W, V, U0, 1e-2, 1e-5, 1e-12, 3, check_every=2)
        torch.cuda.synchronize()
        outs.append((V, W, rc, it, res))
        pl.close()
    (Va, Wa, ra, ia, sa), (Vb, Wb, rb, ib, sb) = outs
    assert torch.equal(Va, Vb) and torch.equal(Wa, Wb)
    assert (ra, ia) == (rb, ib) and abs(sa - sb) <= 1e-12 * abs(sb)
    assert not torch.equal(Va, U0) and not torch.equal(Wa, Va)
