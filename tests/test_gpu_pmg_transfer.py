"""P-multigrid transfers at the orders the other cycle tests do not reach, on
lattices whose blocks of variables do not fill the transfer kernel's last
workgroup, and a state that is only 8-byte aligned."""
import numpy as np
import pytest

import oracle
from oracle import pmg as opmg
from paper_2107_14027_amd import binding as B
from paper_2107_14027_amd import inputs
from gpu_util import NU, T_CFG, ZETA, rel, say

pytestmark = pytest.mark.gpu


def case(P, n, seed=1):
    Unm1 = inputs.tgv(P, n, noise=1e-4, seed=seed)
    Un = oracle.rk4(P, n, Unm1, ZETA, NU, T_CFG, 1e-3, 2)
    return 2 * Un - Unm1, Un, Unm1


@pytest.mark.parametrize("P,n", [(2, (7, 3, 1)), (5, (3, 1, 2)), (6, (1, 2, 2))])
def test_cycle_matches_oracle(P, n):
    import torch
    G, Un, Unm1 = case(P, n)
    say("pmg transfers P=%d n=%s" % (P, n))
    plan = B.Plan(P, n, ZETA, NU, T_CFG)
    mg = B.Pmg(plan)
    U = torch.tensor(G, device="cuda")
    rc, cyc, res = mg.dual_step(U, torch.tensor(Un, device="cuda"), torch.tensor(Unm1, device="cuda"),
                                1e-2, 5e-4, 1e-30, 1)
    torch.cuda.synchronize()
    Uo, _, reso, _ = opmg.pmg_dual_step(P, n, G, Un, Unm1, ZETA, NU, T_CFG, 1e-2, 5e-4, 1e-30, 1)
    assert rel(U.cpu().numpy().reshape(-1), Uo) <= 1e-11
    assert abs(res - reso) <= 1e-9 * reso
    mg.close()
    plan.close()


@pytest.mark.parametrize("prec", [B.FR_F64, B.FR_F32])
def test_unaligned_state(prec):
    import torch
    P, n = 3, (3, 2, 2)
    G, Un, Unm1 = (torch.tensor(x, device="cuda").reshape(-1) for x in case(P, n))
    say("pmg unaligned state prec=%d" % prec)
    plan = B.Plan(P, n, ZETA, NU, T_CFG, precision=prec)
    mg = B.Pmg(plan)
    room = torch.empty(G.numel() + 1, dtype=torch.float64, device="cuda")
    out = []
    for U in (G.clone(), room[1:]):
        U.copy_(G)
        out.append(mg.dual_step(U, Un, Unm1, 1e-2, 1e-3, 1e-30, 2) + (U.clone(),))
    torch.cuda.synchronize()
    assert out[0][:3] == out[1][:3] and torch.equal(out[0][3], out[1][3])
    assert room[1:].data_ptr() % 16 == 8
    mg.close()
    plan.close()
