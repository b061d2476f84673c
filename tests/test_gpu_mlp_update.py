"""The kernel that sums the gradient partials, with and without the block that
sums the loss, behind fr_mlp_grad and fr_mlp_train_step: both calls see one
gradient and one loss, from a single row to several tiles a wave."""
import numpy as np
import pytest

from paper_2107_14027_amd import binding as B
from gpu_util import NU, T_CFG, ZETA, say

pytestmark = pytest.mark.gpu
NPAR, NORM = 5252, 28


@pytest.mark.parametrize("n", [1, 17, 4097, 33000])
def test_grad_and_step_agree(n):
    import torch as t
    rng = np.random.default_rng(n)
    say("mlp update n=%d" % n)
    plan = B.Plan(1, (2, 2, 2), ZETA, NU, T_CFG)
    S0 = rng.uniform(-0.3, 0.3, 3 * NPAR + NORM).astype(np.float32)
    S0[NPAR:NPAR + NORM] = 1.0
    S0[NPAR + NORM:] = 0.0
    X, Y = (t.tensor(rng.standard_normal((n, c)), dtype=t.float32, device="cuda") for c in (12, 4))
    S, S1 = t.tensor(S0, device="cuda"), t.tensor(S0, device="cuda")
    g, g1 = (t.zeros(NPAR, dtype=t.float32, device="cuda") for _ in range(2))
    loss, loss1 = (t.zeros(1, dtype=t.float32, device="cuda") for _ in range(2))
    B.fr_mlp_grad(plan.handle, S, X, Y, g, loss)
    B.fr_mlp_grad(plan.handle, S, X, Y, g1)
    B.fr_mlp_train_step(plan.handle, S, X, Y, 1e-3, 1, loss1)
    B.fr_mlp_train_step(plan.handle, S1, X, Y, 1e-3, 1)
    t.cuda.synchronize()
    assert t.equal(g, g1) and t.equal(loss, loss1) and t.equal(S, S1)
    assert float(loss) > 0.0
    # the first step's moments: (1 - beta) times the gradient and its square, a
    # few roundings of single precision
    m, v = (S[NPAR + NORM + i * NPAR:][:NPAR].double().cpu().numpy() for i in range(2))
    gd = g.double().cpu().numpy()
    assert np.allclose(m, 0.1 * gd, rtol=1e-6, atol=0.0)
    assert np.allclose(v, 1e-3 * gd * gd, rtol=1e-4, atol=1e-30)
    plan.close()
