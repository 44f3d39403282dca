"""Many tiny formulas under the LDS schedule: beyond 512 workgroups several
restarts share one (up to 16 variables 32, up to 32 variables 16, a loop of a
thread per variable), formulas of up to 64 variables take that loop for one
step and the clause-parallel one for more, larger ones the clause-parallel
one.  States and counts are the general single pass's, bitwise."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,group", [(8, 32), (16, 32), (32, 16), (33, 1), (64, 1), (65, 1), (200, 1)])
def test_many_formulas(n, group):
    say(f"[lds many] n={n}")
    R = 32
    cnf = I.concat([I.planted_ksat(n, 4 * n, 3, seed=i) for i in range(700)] + [I.from_clauses([[]], n=1)])
    prob = Problem(cnf, R, schedule="lds")
    assert prob.info()["lds_restarts_per_group"] == group
    ref = Problem(cnf, R, schedule="general", partials="recompute", plan_override="two=0,segdiv=1")
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(n), device="cuda")
    a, b = x.clone(), x.clone()
    for steps in (1, 2, 1, 5):
        la, ua = prob.step(a, steps, trace=True)
        lb, ub = ref.step(b, steps, trace=True)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(ua, ub), steps
        assert torch.allclose(la, lb, rtol=1e-6, atol=1e-30)
