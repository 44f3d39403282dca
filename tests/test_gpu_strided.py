"""The single pass with a lane's restarts 64 apart (more than 64 restarts that
allow no vector loads) against the oracle and, restart by restart, against
the same states in a batch of aligned rows: gradients, steps, Adam moments,
loss and counts; whole variables and split ones, stored and recomputed
clauses."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import parity_at, say

pytestmark = pytest.mark.gpu

CASES = {
    "planted": lambda: I.planted_ksat(700, 2950, 3, seed=3),
    "mixed": lambda: I.structured_mixed(3000, 12000, 3, seed=4),   # split variables
    "batch": lambda: I.concat([I.structured_mixed(2000, 8000, 2, seed=5),
                               I.planted_ksat(90, 380, 3, seed=6), I.from_clauses([[]], n=1)]),
}


@pytest.mark.parametrize("partials", ["auto", "recompute"])
@pytest.mark.parametrize("R", [65, 75, 127, 129, 193, 257, 333])
@pytest.mark.parametrize("case", list(CASES))
def test_odd_restarts(case, R, partials):
    say(f"[strided] {case} R={R} {partials}")
    cnf = CASES[case]()
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::5] = (x[::5] * 2 - 0.5).clamp(0, 1)
    prob = Problem(cnf, R, partials=partials)
    parity_at(prob, cnf, x, f"{case} R={R}")
    # the same restarts among others, in rows of 16 bytes; with one item per
    # wave in both, variables are split alike and every sum is the same
    Q = (R + 3) // 4 * 4
    wide = Problem(cnf, Q, partials=partials, optimizer="adam", plan_override="lpi=64,rpl=4")
    odd = Problem(cnf, R, partials=partials, optimizer="adam", plan_override="lpi=64,rpl=1")
    xw = torch.zeros((cnf.n, Q), device="cuda")
    xw[:, :R] = x
    xo = x.clone()
    sw, so = wide.new_opt_state(xw), odd.new_opt_state(xo)
    lw, uw = wide.step(xw, 3, opt_state=sw, trace=True)
    lo, uo = odd.step(xo, 3, opt_state=so, trace=True)
    torch.cuda.synchronize()
    assert torch.equal(uo, uw[:, :, :R])
    assert torch.allclose(lo, lw[:, :, :R], rtol=1e-6)
    assert torch.allclose(xo, xw[:, :R], rtol=1e-5, atol=1e-6)
    assert torch.allclose(so, sw[:, :, :R], rtol=1e-5, atol=1e-7)
