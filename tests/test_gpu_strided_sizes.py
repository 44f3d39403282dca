"""The single pass at restart counts that allow no vector loads, below and
above the state size from which a lane's restarts lie 64 apart (2^18 entries
up to 128 restarts, 2^21 beyond): gradients, steps, Adam moments, loss and counts against
the oracle and against the same states in a batch of aligned rows."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import parity_at, say

pytestmark = pytest.mark.gpu

CASES = {
    "planted": lambda n: I.planted_ksat(n, 4 * n, 3, seed=3),
    "mixed": lambda n: I.structured_mixed(n, 4 * n, n // 1000, seed=4),   # split variables
    "batch": lambda n: I.concat([I.structured_mixed(n, 2 * n, n // 1000, seed=5),
                                 I.planted_ksat(900, 3800, 3, seed=6), I.from_clauses([[]], n=1)]),
}


@pytest.mark.parametrize("partials", ["auto", "recompute"])
@pytest.mark.parametrize("R,n", [(65, 4000), (65, 5000), (127, 2000), (127, 3000), (129, 17000), (193, 12000),
                                 (257, 8000), (257, 9000), (333, 7000), (999, 2000), (999, 3000)])
@pytest.mark.parametrize("case", list(CASES))
def test_sizes(case, R, n, partials):
    say(f"[strided] {case} n={n} R={R} {partials}")
    cnf = CASES[case](n)
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
    lw, uw = wide.step(xw, 2, opt_state=sw, trace=True)
    lo, uo = odd.step(xo, 2, opt_state=so, trace=True)
    torch.cuda.synchronize()
    assert torch.equal(uo, uw[:, :, :R])
    assert torch.allclose(lo, lw[:, :, :R], rtol=1e-6)
    assert torch.allclose(xo, xw[:, :R], rtol=1e-5, atol=1e-6)
    assert torch.allclose(so, sw[:, :, :R], rtol=1e-5, atol=1e-7)
