"""The flat plan's steps at restart counts that are no multiple of four: four
restarts a lane in the internal rows, the columns past the last restart
dropped.  Each restart's states equal those of a batch with the next multiple
of four (the same plan), for split and unsplit variables, clause rows, one
and several steps, and padded callers' rows, whose padding stays; gradients
and Adam steps (one restart a lane) against the oracle."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import parity_at, say

pytestmark = pytest.mark.gpu

CASES = {
    "planted": lambda: I.planted_ksat(900, 3800, 3, seed=3),
    "zipf": lambda: I.large_zipf(4000, 16000, seed=4),              # split variables, long clauses
    "batch": lambda: I.concat([I.structured_mixed(2000, 8000, 2, seed=5),
                               I.planted_ksat(90, 380, 3, seed=6), I.from_clauses([[]], n=1)]),
}


@pytest.mark.parametrize("R", [17, 18, 31, 33, 47, 50, 63])
@pytest.mark.parametrize("case", list(CASES))
def test_odd(case, R):
    say(f"[flat odd] {case} R={R}")
    cnf = CASES[case]()
    Q = (R + 3) // 4 * 4
    xq = torch.rand((cnf.n, Q), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    xq[::5] = (xq[::5] * 2 - 0.5).clamp(0, 1)
    odd = Problem(cnf, R, plan_override="flat=1")
    even = Problem(cnf, Q, plan_override="flat=1")
    parity_at(odd, cnf, xq[:, :R].contiguous(), f"{case} R={R}")
    for ld in (R, Q, Q + 1):
        x = torch.full((cnf.n, ld), -3.0, device="cuda")
        x[:, :R] = xq[:, :R]
        y = xq.clone()
        for steps in (1, 2):
            lo, uo = odd.step(x, steps, trace=True)
            lq, uq = even.step(y, steps, trace=True)
            torch.cuda.synchronize()
            assert torch.equal(x[:, :R], y[:, :R]), (ld, steps)
            assert torch.equal(uo, uq[:, :, :R])
            assert torch.allclose(lo, lq[:, :, :R], rtol=1e-6)
        assert bool((x[:, R:] == -3.0).all())
    adam = Problem(cnf, R, plan_override="flat=1", optimizer="adam")
    wide = Problem(cnf, Q, plan_override="flat=1", optimizer="adam")
    x, y = xq[:, :R].contiguous(), xq.clone()
    adam.step(x, 2, opt_state=adam.new_opt_state(x))
    wide.step(y, 2, opt_state=wide.new_opt_state(y))
    torch.cuda.synchronize()
    assert torch.allclose(x, y[:, :R], rtol=1e-5, atol=1e-6)
