"""A variable whose segments are summed in parts (more than 1,024 of them):
in 90,000 clauses of 3 literals and some longer ones, against the oracle, in
the flat plan, the single pass and the two-phase plan, aligned restarts and
others; a second variable with fewer segments, and the rest unsplit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import check_update_oracle, parity_at, say, to_oracle

pytestmark = pytest.mark.gpu


def _formula():
    r = np.random.default_rng(8)
    out = []
    for i in range(90_000):
        v = 2 + r.integers(0, 400, 2)
        sg = r.integers(0, 2, 3) * 2 - 1
        c = [int(sg[0]), int(sg[1] * v[0]), int(sg[2] * v[1])]
        if i % 50 == 0:
            c += [int(2 + r.integers(0, 400)) for _ in range(1 + i % 9)]
        out.append([c[(j + i) % len(c)] for j in range(len(c))])
    for i in range(3000):
        out.append([402, int(2 + r.integers(0, 400)), -403])
    return I.from_clauses(out, n=403)


@pytest.mark.parametrize("R,plan", [(1, ""), (16, ""), (20, ""), (33, ""), (16, "two=1"), (64, "flat=0,two=0"),
                                    (75, ""), (100, ""), (130, "")])
def test_parts(R, plan):
    say(f"[parts] R={R} {plan}")
    cnf = _formula()
    prob = Problem(cnf, R, schedule="general", plan_override=plan or None)
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::3] = (x[::3] * 2 - 0.5).clamp(0, 1)
    parity_at(prob, cnf, x, plan)
    xr = to_oracle(x, R)
    _, g, A = oracle.grad(cnf, xr, with_abs=True)
    x1 = x.clone()
    prob.step(x1, 1)
    torch.cuda.synchronize()
    check_update_oracle(x1, xr, g, A, prob.lr, R, plan)
    x2 = x.clone()
    prob.step(x2, 1)
    torch.cuda.synchronize()
    assert torch.equal(x1, x2)
