"""The clause-parallel LDS step loop against the general single pass: the
same products summed in the same order, so states and counts are bitwise
equal and the loss (its sum has another order) agrees to 1e-6; and against
the oracle where AUTO takes it.

The sizes lie around the kernel's limits: 2 or 4 or 8 clauses of up to three
literals a thread (512, 1,024, 2,048, 4,096 and 8,192 clauses), slices of 64
variables, clauses of 4 to 8 literals, formulas without clauses or with
empty ones, and batches of at least 8 formulas (a formula's restarts on one
XCD)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import check_counts, check_loss, check_update, say, to_oracle

pytestmark = pytest.mark.gpu


def _mixed(n, m, seed):
    """Clauses of 0 to 8 literals over n variables, repeats allowed."""
    r = np.random.default_rng(seed)
    out = []
    for k in r.integers(0, 9, m):
        v = r.integers(1, n + 1, int(k))
        out.append([int(a) * (1 if s else -1) for a, s in zip(v, r.random(int(k)) < 0.5)])
    return I.from_clauses(out, n=n)


FORMULAS = {
    **{f"m{m}": (lambda m=m: I.planted_ksat(max(m // 4, 63), m, 3, seed=m))
       for m in (511, 512, 513, 1025, 2048, 2049, 4097, 8192)},
    "n64": lambda: I.planted_ksat(64, 260, 3, seed=1),
    "n65": lambda: I.planted_ksat(65, 260, 3, seed=2),
    "one": lambda: I.from_clauses([[1], [-1]], n=1),
    "lengths": lambda: _mixed(70, 300, 3),
    "lengths_many": lambda: _mixed(500, 1500, 4),
    "batch7": lambda: I.concat([_mixed(20 + i, 60, i) for i in range(7)]),
    "batch13": lambda: I.concat([_mixed(20 + 9 * i, 80 + i, i) for i in range(11)] +
                                [I.from_clauses([[]], n=1), I.from_clauses([], n=3)]),
}


@pytest.mark.parametrize("R", [1, 3, 64])
@pytest.mark.parametrize("case", list(FORMULAS))
def test_matches_single_pass(case, R):
    say(f"[clause-lds] {case} R={R}")
    cnf = FORMULAS[case]()
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::7] = 0.0
    x[3::11] = 1.0
    a = Problem(cnf, R, schedule="lds")
    b = Problem(cnf, R, schedule="general", partials="recompute", plan_override="two=0,segdiv=1")
    c = Problem(cnf, R)
    assert c.info()["schedule"] == "lds"
    xa, xb, xc = x.clone(), x.clone(), x.clone()
    la, ua = a.step(xa, 4, trace=True)
    lb, ub = b.step(xb, 4, trace=True)
    c.step(xc, 1)
    lc, uc = c.step(xc, 3, trace=True)
    torch.cuda.synchronize()
    assert torch.equal(xa, xb) and torch.equal(ua, ub)
    assert torch.allclose(la, lb, rtol=1e-6, atol=1e-30)
    assert torch.equal(xa, xc) and torch.equal(ua[1:], uc) and torch.equal(la[1:], lc)
    xr = to_oracle(x, R)
    loss, g, _ = oracle.grad(cnf, xr, with_abs=True)
    x1 = x.clone()
    l1, u1 = c.step(x1, 1, trace=True)
    torch.cuda.synchronize()
    check_loss(l1[0], loss, cnf, case)
    check_counts(u1[0], oracle.unsat(cnf, xr), case)
    check_update(x1, oracle.step_sgd(xr, g, c.lr), xr, R, case)
