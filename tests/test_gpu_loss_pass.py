"""The loss-only pass against the oracle: clauses of 0 to 12 literals in
batches of four, the last batch of a chunk cut short, the list sorted by the
most frequent variable (states above 32 MB) or in clause order, restart tiles
mapped to XCDs (2, 4, 8 tiles) or not, unaligned states, and formulas whose
clauses are all empty."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import check_loss, say, to_oracle

pytestmark = pytest.mark.gpu


def _lengths(n, m, seed):
    r = np.random.default_rng(seed)
    out = []
    for k in r.integers(0, 13, m):
        v = r.integers(1, n + 1, int(k))
        out.append([int(a) * (1 if s else -1) for a, s in zip(v, r.random(int(k)) < 0.5)])
    return I.from_clauses(out, n=n)


CASES = {
    "few": lambda: _lengths(9, 5, 1),
    "lengths": lambda: _lengths(400, 3001, 2),
    "sorted": lambda: _lengths(33001, 70003, 3),
    "planted": lambda: I.planted_ksat(33001, 137000, 3, seed=4),
    "empty": lambda: I.from_clauses([[], [], []], n=2),
    "batch": lambda: I.concat([_lengths(30 + i, 90, i) for i in range(5)] + [I.from_clauses([[]], n=1)]),
}


@pytest.mark.parametrize("R,ld", [(1, 1), (30, 30), (64, 67), (256, 256), (333, 333), (512, 512),
                                  (1000, 1000), (1024, 1024)])
@pytest.mark.parametrize("case", list(CASES))
def test_loss(case, R, ld):
    say(f"[loss] {case} R={R} ld={ld}")
    cnf = CASES[case]()
    prob = Problem(cnf, R)
    x = torch.rand((cnf.n, ld), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::3] = (x[::3] * 1.5 - 0.25).clamp(0, 1)
    loss = prob.loss(x)
    torch.cuda.synchronize()
    cols = sorted({0, R // 2, R - 1, min(R - 1, 255), min(R - 1, 256)})
    want = oracle.grad(cnf, to_oracle(x, R)[cols], with_abs=True)[0]
    check_loss(loss[:, cols], want, cnf, case)
