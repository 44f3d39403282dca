"""The loss-only pass over its instances: clauses in flight a slot and the
tail of a clause change with the lanes of an item, the restarts of a lane and
the longest clause (3 | 4, 8 | 9 literals); tails of one to four literals, and
clauses long enough for several trips.  Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import check_loss, say, to_oracle

pytestmark = pytest.mark.gpu


def _formula(kmax):
    """Clauses of 0 to 3 and of up to kmax literals, the first and last clause
    of the longest kind."""
    r = np.random.default_rng(kmax)
    lens = np.concatenate([[kmax], r.integers(0, 4, 200), r.integers(max(kmax - 4, 0), kmax + 1, 117), [kmax]])
    out = []
    for k in lens:
        v = r.integers(1, 151, int(k))
        out.append([int(a) * (1 if s else -1) for a, s in zip(v, r.random(int(k)) < 0.5)])
    return I.from_clauses(out, n=150)


@pytest.mark.parametrize("R", [1, 3, 7, 9, 16, 17, 20, 30, 33, 64, 66, 100, 130, 132, 260])
@pytest.mark.parametrize("kmax", [3, 4, 7, 8, 9, 70])
def test_loss(kmax, R):
    say(f"[loss] longest {kmax} R={R}")
    cnf = I.concat([_formula(kmax), _formula(kmax), I.from_clauses([[]], n=1)])
    prob = Problem(cnf, R)
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::3] = (x[::3] * 1.5 - 0.25).clamp(0, 1)
    loss = prob.loss(x)
    torch.cuda.synchronize()
    check_loss(loss, oracle.grad(cnf, to_oracle(x, R), with_abs=True)[0], cnf, f"{kmax} {R}")
