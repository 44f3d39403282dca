"""Which form a Gumbel step takes by the longest clause and the restarts: bit
planes (one variable-pass launch) up to the limit, the float passes (a
gradient and an update) above it; both against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import from_oracle, say, to_oracle

pytestmark = pytest.mark.gpu


def _formula(k):
    r = np.random.default_rng(k)
    out = [[int(a) * (1 if s else -1) for a, s in zip(r.integers(1, 201, w), r.random(w) < 0.5)]
           for w in [3] * 700 + [k] * 5]
    return I.from_clauses(out, n=200)


@pytest.mark.parametrize("R,longest", [(1, 3), (15, 3), (16, 4), (32, 4), (33, 8), (64, 8), (65, 32),
                                       (499, 32), (500, 64)])
@pytest.mark.parametrize("over", [0, 1])
def test_form(R, longest, over):
    k = longest + over
    say(f"[hard] longest {k} R={R}")
    cnf = _formula(k)
    prob = Problem(cnf, R, optimizer="sgd", lr=0.1)
    d = from_oracle(np.random.default_rng(R).normal(size=(R, cnf.n)))
    d0 = to_oracle(d, R)
    noise = prob.gumbel_noise(3, 0)
    prob.profile(True)
    lt, ut = prob.gumbel_step(d, 1, seed=3, trace=True)
    launches = prob.kernel_times()["var_pass"][0]
    assert launches == 1 if over == 0 else launches > 1
    ref = oracle.gumbel_step(cnf, d0, to_oracle(noise, R), tau=1.0, lr=prob.lr, adam=False)
    assert np.array_equal(ut[0].cpu().numpy(), ref["unsat"])
    assert np.array_equal(lt[0].cpu().numpy(), ref["loss"].astype(np.float32))
    got, want = to_oracle(d, R), ref["d"]
    assert np.all(np.abs(got - want) <= 2e-6 * np.abs(want - d0) + 2.0 ** -23 * np.abs(want))
