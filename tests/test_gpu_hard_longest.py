"""Which form a Gumbel step takes by the longest clause, the restarts and the
variables: bit planes (one variable-pass launch) up to the limit, the float
passes (a gradient and an update) above it; both against the oracle, with
clauses of 0 literals up to the longest among those of three."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import from_oracle, say, to_oracle

pytestmark = pytest.mark.gpu


def _formula(n, k):
    r = np.random.default_rng(k)
    lens = [3] * (2 * n) + list(range(k + 1)) * 3 + [k] * 5
    out = [[int(a) * (1 if s else -1) for a, s in zip(r.integers(1, n + 1, w), r.random(w) < 0.5)]
           for w in lens]
    return I.from_clauses(out, n=n)


@pytest.mark.parametrize("n,R,longest", [
    (200, 15, 3), (200, 64, 3), (999, 33, 3), (1000, 15, 3), (1000, 16, 4), (1000, 64, 4), (16383, 64, 4),
    (16384, 32, 4), (16384, 33, 8), (200, 65, 8), (200, 500, 8), (4095, 128, 8), (4096, 128, 16), (8191, 65, 16),
    (8192, 65, 24), (2048, 1000, 32), (4096, 500, 32), (8192, 512, 64)])
@pytest.mark.parametrize("over", [0, 1])
def test_form(n, R, longest, over):
    k = longest + over
    say(f"[hard] longest {k} n={n} R={R}")
    cnf = _formula(n, k)
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
