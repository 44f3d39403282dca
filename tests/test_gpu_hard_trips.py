"""The bit-plane Gumbel step where a wave takes several groups of variables
one after another, so each group's counts go through the LDS that held the
group before: against the oracle at the same differences and noise.

Sizes: a workgroup's share is above one trip from 4,096 times 64 variables at
up to 64 restarts (one and four restarts a lane), and from 4,096 times 4
variables where a wave takes 16 words."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import from_oracle, say, to_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(600_001, 1), (600_001, 4), (34_000, 1026)])
def test_several_trips_a_wave(n, R):
    say(f"[hard] n={n} R={R}")
    cnf = I.planted_ksat(n, int(3.7 * n), 3, seed=n + R)
    prob = Problem(cnf, R, optimizer="sgd", lr=0.1)
    d = from_oracle(np.random.default_rng(R).normal(size=(R, n)))
    d0 = to_oracle(d, R)
    noise = prob.gumbel_noise(5, 0)
    lt, ut = prob.gumbel_step(d, 1, seed=5, trace=True)
    torch.cuda.synchronize()
    ref = oracle.gumbel_step(cnf, d0, to_oracle(noise, R), tau=1.0, lr=prob.lr, adam=False)
    assert np.array_equal(ut[0].cpu().numpy(), ref["unsat"])
    assert np.array_equal(lt[0].cpu().numpy(), ref["loss"].astype(np.float32))
    # the step is computed in FP64 and rounded once on each side
    got, want = to_oracle(d, R), ref["d"]
    assert np.all(np.abs(got - want) <= 2e-6 * np.abs(want - d0) + 2.0 ** -23 * np.abs(want))
