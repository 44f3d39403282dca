"""The straight-through Gumbel step on bit planes against the oracle at the
same logit differences and noise: loss and unsat counts exactly, the new
differences within the bound of the other Gumbel tests.

The cases lie where the counting can go wrong: words of 64 restarts and the
lanes a wave gives them (1 to 16), 63 | 64 and 255 | 256 occurrences of one
variable (planes; the float path from 256 on), the unsat counters' overflow,
clauses of 1, 2, 3 and more literals, repeated literals, empty clauses and
formulas, and given noise."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import from_oracle, say, to_oracle

pytestmark = pytest.mark.gpu


def _lengths(n, m, seed):
    r = np.random.default_rng(seed)
    out = []
    for k in r.integers(0, 12, m):
        v = r.integers(1, n + 1, int(k))
        out.append([int(a) * (1 if s else -1) for a, s in zip(v, r.random(int(k)) < 0.5)])
    return I.from_clauses(out, n=n)


def _star(occ):
    """Variable 1 in `occ` clauses, first and negated in every other one."""
    out = []
    for i in range(occ):
        a = 1 if i % 3 else -1
        c = [a, 2 + i % 7, -(9 + i % 5)]
        out.append(c if i % 2 else c[::-1])
    return I.from_clauses(out, n=14)


CASES = {
    "planted": lambda: I.planted_ksat(301, 1280, 3, seed=5),
    "lengths": lambda: _lengths(60, 300, 6),
    "star63": lambda: _star(63),
    "star64": lambda: _star(64),
    "star255": lambda: _star(255),
    "star256": lambda: _star(256),
    "batch": lambda: I.concat([_lengths(20 + 7 * i, 50 + i, i) for i in range(9)] +
                              [I.from_clauses([[], []], n=2), I.from_clauses([], n=3)]),
}


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("R", [1, 64, 65, 130, 500, 1030])
@pytest.mark.parametrize("case", list(CASES))
def test_step_against_oracle(case, R, given):
    say(f"[hard] {case} R={R} given={given}")
    cnf = CASES[case]()
    prob = Problem(cnf, R, optimizer="adam", lr=0.5)
    rng = np.random.default_rng(R)
    d = from_oracle(rng.normal(size=(R, cnf.n)))
    st = prob.new_opt_state(d)
    for t in range(2):
        d0, mom, vel = to_oracle(d, R), to_oracle(st[0], R), to_oracle(st[1], R)
        noise = prob.gumbel_noise(77, t)
        lt, ut = prob.gumbel_step(d, 1, opt_state=st, seed=77, step0=t, tau=0.75, trace=True,
                                  noise=noise[None].contiguous() if given else None)
        torch.cuda.synchronize()
        ref = oracle.gumbel_step(cnf, d0, to_oracle(noise, R), tau=0.75, lr=prob.lr,
                                 b1=float(np.float32(0.9)), b2=float(np.float32(0.999)),
                                 eps=float(np.float32(1e-8)), t=t + 1, adam=True, mom=mom, vel=vel)
        assert np.array_equal(ut[0].cpu().numpy(), ref["unsat"])
        assert np.array_equal(lt[0].cpu().numpy(), ref["loss"].astype(np.float32))
        got, want = to_oracle(d, R), ref["d"]
        tol = 1e-5 * np.abs(want - d0) + 2e-6 * 0.5 + 2.0 ** -23 * np.abs(want)
        assert np.all(np.abs(got - want) <= tol)


def test_untraced_and_several_steps():
    """Steps without traces and several steps a call give the same states."""
    cnf = CASES["planted"]()
    a = Problem(cnf, 200, optimizer="sgd", lr=0.1)
    x = from_oracle(np.random.default_rng(1).normal(size=(200, cnf.n)))
    y = x.clone()
    a.gumbel_step(x, 4, seed=3, trace=False)
    for t in range(4):
        a.gumbel_step(y, 1, seed=3, step0=t, trace=True)
    torch.cuda.synchronize()
    assert torch.equal(x, y)


def test_noise_equals_fp64_logarithm():
    """The drawn noise is the FP64 logarithm of u / (1 - u) rounded once, at
    a million of the 2^24 values of u."""
    prob = Problem(I.planted_ksat(4000, 16000, 3, seed=9), 256)
    l = prob.gumbel_noise(0xABCDEF, 3)
    torch.cuda.synchronize()
    assert np.array_equal(to_oracle(l, 256).astype(np.float32),
                          np.asarray(oracle.gumbel_noise(0xABCDEF, 3, 4000, 256), np.float32))
