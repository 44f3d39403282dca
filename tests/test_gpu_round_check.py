"""The round check's unsat counts, best restarts and assignments against the
oracle, exactly, where its kernels change: 16, 32 and 64 restarts a word,
rows of 16 bytes or not, a formula's words in LDS (at most 32,768 of 32 bits
or 16,384 of 64) or not, clauses longer than 8, and more clauses per lane
than its counters hold."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say, to_oracle

pytestmark = pytest.mark.gpu


def _lengths(n, m, seed):
    r = np.random.default_rng(seed)
    out = []
    for k in r.integers(0, 13, m):
        v = r.integers(1, n + 1, int(k))
        out.append([int(a) * (1 if s else -1) for a, s in zip(v, r.random(int(k)) < 0.5)])
    return I.from_clauses(out, n=n)


CASES = {
    "small": lambda: I.planted_ksat(100, 420, 3, seed=1),
    "lengths": lambda: _lengths(300, 2500, 2),
    "lds64": lambda: I.planted_ksat(16384, 66000, 3, seed=3),
    "no_lds64": lambda: I.planted_ksat(16385, 66000, 3, seed=4),
    "no_lds32": lambda: I.planted_ksat(32769, 132000, 3, seed=5),
    "batch": lambda: I.concat([I.planted_ksat(50 + 900 * i, 200 + 3700 * i, 3, seed=i) for i in range(6)] +
                              [I.from_clauses([[]], n=1), I.from_clauses([], n=2)]),
}


def _check(cnf, R, ld, what):
    prob = Problem(cnf, R)
    x = torch.rand((cnf.n, ld), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    x[::5] = 0.5
    unsat, best, assign = prob.round_check(x)
    torch.cuda.synchronize()
    xr = to_oracle(x, R)
    want = oracle.unsat(cnf, xr)
    assert np.array_equal(unsat.cpu().numpy(), want), what
    bref = want.argmin(axis=1)
    assert np.array_equal(best.cpu().numpy(), bref), what
    aref = (xr[bref[cnf.formula_of_var()], np.arange(cnf.n)] > 0.5).astype(np.uint8)
    assert np.array_equal(assign.cpu().numpy(), aref), what


@pytest.mark.parametrize("R,ld", [(1, 1), (16, 16), (20, 20), (20, 23), (32, 32), (33, 33), (64, 64),
                                  (75, 75), (76, 80), (130, 132)])
@pytest.mark.parametrize("case", list(CASES))
def test_round_check(case, R, ld):
    say(f"[round check] {case} R={R} ld={ld}")
    _check(CASES[case](), R, ld, case)


def test_full_counters():
    """About 35 clauses a lane, five bits of counter."""
    cnf = I.planted_ksat(300, 1_200_000, 3, seed=6)
    R = 1024
    prob = Problem(cnf, R)
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    unsat, _, _ = prob.round_check(x)
    torch.cuda.synchronize()
    cols = [0, 1, 63, 64, 500, 1023]
    want = oracle.unsat(cnf, to_oracle(x, R)[cols])
    assert np.array_equal(unsat.cpu().numpy()[:, cols], want)
