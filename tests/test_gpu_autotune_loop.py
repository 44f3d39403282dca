"""The autotuner and the clause-parallel step loop: a candidate where AUTO or
the LDS schedule may take it, expressed by the plan key cl, also through the
plan cache; not one where it cannot run."""
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem, autotune
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _x(n, R):
    return torch.rand((n, R), generator=torch.Generator("cuda").manual_seed(n + R), device="cuda")


@pytest.mark.parametrize("R", [16, 100])
def test_small_problem_keeps_the_loop(R, tmp_path, monkeypatch):
    say(f"[autotune] loop R={R}")
    cnf = I.planted_ksat(200, 852, 3, seed=1)
    x0 = _x(cnf.n, R)
    assert Problem(cnf, R).info()["schedule"] == "lds"
    plan, ms = autotune(cnf, R, x0, steps=20)
    assert plan == "cl=1" and ms > 0  # ten times the speed of the general passes here
    tuned = Problem(cnf, R, plan_override=plan)
    assert tuned.info()["schedule"] == "lds"
    a, b = x0.clone(), x0.clone()
    tuned.step(a, 5)
    Problem(cnf, R).step(b, 5)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert Problem(cnf, R, plan_override="cl=0").info()["schedule"] == "general"
    monkeypatch.setenv("GALSAT_PLAN_CACHE", str(tmp_path / "plans.txt"))
    assert autotune(cnf, R, x0, steps=20)[0] == "cl=1"
    assert Problem(cnf, R).info()["schedule"] == "lds"
    # the recorded plan leaves other uses of the shape their own choice
    assert Problem(cnf, R, optimizer="adam").info()["schedule"] == "general"


def test_lds_schedule_keeps_the_loop():
    say("[autotune] lds")
    cnf = I.planted_ksat(200, 852, 3, seed=1)
    plan, _ = autotune(cnf, 64, _x(cnf.n, 64), steps=50, schedule="lds")
    assert plan == "ldsrg=0,cl=1"  # five times the speed of the other form here
    assert Problem(cnf, 64, schedule="lds", plan_override=plan).info()["lds_restarts_per_group"] == 1


def test_forced_for_many_tiny_formulas():
    """cl=1 and cl=0 where the rule takes the other form: the same states."""
    cnf = I.concat([I.planted_ksat(16, 64, 3, seed=i) for i in range(700)])
    x = _x(cnf.n, 32)
    got = []
    for plan, group in ((None, 32), ("cl=1", 1), ("cl=0", 32)):
        p = Problem(cnf, 32, schedule="lds", plan_override=plan)
        assert p.info()["lds_restarts_per_group"] == group
        y = x.clone()
        p.step(y, 3)
        got.append(y)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("case", ["long clause", "adam", "large"])
def test_not_where_it_cannot_run(case):
    say(f"[autotune] {case}")
    kw = {"optimizer": "adam"} if case == "adam" else {}
    cnf = I.planted_ksat(200, 800, 3, seed=2)
    if case == "long clause":
        cnf = I.from_clauses([list(range(1, 10))] + [[1, -2, 3]] * 5, n=20)
    if case == "large":
        cnf = I.planted_ksat(4000, 16_000, 3, seed=2)
    plan, _ = autotune(cnf, 16, _x(cnf.n, 16), steps=2, **kw)
    assert "cl=" not in plan and plan
    assert Problem(cnf, 16, plan_override="cl=1", **kw).info()["schedule"] == "general"
