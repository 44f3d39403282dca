"""The state copies of a step at the sizes where their loops change: below a
workgroup, one word a thread, several words a thread and a rest (from
33,554,432 values in one run), rows of one and of four restarts a lane.  The
variables no clause names keep their values bitwise, padding columns too."""
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,ld", [(3, 1, 1), (257, 1, 1), (1_025, 4, 4), (65_537, 75, 75), (460_001, 75, 75),
                                    (8_388_609, 4, 4), (70_001, 75, 80), (70_001, 64, 68), (300_001, 3, 5)])
def test_copies(n, R, ld):
    say(f"[copy] n={n} R={R} ld={ld}")
    cnf = I.from_clauses([[1, -2, 3]], n=n)
    x = torch.rand((n, ld), generator=torch.Generator("cuda").manual_seed(n), device="cuda")
    prob = Problem(cnf, R, schedule="general")
    for steps in (1, 2, 3):
        y = x.clone()
        prob.step(y, steps)
        torch.cuda.synchronize()
        assert torch.equal(y[3:], x[3:]) and torch.equal(y[:, R:], x[:, R:])
        assert not torch.equal(y[:3, :R], x[:3, :R])
