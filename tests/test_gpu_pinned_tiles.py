"""Two and four restart tiles of one formula: one launch while the state is
small or the numbering has locality, a launch per share of the cache beyond
(as many launches as tiles there).  Loss and gradient are those of the plan
without pinning, bitwise."""
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family,n,R,launches", [("planted", 30_000, 512, 1), ("planted", 30_000, 1000, 1),
                                                 ("planted", 420_000, 512, 2), ("planted", 270_000, 1000, 4),
                                                 ("mixed", 270_000, 1000, 1)])
def test_launches(family, n, R, launches):
    say(f"[pinned] {family} n={n} R={R}")
    cnf = I.planted_ksat(n, 4 * n, 3, seed=1) if family == "planted" else \
        I.structured_mixed(n, 4 * n, n // 1000, seed=1)
    x = torch.rand((n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    prob = Problem(cnf, R)
    loss, g = prob.loss_grad(x)
    prob.profile(True)
    prob.loss_grad(x)
    assert prob.kernel_times()["var_pass"][0] == launches
    prob.close()
    plain = Problem(cnf, R, plan_override="xpin=0")
    loss0, g0 = plain.loss_grad(x)
    torch.cuda.synchronize()
    assert torch.equal(loss, loss0) and torch.equal(g, g0)
