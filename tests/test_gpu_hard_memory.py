"""What a handle holds for the Gumbel step on bit planes: the records (8
bytes an occurrence), the bits, the chunks' unsat rows and the chunk tables,
and the noise where it is drawn; nothing of what building them needed.  The
float passes hold the noise only."""
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [True, False])
def test_tables(given):
    say(f"[hard memory] given={given}")
    n, R = 1000, 64
    cnf = I.planted_ksat(n, 4000, 3, seed=1)
    prob = Problem(cnf, R, lr=0.1)
    d = torch.randn((n, R), device="cuda")
    noise = torch.randn((1, n, R), device="cuda") if given else None
    before = prob.info()["device_bytes"]
    for _ in range(2):
        prob.gumbel_step(d, 1, seed=1, noise=noise, trace=True)
    torch.cuda.synchronize()
    chunks = (n + 63) // 64  # 64 variables a workgroup's trip, one word of restarts
    want = 8 * cnf.L + 8 * n + 4 * chunks * R + 8 * chunks + 4 * 2 + (0 if given else 4 * n * R)
    assert prob.info()["device_bytes"] - before == want


def test_float_passes():
    n, R = 1000, 64
    cnf = I.from_clauses([[i + 1, 1000] for i in range(300)], n=n)  # 300 occurrences of one variable
    prob = Problem(cnf, R, lr=0.1)
    d = torch.randn((n, R), device="cuda")
    before = prob.info()["device_bytes"]
    prob.gumbel_step(d, 1, seed=1, trace=True)
    torch.cuda.synchronize()
    assert prob.info()["device_bytes"] - before == 4 * n * R
