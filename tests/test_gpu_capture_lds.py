"""Calls whose kernels take more than 64 KB of LDS under the caller's graph
capture: the step loop that AUTO takes and the round check, replayed with
eager work between the replays."""
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2000, 30_000])
def test_capture(n):
    say(f"[capture] n={n}")
    cnf = I.planted_ksat(n, 4 * n, 3, seed=n)
    prob = Problem(cnf, 16)
    x = torch.rand((n, 16), device="cuda")
    out = [torch.empty((2, 1, 16), device="cuda"), torch.empty((2, 1, 16), dtype=torch.int32, device="cuda")]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prob.step(x, 2, trace=True, loss_trace=out[0], unsat_trace=out[1])
        check = prob.round_check(x)
    for rep in range(3):
        x0 = prob.init_state(rep)
        x.copy_(x0)
        graph.replay()
        got = [t.clone() for t in (x, *out, *check)]
        y = x0.clone()
        lt, ut = prob.step(y, 2, trace=True)
        want = (y, lt, ut) + tuple(prob.round_check(y))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)), rep
