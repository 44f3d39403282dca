"""Handles of several sizes in several threads: launches of one kernel with
different amounts of LDS above 64 KB (the step loop and the round check) give
what they give one after another."""
import threading

import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _run(prob, x0, stream, reps, out):
    try:
        with torch.cuda.stream(stream):
            for _ in range(reps):
                x = x0.clone()
                prob.step(x, 2)
                out.append((x,) + tuple(prob.round_check(x)))
        stream.synchronize()
    except Exception as e:  # reported by the test
        out.append(e)


def test_threads():
    cases = []
    for n in (1500, 1700, 1900, 2000):
        cnf = I.planted_ksat(n, 4 * n, 3, seed=n)
        cases.append((cnf, 16))
    for n in (20_000, 24_000, 30_000):  # 80 to 120 KB of words in the round check
        cases.append((I.planted_ksat(n, 4 * n, 3, seed=n), 16))
    say("[lds threads]")
    probs = [Problem(cnf, R) for cnf, R in cases]
    states = [torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(cnf.n), device="cuda")
              for cnf, R in cases]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    want = [[] for _ in cases]
    for i, p in enumerate(probs):
        _run(p, states[i], streams[i], 1, want[i])
    got = [[] for _ in cases]
    threads = [threading.Thread(target=_run, args=(p, states[i], streams[i], 20, got[i]))
               for i, p in enumerate(probs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for w, g in zip(want, got):
        assert len(g) == 20
        for r in g:
            assert not isinstance(r, Exception), r
            assert all(torch.equal(a, b) for a, b in zip(r, w[0]))
