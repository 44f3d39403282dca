"""Initial states and the copies around a step: rows of 16 bytes or not,
strides above the restarts, bases off the 16-byte grid; padding columns stay
as they were, and a step gives the same states at every layout."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say, to_oracle

pytestmark = pytest.mark.gpu


def _view(n, ld, off, fill):
    """[n, ld] with its first element `off` floats into an allocation."""
    base = torch.full((n * ld + off,), fill, device="cuda")
    return base[off:].view(n, ld)


@pytest.mark.parametrize("R", [1, 3, 4, 20, 33, 64, 75, 130, 256, 260])
def test_layouts(R):
    say(f"[rows] R={R}")
    cnf = I.planted_ksat(1003, 4200, 3, seed=7)
    prob = Problem(cnf, R, schedule="general")
    ref = oracle.init_state(99, cnf.n, R)
    want = None
    for ld, off in ((R, 0), (R + 1, 0), ((R + 3) // 4 * 4, 0), ((R + 7) // 4 * 4, 0), (R, 1),
                    ((R + 3) // 4 * 4, 2)):
        x = prob.init_state(99, _view(cnf.n, ld, off, -7.0))
        torch.cuda.synchronize()
        assert np.array_equal(to_oracle(x, R), ref), (ld, off)
        for steps in (1, 2):
            prob.step(x, steps)
        torch.cuda.synchronize()
        assert bool((x[:, R:] == -7.0).all())
        got = x[:, :R].clone()
        want = got if want is None else want
        assert torch.equal(got, want), (ld, off)


def test_batch_chunks_are_balanced():
    """Many small formulas, a few large ones: each formula as by itself."""
    sizes = [30] * 40 + [700, 2100, 90]
    cnf = I.concat([I.planted_ksat(s, 4 * s, 3, seed=i) for i, s in enumerate(sizes)])
    for R in (16, 75):
        prob = Problem(cnf, R, schedule="general")
        x = prob.init_state(5)
        loss, g = prob.loss_grad(x)
        for f in (0, 39, 40, 41, 42):
            one = cnf.sub(f)
            v0, v1 = cnf.formula_var_begin[f], cnf.formula_var_begin[f + 1]
            l1, g1 = Problem(one, R, schedule="general").loss_grad(x[v0:v1].contiguous())
            assert torch.allclose(loss[f], l1[0], rtol=1e-6)
            assert torch.allclose(g[v0:v1], g1, rtol=1e-5, atol=1e-5)
