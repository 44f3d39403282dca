"""Variable chunks of formula batches on the single pass: the floor on a
chunk's cost leaves several rounds of workgroups on the chip (2,048 at once),
and the results are the oracle's."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import parity_at, say

pytestmark = pytest.mark.gpu


def _batch(F, lo, hi):
    r = np.random.default_rng(F)
    return I.concat([I.planted_ksat(int(n), 4 * int(n), 3, seed=i)
                     for i, n in enumerate(r.integers(lo, hi + 1, F))])


@pytest.mark.parametrize("R,tiles", [(75, 2), (128, 1), (250, 2)])
def test_single_pass_rounds(R, tiles):
    say(f"[chunks] single pass R={R}")
    cnf = _batch(64, 50, 2000)
    prob = Problem(cnf, R, schedule="general")
    assert prob.info()["var_chunks"] * tiles >= 2 * 2048
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    parity_at(prob, cnf, x, f"batch R={R}")
