"""What a handle holds for the loss pass's sorted list: one copy of the clause
offsets and literals from 32 MB of state on, and nothing of the sort."""
import pytest

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_sorted_list():
    n, m = 100_000, 1_000_000
    cnf = I.planted_ksat(n, m, 3, seed=1)
    held = {}
    for R in (80, 84, 88):  # 32.0, 33.6 and 35.2 million bytes of state
        say(f"[loss memory] R={R}")
        prob = Problem(cnf, R, validate=False)
        held[R] = prob.info()["device_bytes"]
        prob.close()
    # four more restarts cost as much in the states and partial rows as the
    # four after them; the rest is the list
    assert held[84] - held[80] - (held[88] - held[84]) == 4 * (m + 1) + 4 * cnf.L
