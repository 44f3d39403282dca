"""The sums of per-chunk loss and unsat rows (k_finalize) against the oracle:
16, 32 or 64 restarts a row of lanes, one block per formula or a formula's
rows in parts, one trip of a block or several, and formulas whose cost lies
mostly in split variables."""
import pytest
import torch

import oracle
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import check_counts, check_loss, parity_at, say, to_oracle

pytestmark = pytest.mark.gpu

CASES = {
    "planted": lambda: I.planted_ksat(5000, 21000, 3, seed=11),       # about 2,000 rows
    "tiny": lambda: I.planted_ksat(20, 84, 3, seed=12),
    "batch": lambda: I.concat([I.planted_ksat(60 + 40 * i, 240 + 160 * i, 3, seed=i)
                               for i in range(20)]),
    "hot": lambda: I.structured_mixed(3000, 12000, 3, seed=13),       # split variables
}


@pytest.mark.parametrize("R", [1, 16, 17, 32, 33, 64, 65, 200])
@pytest.mark.parametrize("case", list(CASES))
def test_row_sums(case, R):
    say(f"[finalize] {case} R={R}")
    cnf = CASES[case]()
    prob = Problem(cnf, R, schedule="general")
    x = torch.rand((cnf.n, R), generator=torch.Generator("cuda").manual_seed(R), device="cuda")
    xr = to_oracle(x, R)
    parity_at(prob, cnf, x, case)
    loss_only = prob.loss(x)
    x1 = x.clone()
    lt, ut = prob.step(x1, 1, trace=True)
    torch.cuda.synchronize()
    loss = oracle.grad(cnf, xr, with_abs=True)[0]
    check_loss(loss_only, loss, cnf, case)
    check_loss(lt[0], loss, cnf, case)
    check_counts(ut[0], oracle.unsat(cnf, xr), case)
