"""What galsat_get_info says of the step loops: restarts a workgroup and
staging under AUTO as under the LDS schedule, none under the general one."""
import pytest

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule,plan,want", [
    ("auto", None, ("lds", 1, 1)), ("lds", None, ("lds", 1, 1)), ("lds", "ldsrg=8", ("lds", 8, 1)),
    ("lds", "ldsrg=2,ldsstage=0", ("lds", 2, 0)), ("auto", "cl=0", ("general", 0, 0)),
    ("general", None, ("general", 0, 0)), ("plain", None, ("plain", 0, 0))])
def test_info(schedule, plan, want):
    cnf = I.planted_ksat(200, 852, 3, seed=1)
    i = Problem(cnf, 16, schedule=schedule, plan_override=plan).info()
    assert (i["schedule"], i["lds_restarts_per_group"], i["lds_staged"]) == want
