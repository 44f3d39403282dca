"""Selections at the edges of k_select: 512 | 513 selected (ordered by
counting, or by compaction), formulas around whole sweeps of a workgroup
(16,384 values) and whole parts (8,192; a last part of one value), keys that fall into one bin of 2,048, and values far apart;
batches (device offsets) and one formula (none)."""
import numpy as np
import pytest
import torch

from oracle import handoff as H
from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

SIZES = {"one": [1], "edge": [16384], "over": [16385], "parts": [8193], "long": [120000], "wave": [63, 64, 65, 1023, 1024, 1025],
         "batch": [5, 40, 700, 3000, 20000]}


def _values(kind, n, rng):
    if kind == "near":      # one bin of the first histogram but for one value
        v = np.float32(1.0) - rng.integers(0, 3000, n).astype(np.float32) * np.float32(2.0 ** -24)
        v[0] = 0.5
    elif kind == "far":
        v = rng.choice(np.float32([0.0, 1e-45, 1e-30, 0.5, 1.0, 3e38, np.inf]), n)
    elif kind == "few":
        v = rng.choice(np.float32([0.5, 0.75, 1.0]), n)
    else:
        v = rng.uniform(0.5, 1.0, n).astype(np.float32)
    return v.astype(np.float32)


@pytest.mark.parametrize("count", [1, 7, 512, 513, 5000])
@pytest.mark.parametrize("kind", ["near", "far", "few", "spread"])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_selection_edges(sizes, kind, count):
    say(f"[select] {sizes} {kind} {count}")
    cnf = I.concat([I.from_clauses([[1]], n=n) for n in SIZES[sizes]])
    prob = Problem(cnf, 1)
    rng = np.random.default_rng(count)
    vals = np.stack([_values(kind, cnf.n, rng) for _ in range(2)])
    conf = torch.tensor(vals, device="cuda")
    for highest in (True, False):
        off, ids = prob.select_vars(conf, highest=highest, frac=0.0, min_count=count)
        torch.cuda.synchronize()
        ids = ids.cpu().numpy()
        for f in range(cnf.F):
            v0, v1 = cnf.formula_var_begin[f], cnf.formula_var_begin[f + 1]
            cnt = H.select_count(v1 - v0, 0.0, count)
            assert off[f + 1] - off[f] == cnt
            for k in range(2):
                want = v0 + H.select(vals[k, v0:v1], cnt, highest=highest)
                assert np.array_equal(ids[k, off[f]:off[f + 1]], want), (f, k, highest)


def test_candidate_runs():
    """More candidates than a thread's run: each equals the one drawn alone."""
    cnf = I.planted_ksat(70_000, 280_000, 3, seed=3)
    prob = Problem(cnf, 4)
    d = torch.randn((cnf.n, 4), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    best = torch.tensor([2], dtype=torch.int32, device="cuda")
    assign, conf = prob.candidates(d, best, num=37, seed=5)
    noise = torch.stack([prob.gumbel_noise(5, k)[:, 0] for k in range(37)])
    torch.cuda.synchronize()
    z = d[:, 2] + noise
    assert torch.equal(assign, (z > 0).to(torch.uint8))
    p = torch.sigmoid((d[:, 2].double() + noise.double()).abs()).float()
    assert torch.allclose(conf, p, rtol=1.2e-7, atol=0)
