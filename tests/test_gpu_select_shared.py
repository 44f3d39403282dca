"""Selections that share a handle's workspace: on two streams at once, with a
workspace that grows, and under graph capture (replayed between eager calls);
and confidences that are NaN or negative, whose order is that of their bits."""
import numpy as np
import pytest
import torch

from paper_2603_28796_amd import inputs as I
from paper_2603_28796_amd.galsat import Problem
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _cnf(sizes):
    return I.concat([I.from_clauses([[1]], n=n) for n in sizes])


def _want(conf, cnf, count, highest):
    """Ids by the bits of the confidence, ties to the lower id, in order."""
    out = []
    for row in conf:
        ids = []
        for f in range(cnf.F):
            v0, v1 = cnf.formula_var_begin[f], cnf.formula_var_begin[f + 1]
            b = row[v0:v1].view(np.uint32).astype(np.int64)
            order = np.lexsort((np.arange(v1 - v0), -b if highest else b))
            ids.append(v0 + np.sort(order[:min(count, v1 - v0)]))
        out.append(np.concatenate(ids))
    return np.stack(out)


@pytest.mark.parametrize("sizes", [[100_000], [30_000, 17, 9_000]])
def test_two_streams(sizes):
    say(f"[select] two streams {sizes}")
    cnf = _cnf(sizes)
    prob = Problem(cnf, 1)
    conf = [torch.rand((20, cnf.n), generator=torch.Generator("cuda").manual_seed(i), device="cuda")
            for i in range(2)]
    count = [40, 25] if cnf.F > 1 else [40, 40]  # other offsets on the other stream
    want = [_want(c.cpu().numpy(), cnf, k, True) for c, k in zip(conf, count)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for rep in range(10):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got.append((i, prob.select_vars(conf[i], highest=True, frac=0.0, min_count=count[i])[1]))
    torch.cuda.synchronize()
    for i, ids in got:
        assert np.array_equal(ids.cpu().numpy(), want[i]), i


def test_workspace_grows():
    """13 parts of 50 keys a candidate; only the largest workspace is held."""
    say("[select] workspace")
    cnf = _cnf([100_000])
    prob = Problem(cnf, 1)
    conf = torch.rand((100, cnf.n), generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    before = prob.info()["device_bytes"]
    for num in (10, 100, 5):
        _, ids = prob.select_vars(conf[:num], highest=False, frac=0.0, min_count=50)
        assert np.array_equal(ids.cpu().numpy(), _want(conf[:num].cpu().numpy(), cnf, 50, False))
    assert prob.info()["device_bytes"] - before == 8 * 13 * 50 * 100


@pytest.mark.parametrize("sizes", [[100_000], [30_000, 17, 9_000]])
def test_capture(sizes):
    say(f"[select] capture {sizes}")
    cnf = _cnf(sizes)
    prob = Problem(cnf, 1)
    conf = torch.rand((3, cnf.n), device="cuda")
    prob.select_vars(conf, frac=0.0, min_count=30)  # the offsets' allocation
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _, ids = prob.select_vars(conf, highest=True, frac=0.0, min_count=30)
    for rep in range(3):
        conf.copy_(torch.rand((3, cnf.n), generator=torch.Generator("cuda").manual_seed(rep), device="cuda"))
        prob.select_vars(conf, highest=False, frac=0.0, min_count=7)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), _want(conf.cpu().numpy(), cnf, 30, True)), rep


@pytest.mark.parametrize("count", [1, 40, 600])
@pytest.mark.parametrize("sizes", [[100_000], [70, 20_000]])
def test_bits_order(sizes, count):
    say(f"[select] NaN {sizes} {count}")
    cnf = _cnf(sizes)
    prob = Problem(cnf, 1)
    r = np.random.default_rng(count)
    conf = r.choice(np.float32([0.5, 0.75, 1.0, 0.0, -0.0, -1.0, np.inf, -np.inf, np.nan]), (2, cnf.n))
    conf[:, ::3] = r.random((2, len(conf[0, ::3])), dtype=np.float32)
    conf[1, 5:60] = np.uint32(0xffc00001).view(np.float32)  # NaN with the sign set
    conf = np.ascontiguousarray(conf, dtype=np.float32)
    dev = torch.from_numpy(conf).cuda()
    for highest in (True, False):
        _, ids = prob.select_vars(dev, highest=highest, frac=0.0, min_count=count)
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), _want(conf, cnf, count, highest)), highest
