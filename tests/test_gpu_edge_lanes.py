"""A handle that chose lanes for st_check_edges goes back to the one-kernel check
with a state split of -1: that check allocates nothing, so a call larger than
any before it can be captured."""
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workload", ["arm6", "disc2d"])
def test_split_minus_one_returns_to_the_one_kernel_check(workload):
    from paper_2609_30533_amd.lib import Problem
    torch = torch_cuda()
    prob = scenes.WORKLOADS[workload](5)
    prob.params.cap_fwd, prob.params.cap_bwd = 256, 64
    gp = Problem(prob)
    xa, xb = scenes.synthetic_edges(prob, 20011, seed=3, bridge_mix=True)
    da, db = to_dev(xa), to_dev(xb)
    banner("lanes chosen and taken back, %s" % workload)
    gp.set_tuning(lanes_check=16)
    gp.set_state_split(check=2)
    a, b = da[:300].contiguous(), db[:300].contiguous()
    few = gp.check_edges(a, b)
    gp.set_state_split(check=-1)
    again = gp.check_edges(a, b)
    assert torch.equal(few[0], again[0]) and torch.equal(few[1], again[1])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        free, hit = gp.check_edges(da, db)
    want = gp.check_edges(da, db)
    for _ in range(3):
        free.fill_(9)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(free, want[0]) and torch.equal(hit, want[1])
