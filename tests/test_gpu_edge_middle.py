"""The one-kernel edge check in launches of middling size, where a block's waves
share its edges: against the chunked path at the sizes where the launch shape
changes, with short, long and mixed edges, waypoint times of their own, and in a
captured graph; and not slower than the chunked path, which it stands for."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _scene(workload, own_times=False, h_div=1):
    prob = scenes.WORKLOADS[workload](5)
    prob.params.cap_fwd, prob.params.cap_bwd = 256, 64
    prob.params.h /= h_div
    if workload == "arm7rr":
        prob.wp[8:, :, 1] += 3.0  # most obstacles aside, so that many edges are free
    if own_times:
        rng = np.random.default_rng(1)
        for o in range(prob.n_obs):
            t = prob.wp[o, :, 0]
            prob.wp[o, 1:-1, 0] = np.sort(scenes.f32(rng.uniform(t[0], t[-1], len(t) - 2)))
    return prob


def _mixed_edges(prob, E, seed):
    """Short edges with long free ones at random places among them."""
    xa, xb = scenes.synthetic_edges(prob, E, seed=seed)
    ya, yb = scenes.synthetic_edges(prob, max(E // 20, 2), seed=seed + 1, bridge_mix=True)
    at = np.random.default_rng(seed).choice(E, size=len(ya), replace=False)
    xa[at], xb[at] = ya, yb
    return xa, xb


def _pair(prob):
    from paper_2609_30533_amd.lib import Problem
    one, chunked = Problem(prob), Problem(prob)
    chunked.set_tuning(lanes_check=32)
    return one, chunked


def _compare(prob, xa, xb, what):
    torch = torch_cuda()
    one, chunked = _pair(prob)
    da, db = to_dev(xa), to_dev(xb)
    E = len(xa)
    banner("edge shapes %s: %d edges" % (what, E))
    ref_free, ref_hit = chunked.check_edges(da, db)
    free = torch.full((E,), 7, dtype=torch.uint8, device="cuda")
    hit = torch.full((E,), -7, dtype=torch.int32, device="cuda")
    if E <= 65536:
        one.check_edges_noalloc(da, db, free, hit)
        torch.cuda.synchronize()
        assert torch.equal(free, ref_free) and torch.equal(hit, ref_hit)
    free2, hit2 = one.check_edges(da, db)
    assert torch.equal(free2, ref_free) and torch.equal(hit2, ref_hit)
    return ref_free


@pytest.mark.parametrize("workload", ["arm6", "arm7rr", "arm6static", "disc2d"])
@pytest.mark.parametrize("E", [257, 512, 513, 768, 769, 1025, 1166, 2049, 2560, 2561, 4097, 8192, 8193, 49152, 49153])
def test_shapes_match_chunked(workload, E):
    prob = _scene(workload)
    _compare(prob, *scenes.synthetic_edges(prob, E, seed=E, bridge_mix=E % 2 == 1), workload)


@pytest.mark.parametrize("workload", ["arm6", "arm7rr", "arm6static", "disc2d"])
@pytest.mark.parametrize("E", [300, 1500, 9000, 20011, 60000])
def test_long_edges_among_short_ones(workload, E):
    """A tenth of the step: free edges of hundreds to thousands of states."""
    prob = _scene(workload, h_div=10)
    free = _compare(prob, *_mixed_edges(prob, E, E), "long " + workload)
    assert 0 < int(free.sum()) < E


@pytest.mark.parametrize("workload", ["arm6", "arm7rr", "arm6static"])
@pytest.mark.parametrize("E", [700, 3000, 12000])
def test_own_waypoint_times(workload, E):
    prob = _scene(workload, own_times=True)
    _compare(prob, *scenes.synthetic_edges(prob, E, seed=E, bridge_mix=True), "own times " + workload)


@pytest.mark.parametrize("E", [700, 2000, 20000])
def test_captured_after_a_call_of_another_size(E):
    """Nothing is allocated on the way, whatever sizes were called before."""
    from paper_2609_30533_amd.lib import Problem
    torch = torch_cuda()
    prob = _scene("arm6")
    gp = Problem(prob)
    xa, xb = scenes.synthetic_edges(prob, E, seed=3, bridge_mix=True)
    da, db = to_dev(xa), to_dev(xb)
    banner("captured check of %d edges" % E)
    gp.check_edges(da[:100].contiguous(), db[:100].contiguous())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        free, hit = gp.check_edges(da, db)
    want = gp.check_edges(da, db)
    for k in range(3):
        free.fill_(9)
        hit.fill_(-9)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(free, want[0]) and torch.equal(hit, want[1]), k
        gp.check_edges(da[:50 + k].contiguous(), db[:50 + k].contiguous())


def _us(f):
    torch = torch_cuda()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = np.inf
    for _ in range(5):
        ev[0].record()
        for _ in range(20):
            f()
        ev[1].record()
        torch.cuda.synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]) * 50.0)
    return best


@pytest.mark.parametrize("workload,own_times,h_div,E,bridge", [
    ("arm7rr", False, 1, 700, True), ("arm7rr", False, 1, 3000, False), ("arm6static", False, 1, 6000, True),
    ("arm7rr", False, 10, 700, None), ("arm7rr", False, 10, 12000, None), ("arm7rr", True, 1, 3000, False),
    ("arm7rr", True, 1, 12000, True)])
def test_not_slower_than_chunked(workload, own_times, h_div, E, bridge):
    """A single wave per edge took 1.3 to 3 times as long as the chunked kernels here."""
    prob = _scene(workload, own_times, h_div)
    xa, xb = _mixed_edges(prob, E, 3) if bridge is None else scenes.synthetic_edges(prob, E, seed=7, bridge_mix=bridge)
    one, chunked = _pair(prob)
    da, db = to_dev(xa), to_dev(xb)
    t1, t2 = _us(lambda: one.check_edges(da, db)), _us(lambda: chunked.check_edges(da, db))
    banner("%s %d edges: one kernel %.1f us, chunked %.1f us" % (workload, E, t1, t2))
    assert t1 <= 1.15 * t2
