"""The one-kernel edge check against the chunked path it is chosen over: the
same free flags and first hits, at the sizes where the launch shape changes
(waves per edge, edges per wave, a ragged last wave) and where a phase of
states ends (edges shorter and longer than several phases)."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _compare(prob, xa, xb, what):
    from paper_2609_30533_amd.lib import Problem
    torch = torch_cuda()
    prob.params.cap_fwd, prob.params.cap_bwd = 256, 64
    one, chunked = Problem(prob), Problem(prob)
    chunked.set_tuning(lanes_check=32)
    da, db = to_dev(xa), to_dev(xb)
    banner("edge paths %s: %d edges" % (what, len(xa)))
    ref_free, ref_hit = chunked.check_edges(da, db)
    free, hit = one.check_edges(da, db)
    torch.cuda.synchronize()
    assert torch.equal(free, ref_free) and torch.equal(hit, ref_hit)
    free2, none = one.check_edges(da, db, first_hit=False)
    assert none is None and torch.equal(free2, ref_free)
    return free.cpu().numpy(), hit.cpu().numpy()


@pytest.mark.parametrize("workload", ["disc2d", "arm6", "arm7rr", "arm6static"])
@pytest.mark.parametrize("E", [1, 2, 257, 513, 1024, 1025, 3073, 6200, 20011])
def test_one_kernel_matches_chunked(workload, E):
    prob = scenes.WORKLOADS[workload](5)
    if workload == "arm7rr":
        prob.wp[8:, :, 1] += 3.0  # most obstacles aside, so that many edges are free
    xa, xb = scenes.synthetic_edges(prob, E, seed=E, bridge_mix=E % 2 == 1)
    _compare(prob, xa, xb, workload)


@pytest.mark.parametrize("E", [3, 40, 1500])
def test_long_edges(E):
    """Edges of 1 to about 20000 states (beyond the widest phase)."""
    prob = scenes.disc2d(3, n_obs=2)
    prob.params.h = 5e-4
    rng = np.random.default_rng(E)
    xa, xb = scenes.synthetic_edges(prob, E, seed=E, bridge_mix=True)
    xb[:, 2] = np.minimum(xa[:, 2] + rng.uniform(0, 10, E) ** 2 / 10, 10).astype(np.float32)
    xb[0] = xa[0]
    free, hit = _compare(prob, xa, xb, "long")
    assert E < 1500 or (free.any() and not free.all())


def test_scene_at_the_size_limit():
    """A scene that fills the documented 64 KB of staged tables."""
    prob = scenes.arm6(1, n_obs=64, n_wp=31)
    prob.obs_r = scenes.f32(np.full(64, 0.03))
    for E in (5, 4100, 70000):
        xa, xb = scenes.synthetic_edges(prob, E, seed=E)
        _compare(prob, xa, xb, "large scene")
