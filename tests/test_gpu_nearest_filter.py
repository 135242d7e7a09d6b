"""The filtered scan of large node sets against the plain scan it stands for:
identical indices and distances, bit for bit.  The queries are given once
together (filtered: 2^27 pairs and more) and once in groups small enough for
the plain scan."""
import math

import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


def _problem(maker, n_fwd, bwd, seed, groups=4):
    from paper_2609_30533_amd.lib import Problem
    prob = maker(2)
    p = prob.params
    p.cap_fwd, p.cap_bwd, p.n_groups = n_fwd, bwd, groups
    rng = np.random.default_rng(seed)
    total = n_fwd + groups * bwd
    x = rng.uniform(np.r_[prob.q_lo, 0], np.r_[prob.q_hi, prob.t_max], size=(total, prob.d + 1)).astype(np.float32)
    rootT = rng.uniform(prob.t_min, prob.t_max, size=total).astype(np.float32)
    return prob, Problem(prob), x, rootT, rng


def _import(prob, gp, x, rootT, counts, U=math.inf):
    n, N = len(x), prob.params.n_groups
    par = np.full(n, -1, np.int32)
    slots = (np.full(N, 5.0), np.ones(N, np.int32), np.zeros(N, np.uint32), np.zeros(N, np.int64))
    gp.import_state(np.asarray(counts, np.int64), x, par, np.zeros(n, np.float32), rootT, U, math.inf, -1, -1, 0,
                    slots)


def _compare(gp, xq, nodes, what, **kw):
    torch = torch_cuda()
    dq = to_dev(xq)
    assert len(xq) * nodes >= 1 << 27
    banner("filtered scan %s: %d queries, %d nodes" % (what, len(xq), nodes))
    idx, dist = gp.nearest(dq, **kw)
    step = max(1, ((1 << 27) // nodes - 256) // 2)
    for i in range(0, len(xq), step):
        ri, rd = gp.nearest(dq[i:i + step].contiguous(), **kw)
        assert torch.equal(ri, idx[i:i + step]), what
        assert torch.equal(rd, dist[i:i + step]), what
    return idx.cpu().numpy(), dist.cpu().numpy()


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("name,maker,n,m", [("disc", scenes.disc2d, 70001, 2100), ("arm6", scenes.arm6, 33333, 4111),
                                            ("arm7", scenes.arm7rr, 20480, 8192)])
def test_forward_tree(name, maker, n, m, metric):
    prob, gp, x, rootT, rng = _problem(maker, n, 64, 1)
    x[n // 2:n // 2 + 500] = x[:500]  # duplicates: the lowest index wins
    _import(prob, gp, x, rootT, [n] + [0] * 4)
    xq = scenes.synthetic_states(prob, m, seed=7)
    xq[:100] = x[n // 2:n // 2 + 100]  # on a node (distance 0 in configuration)
    xq[100:200, -1] = 0.0              # nothing precedes these
    idx, dist = _compare(gp, xq, n, name, metric=metric, sigma=1)
    if metric == 0:
        assert (idx[100:200] == -1).all() and (idx >= 0).mean() > 0.5
    else:
        # the duplicate's first copy, or another node at distance zero before it
        assert (idx[:100] <= np.arange(100)).all() and (dist[:100] == 0).all()


def test_backward_trees_with_hidden_ones():
    """Every backward pool in one set; trees rooted at or after U are hidden."""
    prob, gp, x, rootT, rng = _problem(scenes.arm6, 256, 12000, 2)
    _import(prob, gp, x, rootT, [256, 12000, 11000, 1, 11999], U=0.5 * (prob.t_min + prob.t_max))
    idx, _ = _compare(gp, scenes.synthetic_states(prob, 4096, seed=9), 35000, "backward", set_id=-2, metric=0, sigma=-1)
    assert (rootT[idx[idx >= 0]] < 0.5 * (prob.t_min + prob.t_max)).all() and (idx >= 0).any()


@pytest.mark.parametrize("metric", [0, 1])
def test_coordinates_the_filter_cannot_bound(metric):
    """Coordinates far from the origin, beyond the filter's range, infinite and
    NaN ones, among the nodes and the queries."""
    prob, gp, x, rootT, rng = _problem(scenes.arm6, 40000, 64, 3)
    d = prob.d
    x[1000:9000, :d] += 1000.0
    x[9000:9100, 0] = 1e18
    x[9100:9200, 1] = 3e38
    x[9200:9300, 2] = np.inf
    x[9300:9400, 3] = np.nan
    x[9400:9500, d] = np.nan
    x[9500:9600, d] = -1e25
    x[9600:9700, d] = -np.inf
    _import(prob, gp, x, rootT, [40000] + [0] * 4)
    xq = scenes.synthetic_states(prob, 4096, seed=11)
    xq[:500, :d] += 1000.0
    xq[500:600, 0] = 1e18
    xq[600:650, 1] = np.nan
    xq[650:700, d] = np.inf
    xq[700:750, d] = np.nan
    xq[750:800, d] = 1e30
    xq[800:900, :d] = x[9000:9100, :d]
    _compare(gp, xq, 40000, "odd coordinates", metric=metric, sigma=1)
