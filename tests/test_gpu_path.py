"""The incumbent's path and a reset state: chains up to and beyond what the
pinned result holds, read by several threads at once, and the roots that a reset
writes."""
import threading

import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,nb", [(1, 1), (1, 127), (64, 64), (128, 1), (500, 37)])
def test_path_of_given_chains(nf, nb):
    from paper_2609_30533_amd.lib import Problem
    torch_cuda()
    banner("path of chains %d + %d" % (nf, nb))
    prob = scenes.disc2d(0)
    prob.params.cap_fwd, prob.params.cap_bwd = 1024, 256
    gp = Problem(prob)
    total = 1024 + prob.params.n_groups * 256
    x = np.random.default_rng(nf).random((total, 3), dtype=np.float32)
    counts = np.zeros(1 + prob.params.n_groups, np.int64)
    counts[0], counts[1] = nf, nb
    parent = np.full(total, -1, np.int32)
    # every chain node is its predecessor's child, in a shuffled order of ids
    f = np.r_[0, 1 + np.random.default_rng(1).permutation(nf - 1)]
    b = 1024 + np.r_[0, 1 + np.random.default_rng(2).permutation(nb - 1)]
    parent[f[1:]], parent[b[1:]] = f[:-1], b[:-1]
    z = np.zeros(total, np.float32)
    gp.import_state(counts, x, parent, z, z, 7.0, 3.0, f[-1], b[-1], 5)
    expect = np.r_[x[f], x[b[::-1]]].astype(np.float64)
    got = [None] * 4

    def read(k):
        got[k] = [gp.path() for _ in range(8)]

    threads = [threading.Thread(target=read, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for paths in got:
        for p in paths:
            assert np.array_equal(p["states"], expect)
            assert p["U"] == 7.0 and p["C"] == 3.0


@pytest.mark.parametrize("name", ["disc2d", "arm7rr"])
def test_reset_writes_the_fresh_state(name):
    from paper_2609_30533_amd.lib import Problem
    torch_cuda()
    banner("reset %s" % name)
    prob = getattr(scenes, name)(3)
    prob.params.batch, prob.params.cap_fwd, prob.params.cap_bwd = 256, 4096, 512
    gp = Problem(prob)
    first = gp.export()
    assert first["counts"][0] == 1 and np.array_equal(first["x"][0, :prob.d], scenes.f32(prob.q_start))
    assert first["x"][0, prob.d] == 0.0
    gp.iterate(4)
    gp.reset()
    again = gp.export()
    for k in ("counts", "x", "parent", "cost", "rootT"):
        n = first["counts"]
        if k == "counts":
            assert np.array_equal(first[k], again[k])
            continue
        # the live nodes of every pool (one root each)
        base = np.r_[0, prob.params.cap_fwd + prob.params.cap_bwd * np.arange(len(n) - 1)]
        live = base[n > 0]
        assert np.array_equal(np.asarray(first[k])[live], np.asarray(again[k])[live])
        if k == "x" and name == "arm7rr":
            assert len(live) > 1
            for i, t in zip(live[1:], first["rootT"][live[1:]]):
                assert np.array_equal(first["x"][i], np.r_[scenes.f32(prob.q_goal), t].astype(np.float32))
