"""Insertion of an extend step against a sequential model: per pool, workers in
index order, a virtual root ahead of its first node, and what does not fit
dropped, with one and several chunks of workers per block, a single worker, and
pools that run full within a chunk and ahead of one."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make,B,cap_fwd,cap_bwd", [
    ("disc2d", 1, 1 << 14, 1 << 12), ("disc2d", 513, 1 << 14, 1 << 12), ("disc2d", 8193, 1 << 15, 1 << 14),
    ("disc2d", 20011, 1 << 16, 1 << 14), ("disc2d", 20011, 5000, 700), ("disc2d", 4096, 333, 5),
    ("arm6", 4096, 1 << 14, 1 << 12), ("arm7rr", 8192, 1 << 14, 40)])
def test_insertion_follows_the_sequential_rule(make, B, cap_fwd, cap_bwd):
    from paper_2609_30533_amd.lib import FLAG_USE_NEW, STATUS_ADVANCED, STATUS_DROPPED, Problem
    torch_cuda()
    banner("insertion %s, %d samples, capacities %d and %d" % (make, B, cap_fwd, cap_bwd))
    prob = getattr(scenes, make)(1)
    prob.params.batch, prob.params.cap_fwd, prob.params.cap_bwd = B, cap_fwd, cap_bwd
    gp = Problem(prob)
    rooted = prob.params.variant == scenes.VARIANT_IR
    inserted = 0
    for it in range(3):
        count = gp.export()["counts"].copy()
        s_dev = gp.sample(it)
        s = {k: v.cpu().numpy() for k, v in s_dev.items()}
        o = {k: v.cpu().numpy() for k, v in gp.extend(s_dev).items()}
        t = gp.export()
        base = np.r_[0, cap_fwd + cap_bwd * np.arange(len(count) - 1)]
        cap = np.r_[cap_fwd, np.full(len(count) - 1, cap_bwd)]
        at, end = count.copy(), count.copy()
        for w in np.nonzero((o["status"] == STATUS_ADVANCED) | (o["status"] == STATUS_DROPPED))[0]:
            p = 0 if s["dir"][w] == 0 else 1 + s["grp"][w]
            virt = rooted and p > 0 and bool(s["flags"][w] & FLAG_USE_NEW)
            need = 2 if virt else 1
            if at[p] + need > cap[p]:
                assert o["status"][w] == STATUS_DROPPED and o["new_idx"][w] == -1
            else:
                assert o["status"][w] == STATUS_ADVANCED
                i = base[p] + at[p] + need - 1
                assert o["new_idx"][w] == i and o["parent"][w] == t["parent"][i]
                assert np.array_equal(t["x"][i], o["xnew"][:, w])
                if virt:
                    assert t["parent"][i] == i - 1 and t["parent"][i - 1] == -1
                    assert np.array_equal(t["x"][i - 1], np.r_[scenes.f32(prob.q_goal), s["T"][w]].astype(np.float32))
                end[p] = at[p] + need
                inserted += 1
            at[p] += need
        assert np.array_equal(t["counts"], end)
    assert inserted > 0 or B == 1 or make == "arm7rr"
