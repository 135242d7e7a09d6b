"""The extend step's bucketed nearest-node scans, whose blocks are dealt out over
tiles and slices on the device, against single calls over the same queries: sets
of no, one and many tiles, with slices that fit the grid and that are cut to it."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make,B,steps", [("disc2d", 1, 2), ("disc2d", 257, 6), ("disc2d", 40011, 2), ("arm6", 8192, 3),
                                          ("arm7rr", 8192, 3)])
def test_bucketed_scans_agree_with_single_calls(make, B, steps):
    from paper_2609_30533_amd.lib import FLAG_SKIP, FLAG_USE_NEW, STATUS_ADVANCED, Problem
    torch = torch_cuda()
    banner("bucketed scans %s, %d samples" % (make, B))
    prob = getattr(scenes, make)(1)
    prob.params.batch = B
    rr = prob.params.variant != scenes.VARIANT_IR
    gp = Problem(prob)
    compared = 0
    for it in range(steps):
        s_dev = gp.sample(it)
        s = {k: v.cpu().numpy() for k, v in s_dev.items()}
        live = (s["flags"] & FLAG_SKIP) == 0
        if not rr:
            live &= (s["dir"] == 0) | ((s["flags"] & FLAG_USE_NEW) == 0)
        xq = np.concatenate([s["qr"], s["tr"][None]], axis=0).T.astype(np.float32)
        near = np.full(B, -2, np.int64)
        for grp in [-1] + sorted(set(s["grp"][live & (s["dir"] != 0)].tolist())):
            w = np.nonzero(live & ((s["dir"] == 0) if grp < 0 else ((s["dir"] != 0) & (s["grp"] == grp))))[0]
            if len(w) == 0:
                continue
            idx, _ = gp.nearest(torch.from_numpy(np.ascontiguousarray(xq[w])).cuda(), set_id=grp,
                                metric=1 if rr else 0, sigma=1 if grp < 0 else -1)
            near[w] = idx.cpu().numpy()
        o = {k: v.cpu().numpy() for k, v in gp.extend(s_dev).items()}
        on = (o["status"] == STATUS_ADVANCED) & (near != -2)
        assert np.array_equal(o["parent"][on], near[on])
        # nothing admissible: the worker did not advance
        assert not np.any(o["status"][near == -1] == STATUS_ADVANCED)
        compared += int(on.sum())
    assert compared > 0 or B == 1 or make == "arm7rr"
