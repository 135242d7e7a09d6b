"""The largest numbers of groups and slots (128 of them make 129 pools): extend
steps in lockstep with the oracle, the planner's own iterations against sample
and extend, and batches against single runs.  The last pool's counter is the
one next to the bridge buckets' counters."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests import test_gpu_batch, test_gpu_extend
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu


def _disc(variant, groups, batch):
    prob = scenes.disc2d(2, params=scenes.Params(variant=variant, n_groups=groups))
    return test_gpu_extend._small(prob, batch, 1 << 14, 1 << 9)


def _arm(groups, batch):
    prob = test_gpu_extend._small(scenes.arm7rr(2, n_obs=8), batch, 1 << 14, 1 << 9, groups)
    return prob


CASES = [("disc2d-%s-%d" % ("rr" if v else "ir", n), lambda v=v, n=n: _disc(v, n, 2048)) for v in (0, 1)
         for n in (127, 128)] + [("arm7-rr-%d" % n, lambda n=n: _arm(n, 1500)) for n in (127, 128)]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_extend_lockstep(oracle_lib, name, make):
    """Every decision that the oracle does not exempt agrees."""
    from paper_2609_30533_amd.lib import Problem
    prob = make()
    banner("extend %s" % name)
    gp, op = Problem(prob), oracle_lib.Planner(prob)
    decided = 0
    for it in range(6):
        st = test_gpu_extend._resync(gp, op, prob)
        s_dev = gp.sample(it)
        s = test_gpu_extend._to_np(s_dev)
        g = test_gpu_extend._to_np(gp.extend(s_dev))
        r = op.extend(dict(dir=s["dir"], flags=s["flags"], grp=s["grp"], T=s["T"].astype(np.float64),
                           qr=s["qr"].astype(np.float64), tr=s["tr"].astype(np.float64)))
        exempt, _ = test_gpu_extend._compare_batch(prob, s, g, r, st["counts"])
        decided += int(((s["flags"] & 1) == 0).sum()) - exempt
    assert decided > 0


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_iterations(name, make):
    test_gpu_extend.test_iterate_equals_sample_and_extend(name, make)


@pytest.mark.parametrize("batch", [64, 700])
def test_batch(oracle_lib, batch):
    probs = [_disc(v, n, batch) for v in (0, 1) for n in (127, 128)] + [_arm(n, batch) for n in (127, 128)]
    test_gpu_batch._batch_vs_single(oracle_lib, probs, "many groups, %d samples" % batch)


def test_last_pool_is_used():
    """The sampler does send workers to the last group, and they are inserted."""
    from paper_2609_30533_amd.lib import Problem
    for variant in (0, 1):
        gp = Problem(_disc(variant, 128, 4096))
        before = gp.export()["counts"][128]
        gp.iterate(6)
        assert gp.export()["counts"][128] > before, variant
        assert np.all(gp.export()["counts"] >= 0)
