"""Batches of few large members (each has the scan blocks a single problem has)
and of many members whose tiles alone fill their share of the scan blocks (one
slice per tile), against single runs."""
import time

import numpy as np
import pytest

from paper_2609_30533_amd import problems, scenes
from tests import test_gpu_batch
from tests.gpu_util import banner, torch_cuda

pytestmark = pytest.mark.gpu


def _large(workload, seed, batch):
    def make(attempt):
        prob = scenes.WORKLOADS[workload](seed, attempt=attempt)
        if workload == "arm7rr":
            prob.wp[8:, :, 1] += 3.0  # random configurations are rarely free among all of them
        return prob

    prob, _ = scenes.redraw_until(make, problems.start_goal_ok, 64)
    prob.params.batch, prob.params.cap_fwd, prob.params.cap_bwd = batch, 1 << 17, 1 << 13
    return prob


def test_large_members(oracle_lib):
    probs = [_large("arm6", s, 4096) for s in (5, 6, 7)] + [_large("arm7rr", s, 8192) for s in (5, 6)]
    test_gpu_batch._batch_vs_single(oracle_lib, probs, "large members")


def test_one_slice_per_tile():
    """100 members of 129 pools: more tiles than a member's share of the blocks."""
    from paper_2609_30533_amd.lib import Batch, Problem
    torch = torch_cuda()
    prob = scenes.disc2d(2, params=scenes.Params(variant=1, n_groups=128))
    prob.params.batch, prob.params.cap_fwd, prob.params.cap_bwd = 2048, 1 << 14, 1 << 8
    banner("100 members of 129 pools")
    mem = [Problem(prob, problem_id=i) for i in range(100)]
    batch = Batch(mem, iters_per_launch=4)
    batch.iterate(12)
    for i in (0, 1, 50, 99):
        one = Problem(prob, problem_id=i)
        one.iterate(12)
        torch.cuda.synchronize()
        (a, ia), (b, ib) = test_gpu_batch._state(one), test_gpu_batch._state(mem[i])
        assert ia["iter"] == ib["iter"] == 12 and a["counts"][0] > 2048
        for k in a:
            assert np.array_equal(a[k], b[k]), (i, k)
    batch.close()


@pytest.mark.parametrize("workload,B", [("arm6", 4096), ("arm7rr", 8192)])
def test_batch_of_one_is_not_much_slower(workload, B):
    """1.7 and 4.3 times a single problem's iterations with 96 scan blocks."""
    from paper_2609_30533_amd.lib import Batch, Problem
    torch = torch_cuda()
    prob = _large(workload, 5, B)

    def best(reset, run):
        t = []
        for _ in range(4):
            reset()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            run()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t) / 32 * 1e6

    one, mem = Problem(prob), Problem(prob)
    batch = Batch([mem], iters_per_launch=4)
    t1 = best(one.reset, lambda: one.iterate(32))
    t2 = best(mem.reset, lambda: batch.iterate(32))
    banner("%s: single %.1f, batch of one %.1f us per iteration" % (workload, t1, t2))
    assert t2 <= 1.45 * t1
    batch.close()
