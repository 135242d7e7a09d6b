"""The filtered scan against the plain one where squared times and distances
come close to the largest float: a sum that the filter forms must not hide a
node whose key is still finite."""
import numpy as np
import pytest

from paper_2609_30533_amd import scenes
from tests import test_gpu_nearest_filter as near

pytestmark = pytest.mark.gpu


def _run(x, xq, metric, what):
    prob, gp, nodes, rootT, _ = near._problem(scenes.disc2d, len(x), 64, 4)
    nodes[:len(x)] = x
    near._import(prob, gp, nodes, rootT, [len(x)] + [0] * 4)
    assert prob.v_max == 1.0
    idx, dist = near._compare(gp, xq, len(x), what, metric=metric, sigma=1)
    assert (idx >= 0).all() and np.isfinite(dist).all()
    return idx


def _queries(m):
    return np.random.default_rng(6).uniform(0, 1, size=(m, 3)).astype(np.float32)


def test_rho_of_very_early_nodes():
    """(v dt)^2 from 1.8e38 to 3.2e38, beyond 2^127; the nearest node is late in the set."""
    n = 32768
    x = np.random.default_rng(5).uniform(0, 1, size=(n, 3)).astype(np.float32)
    x[:, 2] = -np.sqrt(np.linspace(3.2e38, 1.8e38, n)).astype(np.float32)
    assert (_run(x, _queries(4111), 0, "early nodes") >= n // 2).all()


def test_configuration_distance_of_very_far_nodes():
    """Squared distances from 3.397e38 to 3.402e38, which bfloat16 rounds to infinity."""
    n = 32768
    x = np.random.default_rng(5).uniform(0, 1, size=(n, 3)).astype(np.float32)
    x[:, 0] = np.sqrt(np.linspace(3.402e38, 3.397e38, n)).astype(np.float32)
    assert (_run(x, _queries(4111), 1, "far nodes") >= n // 2).all()
