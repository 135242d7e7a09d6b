"""The network's fused kernels at the sizes where their launch shapes change:
examples per encoder tile (obstacles 1 to 64), a ragged last tile, 16 or 32 rows
per trunk block, one and several weight-gradient splits.  Bounds as in
test_gpu_mlp.py (bfloat16 operands, FP32 accumulation)."""
import numpy as np
import pytest

from oracle import mlp as ref
from paper_2609_30533_amd import scenes
from tests.gpu_util import banner, torch_cuda
from tests.test_gpu_mlp import ORDER, _batch, _dev, _flat, _rel, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,O", [(1, 64), (17, 64), (5, 57), (33, 33), (16, 32), (65, 21), (130, 16), (7, 3), (64, 1),
                                 (513, 2), (4097, 4)])
def test_shapes(M, O):
    from paper_2609_30533_amd.lib import Mlp
    torch = torch_cuda()
    banner("mlp shapes M=%d O=%d" % (M, O))
    K = 4
    p = ref.init_params(M + O)
    rng = np.random.default_rng(M)
    for k in p:
        if k.startswith("b"):
            p[k] = scenes.f32(rng.normal(size=p[k].shape) * 0.1).astype(np.float32)
    core, obs, mask, y, ymask, dmask, ubin = _batch(M, O, K, O)
    net = Mlp(M + 3, O)
    net.set_params(_flat(p))
    dc, do, dm, dy, dym, ddm, dub = _dev(core, obs, mask, y, ymask, dmask, ubin)
    for turn in range(2):  # the second step on used buffers
        z = net.forward(dc, do, dm)
        do2 = do.clone()
        net.loss(dy, dym, ddm, dub)
        do.zero_()  # the backward pass uses what the forward pass kept
        net.backward()
        torch.cuda.synchronize()
        do.copy_(do2)
    z = z.cpu().numpy().astype(np.float64)
    g = _unflat(net.grads(), p)
    zr, cache = ref.forward(p, core, obs, mask)
    assert _rel(z, zr) <= 1e-3, _rel(z, zr)
    _, dz = ref.loss(zr, y, ymask, dmask, ubin)
    gr = ref.backward(p, cache, dz)
    for k in ORDER:
        if np.linalg.norm(gr[k]) == 0:
            assert np.allclose(g[k], 0, atol=1e-6), k
            continue
        assert _rel(g[k], gr[k]) <= 1e-2, (k, _rel(g[k], gr[k]))
