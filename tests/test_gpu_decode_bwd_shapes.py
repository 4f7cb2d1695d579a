"""The decode backward over every hidden width it is instantiated for and
Gaussians per anchor at the edges of its output column tiles (one to three per
wave), more anchor tiles than one pass of a block takes (the inputs read ahead),
against the oracle at the bar of the other decode-backward test (1e-4
normwise)."""

import numpy as np
import pytest

from synth import scenes as S
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("width,k,n", [(16, 16, 40), (16, 1, 33), (32, 10, 47), (48, 5, 50), (48, 11, 20),
                                       (64, 12, 50), (64, 16, 31), (64, 10, 9000)])
def test_decode_backward_shapes(orc, width, k, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17898_amd as P
    sc, cam = S.make_gradcheck_scene(seed=width + k, n=n, k=k, width=width)
    idx = np.random.default_rng(n).permutation(n)[:n - n // 10].astype(np.int64)
    G = len(idx) * k
    dgauss = np.random.default_rng(k).standard_normal((14, G)).astype(np.float32)
    say("decode backward", width, k, len(idx))
    ref = orc.decode_backward(sc, idx, cam, dgauss.astype(np.float64))
    ds = P.DeviceScene.from_scene(sc)
    grads = P.SceneGrads(ds)
    vb = P.ViewBuffers(n, k, 64, 64, 1 << 12, gauss_capacity=G)
    vb.decode_bwd(ds, P.make_camera(cam), grads, dgauss=torch.as_tensor(dgauss).cuda(),
                  idx=torch.as_tensor(idx.astype(np.int32)).cuda(),
                  count=torch.tensor([len(idx)], dtype=torch.int32).cuda())
    torch.cuda.synchronize()
    for name, r in ref.items():
        got = grads.all()[name].detach().cpu().numpy().astype(np.float64).reshape(r.shape)
        assert np.linalg.norm(got - r) <= 1e-4 * np.linalg.norm(r), name
