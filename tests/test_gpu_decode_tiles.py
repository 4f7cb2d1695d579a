"""The decode where a block takes several tiles of 32 anchors (inputs read a
tile ahead, anchors two), lists that end inside a tile, and one or two passes
of Gaussians per tile, within the error bounds of the other decode test."""

import numpy as np
import pytest

from synth import scenes as S
from tests.gpu_util import decoded_field_bounds, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bf16,n,k,width", [
    (False, 1, 1, 16), (False, 33, 16, 64), (False, 16385, 2, 32), (False, 40007, 1, 16),
    (True, 31, 8, 48), (True, 65, 16, 64), (True, 32769, 2, 64), (True, 70001, 1, 16)])
def test_decode_tiles(orc, bf16, n, k, width):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17898_amd as P
    sc, cam = S.make_gradcheck_scene(seed=k, n=n, k=k, width=width)
    idx = np.random.default_rng(n).permutation(n).astype(np.int64)
    say("decode tiles", bf16, n, k, width)
    ds = P.DeviceScene.from_scene(sc)
    vb = P.ViewBuffers(n, k, 64, 64, 1 << 12)
    vb.gauss.fill_(float("nan"))
    vb.decode(ds, P.make_camera(cam), P.OCTGS_BF16 if bf16 else P.OCTGS_FP32,
              idx=torch.as_tensor(idx.astype(np.int32)).cuda(),
              count=torch.tensor([n], dtype=torch.int32).cuda())
    torch.cuda.synchronize()
    G = n * k
    assert int(vb.gauss_count.item()) == G
    got = vb.gauss[:, :G].cpu().numpy().astype(np.float64)
    ref = orc.decode(sc, idx, cam)
    assert np.all(np.abs(got - ref) <= decoded_field_bounds(sc, idx, cam, ref, bf16))
