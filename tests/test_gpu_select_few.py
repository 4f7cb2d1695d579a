"""Selection around the number of anchors that one block takes (4,096): lists
and counts bit-exact with the oracle, with and without transition blending."""

import numpy as np
import pytest

from synth import scenes as S
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1025, 3000, 4095, 4096, 4097])
def test_select_few(orc, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17898_amd as P
    sc, _ = S.make_gradcheck_scene(seed=n, n=n, k=2)
    rng = np.random.default_rng(n)
    sc.level = rng.integers(0, 5, n).astype(np.uint8)
    sc.lod_bias = rng.uniform(-0.6, 0.6, n).astype(np.float32)
    sc.n_levels = 5
    cam = S.look_at((1.5, -6.0, 0.5), (0.0, 0.0, 0.4), 64, 40, 30.0)
    ds = P.DeviceScene.from_scene(sc)
    vb = P.ViewBuffers(n, sc.k, cam.width, cam.height, 1 << 10)
    thr, rho = orc.scene_thresholds(sc)
    for blend in (False, True):
        say("select few", n, blend)
        want = orc.select(sc, cam, thr, rho, blend=blend)
        vb.sel_idx.fill_(-1)
        vb.select(ds, P.make_camera(cam, lod_blend=blend), P.raster_params())
        torch.cuda.synchronize()
        assert int(vb.sel_count.item()) == len(want)
        got = vb.sel_idx.cpu().numpy()
        assert np.array_equal(got[:len(want)].astype(np.int64), want)
        assert np.all(got[len(want):] == -1)  # nothing written past the list
    assert n < 1000 or 0 < len(want) < n
