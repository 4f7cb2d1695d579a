"""The composite at the edges of its groups of 8 entries and batches of 64, on
an image of the most tiles that take the eight-wave blocks (400) and one of
more: lists of every such length, pixels that stop inside a group, alphas at
the clamp, alpha_max > 1 (T may go negative) and a t_min above 1 or of 0.
Against the oracle at the bars of the other rasterizer tests (1e-4 on image and
transmittance; entry counts equal but for 0.1 % of the pixels, whose stop
decision lies within rounding of t_min; weights 2e-4 relative)."""

import numpy as np
import pytest

from synth import scenes as S
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2403_17898_amd as P
    P.lib()
    return P


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("W", [320, 336])
@pytest.mark.parametrize("n,opacity,kw", [
    (1, (0.9, 1.0), {}), (7, (0.5, 0.95), {}), (8, (0.5, 0.95), {}), (9, (0.9, 1.0), {}),
    (63, (0.02, 0.2), {}), (64, (0.02, 0.2), {}), (65, (0.3, 1.0), {}), (129, (0.01, 0.1), {}),
    (200, (0.02, 0.15), {}), (73, (0.05, 1.0), {"alpha_min": 1.0 / 255.0}),
    (40, (0.6, 1.4), {"alpha_max": 1.5}), (40, (0.6, 1.0), {"alpha_max": 1.0}),
    (20, (0.1, 0.9), {"t_min": 2.0}), (70, (0.1, 0.9), {"t_min": 0.0}),
])
def test_lists_and_stops(P, orc, W, n, opacity, kw):
    H = 320
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), W, H, 60.0)
    gf = S.random_gaussians(n, cam, 31 * n + W, depth=(4.0, 9.0), scale=(0.4, 3.0), margin=0.0,
                            opacity=opacity)
    say("composite", W, H, n, opacity, kw)
    ref = orc.rasterize(gf, cam, orc.params_array(**kw), weights=True)
    for log in (False, True):
        vb = P.ViewBuffers(n, 1, W, H, max(1, ref["bs"]["n_rect_pairs"]), gauss_capacity=n,
                           log_weights=log)
        vb.gauss.copy_(torch.as_tensor(gf).cuda())
        vb.gauss_count.fill_(n)
        vb.rasterize(P.make_camera(cam), P.raster_params(train=True, **kw))
        torch.cuda.synchronize()
        same = _np(vb.last) == ref["last"]
        assert same.mean() >= 0.999
        assert np.abs(_np(vb.rgb) - ref["img"])[:, same].max() <= 1e-4
        assert np.abs(_np(vb.T) - ref["T"])[same].max() <= 1e-4
        if log:
            np.testing.assert_allclose(_np(vb.gauss_w).astype(np.float64), ref["weights"],
                                       rtol=2e-4, atol=2e-4 * np.abs(ref["weights"]).max())
