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


@pytest.mark.parametrize("W,n,opacity,kw", [
    (320, 1, (0.9, 1.0), {}), (320, 2, (0.1, 0.5), {}), (320, 63, (0.01, 0.05), {}),
    (320, 64, (0.01, 0.05), {}), (320, 65, (0.02, 0.2), {}), (320, 129, (0.01, 0.2), {}),
    (333, 66, (0.02, 0.2), {}), (320, 40, (0.9, 1.0), {}), (333, 31, (0.3, 1.0), {}),
    (320, 50, (0.05, 1.0), {"alpha_min": 1.0 / 255.0}),
])
def test_backward_entry_modes(P, orc, W, n, opacity, kw):
    """Gradients where every pixel counts an entry or only some do, with and
    without alphas near the clamp, for odd and even list lengths around the
    64-entry batches, on whole and partial tiles: 1e-3 normwise per attribute
    group."""
    H = 320
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), W, H, 60.0)
    gf = S.random_gaussians(n, cam, 17 * n + W, depth=(4.0, 9.0), scale=(0.4, 3.0), margin=0.0,
                            opacity=opacity)
    say("composite backward", W, H, n, opacity, kw)
    prm_o = orc.params_array(**kw)
    ref = orc.rasterize(gf, cam, prm_o)
    dimg = np.random.default_rng(n).standard_normal((3, H, W)).astype(np.float32)
    dproj = orc.composite_backward(ref["pj"], ref["bs"], cam, prm_o, dimg.astype(np.float64))
    want = orc.project_backward(gf.astype(np.float64), ref["pj"], cam, prm_o, dproj)
    vb = P.ViewBuffers(n, 1, W, H, max(1, ref["bs"]["n_rect_pairs"]), gauss_capacity=n)
    vb.gauss.copy_(torch.as_tensor(gf).cuda())
    vb.gauss_count.fill_(n)
    prm = P.raster_params(train=True, **kw)
    vb.rasterize(P.make_camera(cam), prm)
    vb.rasterize_bwd(P.make_camera(cam), prm, torch.as_tensor(dimg).cuda())
    torch.cuda.synchronize()
    got = _np(vb.dgauss).astype(np.float64)
    for a, b in ((0, 3), (3, 6), (6, 10), (10, 11), (11, 14)):
        assert np.linalg.norm(got[a:b] - want[a:b]) <= 1e-3 * np.linalg.norm(want[a:b]), (a, b)


@pytest.mark.parametrize("W", [320, 336])
@pytest.mark.parametrize("n,opacity,t_min", [(9, (0.9, 1.4), -0.05), (40, (0.6, 1.4), -0.2),
                                             (130, (0.3, 1.4), -10.0)])
def test_negative_transmittance(P, orc, W, n, opacity, t_min):
    """alpha_max > 1 with t_min < 0: pixels blend on with T < 0.  Bars of the
    first test."""
    H = 320
    kw = {"alpha_max": 1.5, "t_min": t_min}
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), W, H, 60.0)
    gf = S.random_gaussians(n, cam, 31 * n + W, depth=(4.0, 9.0), scale=(0.4, 3.0), margin=0.0,
                            opacity=opacity)
    say("composite T < 0", W, H, n, opacity, t_min)
    ref = orc.rasterize(gf, cam, orc.params_array(**kw), weights=True)
    assert (ref["T"] < 0).any()
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


def test_scattered_stops(P, orc):
    """Lists of several hundred small Gaussians each, so that pixels get done one
    here, one there: in most groups of entries, several of a lane in one group.
    Every entry count equal but for the pixels whose stop decision is within
    rounding; other bars of the first test."""
    W, H, n = 480, 352, 120000
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), W, H, 60.0)
    gf = S.random_gaussians(n, cam, 11, depth=(4.0, 9.0), scale=(0.01, 0.06), margin=0.0,
                            opacity=(0.05, 1.0))
    say("composite scattered stops")
    ref = orc.rasterize(gf, cam, orc.params_array())
    stops = ref["last"][:H, :W].astype(np.int64)
    length = (ref["bs"]["ranges"][:, 1].astype(np.int64) - ref["bs"]["ranges"][:, 0]).reshape(H // 16, W // 16)
    done = stops < np.kron(length, np.ones((16, 16), np.int64))
    tile = stops[160:176, 160:176][done[160:176, 160:176]]
    assert len(set(((tile - 1) // 8).tolist())) >= 20  # groups of one tile in which a pixel stops
    for order in (False, True):
        vb = P.ViewBuffers(n, 1, W, H, ref["bs"]["n_rect_pairs"], gauss_capacity=n)
        vb.gauss.copy_(torch.as_tensor(gf).cuda())
        vb.gauss_count.fill_(n)
        vb.rasterize(P.make_camera(cam), P.raster_params(tile_order=order))
        torch.cuda.synchronize()
        same = _np(vb.last) == ref["last"]
        assert same.mean() >= 0.999
        assert np.abs(_np(vb.rgb) - ref["img"])[:, same].max() <= 1e-4
        assert np.abs(_np(vb.T) - ref["T"])[same].max() <= 1e-4
