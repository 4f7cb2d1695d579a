"""The rasterizer's binning (grouping by screen bin, per-bin sort, tile lists)
at the sizes where its paths change: each bin shape with partial edge bins,
rectangles around the keep mask's 64 tiles and around four bins, lists longer
than one block sorts, runs of equal depths, and an image of several grouping
bands.  Lists, ranges and counts are decisions: bit-exact with the oracle.
Images and gradients at the bars of the other rasterizer tests (1e-4 and 1e-3
normwise)."""

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


def _raster(P, cam, gf, pcap, train):
    n = gf.shape[1]
    vb = P.ViewBuffers(n, 1, cam.width, cam.height, pcap, gauss_capacity=n)
    vb.gauss.copy_(torch.as_tensor(gf).cuda())
    vb.gauss_count.fill_(n)
    prm = P.raster_params(train=train)
    vb.rasterize(P.make_camera(cam), prm)
    torch.cuda.synchronize()
    return vb, prm


def _check_lists(vb, pj, bs):
    st = vb.stats()
    assert st["sync_error"] == 0 and st["pair_overflow"] == 0
    assert st["n_visible"] == pj["n_visible"]
    assert st["n_candidates"] == bs["n_rect_pairs"] and st["n_pairs"] == bs["n_pairs"]
    tile, slot, ranges = vb.sorted_lists()
    assert np.array_equal(ranges, bs["ranges"])
    assert np.array_equal(tile, bs["tile_of"])
    assert np.array_equal(slot, bs["gid_of"])


def _check(P, orc, cam, gf, what):
    """Lists with and without the training outputs, image and gradients."""
    n, H, W = gf.shape[1], cam.height, cam.width
    prm_o = orc.params_array()
    say("bins", what, W, H, n)
    ref = orc.rasterize(gf, cam, prm_o)
    pcap = max(1, ref["bs"]["n_rect_pairs"])  # the tightest that must not overflow
    vb, _ = _raster(P, cam, gf, pcap, False)
    _check_lists(vb, ref["pj"], ref["bs"])
    assert np.abs(_np(vb.rgb) - ref["img"]).max() <= 1e-4
    vb, prm = _raster(P, cam, gf, pcap, True)
    _check_lists(vb, ref["pj"], ref["bs"])
    dimg = np.random.default_rng(n).standard_normal((3, H, W)).astype(np.float32)
    dproj = orc.composite_backward(ref["pj"], ref["bs"], cam, prm_o, dimg.astype(np.float64))
    want = orc.project_backward(gf.astype(np.float64), ref["pj"], cam, prm_o, dproj)
    vb.rasterize_bwd(P.make_camera(cam), prm, torch.as_tensor(dimg).cuda())
    torch.cuda.synchronize()
    got = _np(vb.dgauss).astype(np.float64)
    for a, b in ((0, 3), (3, 6), (6, 10), (10, 11), (11, 14)):
        assert np.linalg.norm(got[a:b] - want[a:b]) <= 1e-3 * np.linalg.norm(want[a:b]), (a, b)
    return ref


@pytest.mark.parametrize("W,H,n,scale", [
    (16, 16, 700, (0.2, 2.0)),      # one tile
    (200, 171, 1025, (0.05, 1.5)),  # bins of one tile; one slot in the second block
    (401, 300, 2048, (0.05, 2.0)),  # 2 x 1 tiles
    (640, 481, 3000, (0.05, 2.0)),  # 2 x 2
    (699, 500, 3000, (0.05, 2.0)),  # 4 x 2
    (1000, 701, 3000, (0.05, 2.0)),  # 4 x 4
    (1601, 1067, 4000, (0.02, 1.5)),  # 8 x 4
])
def test_bin_shapes(P, orc, W, H, n, scale):
    cam = S.look_at((3.0, -20.0, 4.0), (0.0, 0.0, 0.0), W, H, 60.0)
    gf = S.random_gaussians(n, cam, W + H, scale=scale, neg_opacity_frac=0.1, behind_frac=0.05)
    ref = _check(P, orc, cam, gf, "shapes")
    if W >= 400:
        r = ref["pj"]["rect"][ref["pj"]["vis"] > 0].astype(np.int64)
        tiles = (r[:, 2] - r[:, 0]) * (r[:, 3] - r[:, 1])
        say(f"  rectangles of up to 64 tiles {(tiles <= 64).sum()}, more {(tiles > 64).sum()}")
        assert (tiles <= 64).sum() > 100 and (tiles > 64).sum() > 20


@pytest.mark.parametrize("n", [1, 64, 513, 3000])
@pytest.mark.parametrize("neg", [0.0, 0.03, 0.5, 0.97, 1.0])
def test_slots_without_opacity(P, orc, n, neg):
    """Blocks in which none, few, half, most or all slots have no opacity (the
    others are moved together)."""
    cam = S.look_at((3.0, -20.0, 4.0), (0.0, 0.0, 0.0), 333, 200, 60.0)
    gf = S.random_gaussians(n, cam, 7 * n, scale=(0.05, 1.5), neg_opacity_frac=neg)
    _check(P, orc, cam, gf, f"opacity fraction {neg}")


@pytest.mark.parametrize("n,depths", [(512, 0), (513, 0), (1025, 0), (2049, 0), (4096, 0),
                                      (4097, 0), (20000, 0), (3000, 1), (3000, 40), (9000, 7), (17000, 3)])
def test_long_lists_and_ties(P, orc, n, depths):
    """Every Gaussian covers all six tiles of a 48 x 32 image, so each bin's
    list has n entries: up to the block's 4,096, one more, and five merged
    runs; with `depths` only that many distinct depths (ties by slot)."""
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), 48, 32, 60.0)
    gf = S.random_gaussians(n, cam, n + depths, depth=(3.0, 6.0), scale=(1.5, 3.0), margin=0.0,
                            opacity=(0.0005, 0.004))
    if depths:
        # the camera looks along +y from y = -8: depth is y + 8
        gf[1] = (np.float32(0.25) * np.round(np.linspace(-12, -8, depths)))[
            np.random.default_rng(n).integers(0, depths, n)]
    ref = _check(P, orc, cam, gf, f"long lists, depths {depths}")
    assert (ref["bs"]["ranges"][:, 1] - ref["bs"]["ranges"][:, 0] == n).all()


def test_bands(P, orc):
    """65,536 x 1,040 pixels: 8,704 bins of 8 x 4 tiles, grouped in two bands."""
    cam = S.look_at((3.0, -20.0, 4.0), (0.0, 0.0, 0.0), 65536, 1040, 60.0)
    gf = S.random_gaussians(20000, cam, 5, scale=(0.001, 0.05), neg_opacity_frac=0.1)
    say("bins bands")
    pj = orc.project(gf, cam, orc.params_array())
    bs = orc.bin_sort(pj, cam)
    for train in (False, True):
        vb, _ = _raster(P, cam, gf, bs["n_rect_pairs"], train)
        _check_lists(vb, pj, bs)
        del vb
        torch.cuda.empty_cache()


def _crowd(n, W, H, span, big, seed, offset=(0.0, 0.0), scale=(0.005, 0.02), opacity=(0.02, 0.3)):
    """n small Gaussians whose centres lie within `span` pixels, `big` of them
    grown to tens of tiles."""
    cam = S.look_at((0.0, -8.0, 0.0), (0.0, 0.0, 0.0), W, H, 60.0)
    g = np.random.default_rng(seed)
    gf = S.random_gaussians(n, cam, seed, depth=(5.0, 40.0), scale=scale, margin=0.0, opacity=opacity)
    px = (gf[1] + 8.0) / (W / 2 / np.tan(np.radians(30.0)))  # the camera looks along +y
    for a, o in ((0, offset[0]), (2, offset[1])):
        gf[a] = (g.uniform(o - span / 2, o + span / 2, n) * px).astype(np.float32)
    k = g.choice(n, big, replace=False)
    gf[3:6, k] = g.uniform(0.5, 3.0, (3, big)).astype(np.float32)
    return cam, gf


def _long_bins(ref, W, H, sx, sy):
    """Entries of each bin of 2^sx x 2^sy tiles, from the oracle's lists."""
    tx = (W + 15) // 16
    tile, slot = ref["bs"]["tile_of"].astype(np.int64), ref["bs"]["gid_of"].astype(np.int64)
    b = ((tile // tx) >> sy) * 4096 + ((tile % tx) >> sx)
    return {k: (np.unique(slot[b == k]), tile[b == k], slot[b == k]) for k in np.unique(b)}


@pytest.mark.parametrize("W,H,n,span,big,sx,sy,depths", [
    (640, 481, 9000, 24, 60, 1, 1, 0),      # bins of 2 x 2 tiles
    (1000, 701, 14000, 50, 40, 2, 2, 0),    # 4 x 4
    (1601, 1067, 30000, 90, 30, 3, 2, 0),   # 8 x 4: some ten slices
    (1601, 1067, 14000, 90, 30, 3, 2, 5),   # ties by slot across slices
])
def test_long_bins_of_several_tiles(P, orc, W, H, n, span, big, sx, sy, depths):
    """Bins of several tiles with more entries than one block sorts, listed in
    different tiles each, some of them over more than 64 tiles (whose pair
    numbers without a pair are cleared)."""
    cam, gf = _crowd(n, W, H, span, big, n)
    if depths:
        z = gf[1] + 8.0
        zn = np.float32(0.5) * np.round(2.0 * np.linspace(6.0, 30.0, depths))[
            np.random.default_rng(n).integers(0, depths, n)].astype(np.float32)
        gf[0] *= zn / z
        gf[2] *= zn / z
        gf[1] = zn - 8.0
    ref = _check(P, orc, cam, gf, f"long bins of {1 << sx} x {1 << sy} tiles, depths {depths}")
    bins = _long_bins(ref, W, H, sx, sy)
    long = [b for b in bins.values() if len(b[0]) > 4096]
    assert long
    for _, tile, slot in long:  # the tiles' lists differ
        assert len(np.unique(tile)) > 1 and len(np.unique(slot[tile == tile[0]])) < len(np.unique(slot))
    r = ref["pj"]["rect"][ref["pj"]["vis"] > 0].astype(np.int64)
    assert ((r[:, 2] - r[:, 0]) * (r[:, 3] - r[:, 1]) > 64).any()


def test_long_bins_in_bands(P, orc):
    """Bins of more than 4,096 entries (copied by their block) and of more than
    16,384 (by all) in both bands of 65,536 x 1,040 pixels (bin rows 0 to 15, and
    16): their entries are copied before the next band takes the groups."""
    parts = [_crowd(n, 65536, 1040, span, 0, i, offset=o, scale=(0.0001, 0.0004))
             for i, (n, span, o) in enumerate([
                 (7000, 60, (-9000.0, 470.0)), (18000, 10, (5000.0, 470.0)),
                 (7000, 10, (8000.0, -511.0)), (18000, 10, (-7000.0, -511.0))])]
    cam = parts[0][0]
    gf = np.ascontiguousarray(np.concatenate([p[1] for p in parts], axis=1))
    say("bins, long ones in bands")
    pj = orc.project(gf, cam, orc.params_array())
    bs = orc.bin_sort(pj, cam)
    bins = _long_bins({"bs": bs}, cam.width, cam.height, 3, 2)
    for row in (0, 16):
        longest = [len(v[0]) for k, v in bins.items() if k // 4096 == row and len(v[0]) > 4096]
        assert min(longest) <= 16384 < max(longest)
    for train in (False, True):
        vb, _ = _raster(P, cam, gf, bs["n_rect_pairs"], train)
        _check_lists(vb, pj, bs)
        del vb
        torch.cuda.empty_cache()


def test_long_bins_in_flight(P):
    """Views with long bins on eight streams at once, several times over: the
    lists of each are those of the view alone."""
    views = []
    for i in range(8):
        cam, gf = _crowd(60000, 960, 540, 40 + 10 * i, 20, 50 + i)
        vb = P.ViewBuffers(gf.shape[1], 1, 960, 540, 4 << 20, gauss_capacity=gf.shape[1])
        vb.gauss.copy_(torch.as_tensor(gf).cuda())
        vb.gauss_count.fill_(gf.shape[1])
        views.append((vb, P.make_camera(cam)))
    prm = P.raster_params()
    alone = []
    for vb, cam in views:
        vb.rasterize(cam, prm)
        torch.cuda.synchronize()
        assert vb.stats()["sync_error"] == 0 and vb.stats()["pair_overflow"] == 0
        alone.append([x.copy() for x in vb.sorted_lists()] + [vb.rgb.clone()])
    say("bins, long ones in flight")
    streams = [torch.cuda.Stream() for _ in views]
    for _ in range(5):
        for (vb, cam), s in zip(views, streams):
            vb.rasterize(cam, prm, stream=s)
    torch.cuda.synchronize()
    for (vb, _), (tile, slot, ranges, rgb) in zip(views, alone):
        assert vb.stats()["sync_error"] == 0
        t, s, r = vb.sorted_lists()
        assert np.array_equal(t, tile) and np.array_equal(s, slot) and np.array_equal(r, ranges)
        assert torch.equal(vb.rgb, rgb)


def test_long_bins_time(P):
    """300k Gaussians within 64 x 64 pixels, every pixel done after one entry (so
    that the binning is what counts), take no more than four times as long as
    spread over 1000 x 1000: as long with two global sorts, 43 times as long where
    one block sorted all runs of a bin."""
    us = []
    for span in (64, 1000):
        cam, gf = _crowd(300000, 1920, 1080, span, 0, 9)
        vb = P.ViewBuffers(gf.shape[1], 1, 1920, 1080, 4 << 20, gauss_capacity=gf.shape[1])
        vb.gauss.copy_(torch.as_tensor(gf).cuda())
        vb.gauss_count.fill_(gf.shape[1])
        c, prm = P.make_camera(cam), P.raster_params(t_min=2.0)
        best = 1e9
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            vb.rasterize(c, prm)
            b.record()
            b.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        assert vb.stats()["pair_overflow"] == 0
        us.append(best)
    say(f"bins, 300k Gaussians in 64 x 64 px {us[0]:.0f} us, in 1000 x 1000 {us[1]:.0f}")
    assert us[0] <= 4.0 * us[1]
