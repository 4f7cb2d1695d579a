"""Parity of the training losses (photometric L1 + SSIM, volume
regularisation) with the FP64 oracle, through the C ABI.

Bars: the loss within 2e-6 (FP32 sums of 1024 terms in [0, 1] per block,
the block sums then added in double); the image gradient within 1e-4
normwise and 1e-3 of the largest entry elementwise (the gradient
bar used throughout; the windowed variances lose a few bits to cancellation); the volume
gradient within 1e-6 relative (three FP32 products).
"""

import numpy as np
import pytest

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


@pytest.fixture(scope="module")
def LO():
    from oracle import losses as L
    return L


def _images(shape, seed):
    """A smooth image plus detail, and a noisy, shifted copy as the target
    (the statistics of a rendering against its ground truth)."""
    rng = np.random.default_rng(seed)
    H, W = shape[-2:]
    yy, xx = np.mgrid[0:H, 0:W]
    base = 0.5 + 0.3 * np.sin(xx / 7.0 + rng.uniform(0, 6, shape[:-2] + (1, 1))) * np.cos(yy / 11.0)
    img = np.clip(base + 0.1 * rng.standard_normal(shape), 0, 1).astype(np.float32)
    tgt = np.clip(img + 0.05 * rng.standard_normal(shape) + 0.02, 0, 1).astype(np.float32)
    return img, tgt


def _run(P, img, tgt, w_l1, w_ssim):
    x = torch.as_tensor(img).cuda()
    y = torch.as_tensor(tgt).cuda()
    d = torch.full_like(x, 7.0)   # overwritten
    loss = torch.full((1,), 0.5, dtype=torch.float32, device="cuda")  # accumulated
    P.photometric_loss_grad(x, y, d, loss, w_l1, w_ssim)
    torch.cuda.synchronize()
    return float(loss.item()) - 0.5, d.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("shape", [(2, 3, 97, 131), (1, 3, 5, 7), (1, 1, 16, 64), (4, 3, 1066, 1600)])
def test_photometric_parity(P, LO, shape):
    img, tgt = _images(shape, sum(shape))
    say("photometric", shape)
    loss, g = _run(P, img, tgt, 0.8, 0.2)
    rl, rg = LO.photometric_loss_grad(img, tgt, 0.8, 0.2)
    e = np.linalg.norm(g - rg) / np.linalg.norm(rg)
    say(f"  loss {loss:.7f} vs {rl:.7f}; grad rel err {e:.2e}, "
        f"max abs err / max {np.abs(g - rg).max() / np.abs(rg).max():.2e}")
    assert abs(loss - rl) <= 2e-6
    assert e <= 1e-4
    assert np.abs(g - rg).max() <= 1e-3 * np.abs(rg).max()


@pytest.mark.parametrize("hw", [(1, 235), (7, 236), (8, 237), (9, 472), (18, 473), (19, 11),
                                (137, 3), (300, 709)])
def test_photometric_strip_edges(P, LO, hw):
    """Image sizes at the edges of the strip kernel's blocks (236 columns; 8,
    18, ... rows) and windows larger than the image, with as many planes as
    take the call past the 1.6M elements that are done in tiles; one plane
    takes the tiled passes.  Bars of the parity test."""
    for planes in (1, 1600000 // (hw[0] * hw[1]) + 1):
        img, tgt = _images((planes,) + hw, 13 * hw[0] + hw[1])
        say("photometric strip edges", planes, hw)
        loss, g = _run(P, img, tgt, 0.8, 0.2)
        rl, rg = LO.photometric_loss_grad(img, tgt, 0.8, 0.2)
        assert abs(loss - rl) <= 2e-6
        assert np.linalg.norm(g - rg) <= 1e-4 * np.linalg.norm(rg)
        assert np.abs(g - rg).max() <= 1e-3 * np.abs(rg).max()


@pytest.mark.parametrize("planes,hw", [(3, (720, 1180)), (3, (719, 1181)), (3, (731, 1179)),
                                       (1600, (32, 32)), (3, (9000, 65))])
def test_photometric_wide_and_narrow(P, LO, planes, hw):
    """Calls past 1.6M elements: planes of five strips of 236 columns, one
    column more and less (strips), and narrow ones (tiles).  Bars of the parity
    test."""
    img, tgt = _images((planes,) + hw, hw[0] + hw[1])
    say("photometric wide and narrow", planes, hw)
    loss, g = _run(P, img, tgt, 0.8, 0.2)
    rl, rg = LO.photometric_loss_grad(img, tgt, 0.8, 0.2)
    assert abs(loss - rl) <= 2e-6
    assert np.linalg.norm(g - rg) <= 1e-4 * np.linalg.norm(rg)
    assert np.abs(g - rg).max() <= 1e-3 * np.abs(rg).max()


@pytest.mark.parametrize("planes,hw", [(1600, (32, 32)), (7000, (16, 16)), (60, (1000, 40))])
def test_photometric_narrow_time(P, planes, hw):
    """Many narrow planes in one call take no longer than in two calls of half
    of them (which are done in tiles); 236-column strips took 1.35 to 3.6 times
    as long."""
    x, y = torch.rand((planes,) + hw, device="cuda"), torch.rand((planes,) + hw, device="cuda")
    d, loss = torch.empty_like(x), torch.zeros(1, device="cuda")
    ws = P.photometric_loss_grad(x, y, d, loss)

    def best(parts):
        us = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for i in parts:
                P.photometric_loss_grad(x[i], y[i], d[i], loss, ws=ws)
            b.record()
            b.synchronize()
            us.append(1e3 * a.elapsed_time(b))
        return min(us)

    h = planes // 2
    whole, halves = best([slice(None)]), best([slice(0, h), slice(h, None)])
    say(f"photometric narrow {planes} x {hw}: {whole:.0f} us, in halves {halves:.0f}")
    assert whole <= 1.25 * halves


@pytest.mark.parametrize("planes,hw", [(3, (97, 131)), (3, (720, 1280)), (2, (1301, 1417))])
@pytest.mark.parametrize("over", ["img", "target"])
def test_photometric_in_place(P, LO, planes, hw, over):
    """The gradient written over the image or the target: the same as beside
    them, below and above the size that is done in tiles.  Bars of the parity
    test."""
    img, tgt = _images((planes,) + hw, 17 * hw[0] + hw[1])
    for w_ssim in (0.2, 0.0):
        say("photometric in place", planes, hw, over, w_ssim)
        x, y = torch.as_tensor(img).cuda(), torch.as_tensor(tgt).cuda()
        d = x if over == "img" else y
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        P.photometric_loss_grad(x, y, d, loss, 0.8, w_ssim)
        torch.cuda.synchronize()
        g = d.cpu().numpy().astype(np.float64)
        rl, rg = LO.photometric_loss_grad(img, tgt, 0.8, w_ssim)
        assert abs(float(loss.item()) - rl) <= 2e-6
        assert np.linalg.norm(g - rg) <= 1e-4 * np.linalg.norm(rg)
        assert np.abs(g - rg).max() <= 1e-3 * np.abs(rg).max()


def test_l1_only_and_identity(P, LO):
    img, tgt = _images((2, 3, 40, 70), 5)
    loss, g = _run(P, img, tgt, 1.0, 0.0)
    rl, rg = LO.photometric_loss_grad(img, tgt, 1.0, 0.0)
    assert abs(loss - rl) <= 1e-6
    assert np.array_equal(np.sign(g), np.sign(rg))
    np.testing.assert_allclose(g, rg, rtol=1e-6)
    # identical images: SSIM 1, loss 0
    loss, g = _run(P, img, img, 0.8, 0.2)
    assert abs(loss) <= 1e-6
    # gradient entries are O(w_ssim / n) in general; here FP32 leaves ~1e-6 of that
    assert np.abs(g).max() <= 1e-4 * 0.2 / img.size


def test_volume_loss_parity(P, LO):
    from paper_2403_17898_amd import _lib as L
    import ctypes
    rng = np.random.default_rng(8)
    cap, cnt = 5000, 4321
    gd = rng.random((14, cap)).astype(np.float32)
    gd[10] = rng.uniform(-1, 1, cap).astype(np.float32)
    g = torch.as_tensor(gd).cuda()
    c = torch.tensor([cnt], dtype=torch.int32).cuda()
    dg0 = np.full((14, cap), 0.25, np.float32)   # accumulated onto a known value
    dg = torch.as_tensor(dg0).cuda()
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    gs = L.Gaussians()
    gs.capacity, gs.data, gs.count = cap, g.data_ptr(), c.data_ptr()
    L.check(L.lib().octgs_volume_loss_grad(ctypes.byref(gs), 0.01, ctypes.c_void_p(dg.data_ptr()),
                                           ctypes.c_void_p(loss.data_ptr()), None),
            "octgs_volume_loss_grad")
    torch.cuda.synchronize()
    rl, rd = LO.volume_loss_grad(gd, cnt, 0.01)
    assert abs(float(loss.item()) - rl) <= 1e-6 * rl
    got = dg.cpu().numpy().astype(np.float64) - dg0
    np.testing.assert_allclose(got, rd, rtol=1e-6, atol=3e-8)
