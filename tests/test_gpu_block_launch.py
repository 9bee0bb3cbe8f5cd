"""Tiles that run as sixteen 4x4 blocks give the images of whole tiles bit for bit, and the reverse pass the same
entries."""
import numpy as np
import pytest

from paper_2411_00771_amd import scenes
from tests.helpers import gpu_forward, grad_close

pytestmark = pytest.mark.gpu

NAMES = ("rgb", "depth", "depth_med", "normal", "alpha", "T_final", "last", "med")


# tiles: one (ragged, and with blocks outside the image), all blocks up to 640, the heaviest from 641 to 1,279, and above
# that none, the lists being short (the long-tiles test has others); two views in one launch.  Opaque surfels stop pixels within four entries of one
# another, faint ones fill the lists; a few surfels leave all but one of the four places empty.
@pytest.mark.parametrize("W,H,views,capacity,n,opacity", [
    (5, 3, 1, 1 << 20, 4000, 2.0), (16, 16, 1, 1 << 20, 3, 0.0), (16, 16, 1, 1 << 20, 70000, -3.0),
    (320, 256, 1, 1 << 20, 6000, 6.0), (1712, 48, 1, 1 << 21, 6000, 0.0), (160, 256, 2, 1 << 20, 5000, -2.0),
    (640, 256, 1, 1 << 20, 9000, 1.0), (1712, 96, 1, 1 << 20, 9000, 0.0), (640, 510, 1, 1 << 21, 20000, 3.0), (656, 788, 1, 1 << 23, 20000, -1.0)])
def test_blocks_equal_whole_tiles(cuda, W, H, views, capacity, n, opacity):
    import torch
    from paper_2411_00771_amd import raster
    sc = scenes.tiny_scene(int(n + W), n)
    sc.opacity_logit[:] += np.float32(opacity)
    cams = [scenes.tiny_camera(W, H, dist=2.5 + 0.3 * v) for v in range(views)]
    for c in cams:
        c.bg = (0.2, 0.5, 0.7)
    eng, params, cs = gpu_forward(sc, cams, capacity=capacity)
    assert eng.status.item() == 0
    img = {k: getattr(eng, k).clone() for k in NAMES}
    g = torch.Generator(device=cuda).manual_seed(1)
    up = torch.randn(eng.rgb.shape, device=cuda, generator=g) / (W * H)
    one = raster.Grads(params, views)
    eng.backward(params, cs, one, d_rgb=up, d_rgb_ssim=up, d_normal=up)
    order, eng._bins.order = eng._bins.order, None  # whole tiles
    eng.render(cs)
    torch.cuda.synchronize()
    for k in NAMES:
        assert torch.equal(img[k].view(torch.int32), getattr(eng, k).view(torch.int32)), k
    assert float(img["alpha"].max()) > 0
    two = raster.Grads(params, views)
    eng.backward(params, cs, two, d_rgb=up, d_rgb_ssim=up, d_normal=up)
    eng._bins.order = order
    torch.cuda.synchronize()
    for k in ("mean", "log_scale", "quat", "opacity_logit", "sh"):
        # float atomics in another order: see the split-launch test for the bound
        grad_close(k, getattr(one, k).cpu().numpy(), getattr(two, k).cpu().numpy(), rel=1e-4)
