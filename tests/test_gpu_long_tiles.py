"""Launches of 641 tiles and more, whose heavier tiles run as sixteen 4x4 blocks where their lists are long and as four
quadrants elsewhere, give the images of whole tiles bit for bit, and the reverse pass the same entries; how many slots
the bins hold changes nothing."""
import numpy as np
import pytest

from paper_2411_00771_amd import scenes
from tests.helpers import gpu_forward, grad_close

pytestmark = pytest.mark.gpu

NAMES = ("rgb", "depth", "depth_med", "normal", "alpha", "T_final", "last", "med")


# tiles: 646 and 1,200 (single and two views), 1,900 and 3,600 (the reverse alone); 'near' surfels of all lie around
# one point, so that some lists are longer than 512 entries and five halves of the mean and others shorter than 256,
# or (0) all of about one length
@pytest.mark.parametrize("W,H,views,near,capacity", [
    (541, 300, 1, 0.4, 1 << 21), (640, 480, 1, 0.4, 1 << 20), (640, 480, 1, 0.4, 1 << 23), (640, 480, 1, 0.0, 1 << 23),
    (400, 375, 2, 0.3, 1 << 22), (800, 600, 1, 0.3, 1 << 23), (1280, 720, 1, 0.3, 1 << 22)])
def test_maybe_blocks_equal_whole_tiles(cuda, W, H, views, near, capacity):
    import torch
    from paper_2411_00771_amd import raster
    n = 12000
    sc = scenes.tiny_scene(W + H, n)
    k = int(near * n)
    sc.mean[:, :k] *= np.float32(0.06)
    sc.log_scale[:, :k] -= np.float32(1.5)
    sc.opacity_logit[:k] -= np.float32(4.0)
    cams = [scenes.tiny_camera(W, H, dist=3.0 + 0.3 * v) for v in range(views)]
    eng, params, cs = gpu_forward(sc, cams, capacity=capacity)
    assert eng.status.item() == 0
    lists = eng.ranges.diff().sort(descending=True).values.double()
    if near:
        assert float(lists[0]) >= max(512, 2.5 * float(lists.mean())) and float(lists[lists.numel() // 8]) < 256
    img = {name: getattr(eng, name).clone() for name in NAMES}
    g = torch.Generator(device=cuda).manual_seed(1)
    up = torch.randn(eng.rgb.shape, device=cuda, generator=g) / (W * H)
    ups = [dict(d_rgb=up, d_rgb_ssim=up), dict(d_rgb=up, d_rgb_ssim=up, d_normal=up)]

    def grads():
        out = []
        for u in ups:
            gr = raster.Grads(params, views)
            eng.backward(params, cs, gr, **u)
            out.append(gr)
        return out

    one = grads()
    order, eng._bins.order = eng._bins.order, None  # whole tiles
    eng.render(cs)
    torch.cuda.synchronize()
    for name in NAMES:
        assert torch.equal(img[name].view(torch.int32), getattr(eng, name).view(torch.int32)), name
    two = grads()
    eng._bins.order = order
    torch.cuda.synchronize()
    for a, b in zip(one, two):
        for name in ("mean", "log_scale", "quat", "opacity_logit", "sh", "g_view_total", "g_view_ssim"):
            # float atomics in another order: see the split-launch test for the bound
            grad_close(name, getattr(a, name).cpu().numpy(), getattr(b, name).cpu().numpy(), rel=1e-4)
