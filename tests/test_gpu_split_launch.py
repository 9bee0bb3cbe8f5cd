"""How the render launches divide tiles over waves (whole tiles, halves, quadrants; the share depends on the
tile count) changes no image bit and no gradient beyond the summation order."""
import pytest

from paper_2411_00771_amd import scenes
from tests.helpers import gpu_forward, grad_close

pytestmark = pytest.mark.gpu


# tiles: 1 and 42 (all of them blocks, in the contribution pass quadrants), 1,281 (one tile past all quadrants; the
# lists are too short for blocks, so quadrants in both directions), 2,560 / 2,601 (the last all-halves launch, the
# first without), 3,136 and 4,096 (past the reverse's and the forward's fill)
@pytest.mark.parametrize("W,H,views", [(9, 11, 1), (101, 85, 1), (336, 976, 1), (1024, 640, 1), (816, 816, 1),
                                       (896, 896, 1), (512, 512, 4)])
def test_split_changes_nothing(cuda, W, H, views):
    import torch
    from paper_2411_00771_amd import raster
    sc = scenes.tiny_scene(8, 5000)
    cams = [scenes.tiny_camera(W, H, dist=3.0 + 0.1 * v) for v in range(views)]
    eng, params, cs = gpu_forward(sc, cams, capacity=1 << 22)
    assert eng.status.item() == 0
    g = torch.Generator(device=cuda).manual_seed(1)
    up = {k: torch.randn(s, device=cuda, generator=g) / (W * H) for k, s in
          dict(d_rgb=eng.rgb.shape, d_rgb_ssim=eng.rgb.shape, d_depth=eng.depth.shape, d_depth_med=eng.depth.shape,
               d_normal=eng.normal.shape, d_alpha=eng.alpha.shape).items()}
    names = ("rgb", "depth", "depth_med", "normal", "alpha", "T_final", "last", "med")

    def both():
        eng.render(cs)
        img = {k: getattr(eng, k).clone() for k in names}
        out = []
        for keys in (("d_rgb", "d_rgb_ssim"), tuple(up)):
            gr = raster.Grads(params, views)
            eng.backward(params, cs, gr, **{k: up[k] for k in keys})
            out.append(gr)
        c = torch.empty(views, eng.n, device=cuda)
        eng.contribution(cs, 0.5, c_view=c)
        return img, out, c

    img, grads, contrib = both()
    # whole tiles in spatial order, every entry walked
    eng._bins.order = None
    eng._img.qmask = None
    img0, grads0, contrib0 = both()
    torch.cuda.synchronize()
    for k in names:
        assert torch.equal(img[k], img0[k]), k
    grad_close("contribution", contrib.cpu().numpy(), contrib0.cpu().numpy(), rel=1e-5)
    # Both sums run over the same float32 terms in another order: at most about 16 roundings (2^-24 each) of a partial
    # sum deep, relative to the sum of the magnitudes.  With upstream gradients of random sign a surfel of P pixels
    # (here up to about 10^4) keeps 1 / sqrt(P) of that sum: 16 * 6e-8 * 100 = 1e-4 elementwise; the norm over all
    # surfels averages it out.
    for a, b in zip(grads, grads0):
        for k in ("mean", "log_scale", "quat", "opacity_logit", "sh", "g_view_total", "g_view_ssim"):
            grad_close(k, getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy(), rel=1e-4)
