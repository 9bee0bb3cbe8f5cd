"""The parameter chain of several views of many surfels, of which few are visible (a wave then takes 1,024 surfels
instead of 512), equals a call per view adding into the same gradients."""
import numpy as np
import pytest

from paper_2411_00771_amd import scenes
from tests.helpers import grad_close

pytestmark = pytest.mark.gpu


# the visible ones spread over the set, packed into one range (its list full), and at the end of the last one
@pytest.mark.parametrize("n,views,degree,where", [(2_000_385, 2, 3, "spread"), (2_000_513, 3, 1, "packed"),
                                                  (2_097_152, 2, 2, "last")])
def test_few_visible(cuda, n, views, degree, where):
    import torch
    from paper_2411_00771_amd import raster
    gen = torch.Generator(device=cuda).manual_seed(n)
    rand = lambda *s: torch.rand(s, device=cuda, generator=gen)
    k = 3000
    ids = {"spread": torch.randperm(n, device=cuda, generator=gen)[:k], "packed": torch.arange(k, device=cuda) + 1024,
           "last": torch.arange(n - k, n, device=cuda)}[where]
    mean = torch.tensor([[0.0], [0.0], [-50.0]], device=cuda).repeat(1, n)  # behind every camera
    mean[:, ids] = 1.2 * rand(3, k) - 0.6
    p = raster.Params(mean, -4.0 + rand(2, n), torch.randn(4, n, device=cuda, generator=gen),
                      torch.randn(n, device=cuda, generator=gen), rand(n, (degree + 1) ** 2, 3) - 0.3, degree)
    W, H = 96, 80
    cams = [scenes.tiny_camera(W, H, dist=2.5 + 0.4 * v) for v in range(views)]
    eng = raster.Engine(n, W, H, views, capacity=1 << 20)
    arr = eng.cams(cams)
    eng.forward(p, arr)
    seen = int(eng.visible_start[views])
    assert not eng.overflowed() and 0 < seen < n * views // 128
    up = torch.randn(eng.rgb.shape, device=cuda, generator=gen) / (W * H)
    ups = torch.randn(eng.rgb.shape, device=cuda, generator=gen) / (W * H)
    g = raster.Grads(p, views)
    g.g_view_total.fill_(7.0)  # overwritten whole
    g.g_view_ssim.fill_(7.0)
    eng.backward(p, arr, g, d_rgb=up, d_rgb_ssim=ups, d_normal=up)
    one = raster.Engine(n, W, H, 1, capacity=eng.capacity)
    ref = raster.Grads(p, 1)
    for v, cam in enumerate(cams):
        a = one.cams([cam])
        one.forward(p, a)
        one.backward(p, a, ref, d_rgb=up[v:v + 1].contiguous(), d_rgb_ssim=ups[v:v + 1].contiguous(),
                     d_normal=up[v:v + 1].contiguous())
        torch.cuda.synchronize()
        # float atomics of the record gradients in another order: see the split-launch test for the bound
        grad_close("total", g.g_view_total[v].cpu().numpy(), ref.g_view_total[0].cpu().numpy(), rel=1e-4)
        grad_close("ssim", g.g_view_ssim[v].cpu().numpy(), ref.g_view_ssim[0].cpu().numpy(), rel=1e-4)
    for name in ("mean", "log_scale", "quat", "opacity_logit", "sh"):
        a, b = getattr(g, name).cpu().numpy(), getattr(ref, name).cpu().numpy()
        assert np.abs(b).max() > 0
        grad_close(name, a, b, rel=1e-4)
