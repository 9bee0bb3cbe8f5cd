"""The parameter chain of several views of many surfels (ranges of 512 surfels through all views) equals a call per
view adding into the same gradients."""
import numpy as np
import pytest

from paper_2411_00771_amd import scenes
from tests.helpers import grad_close

pytestmark = pytest.mark.gpu


# the smallest set of that path and ragged ones (a last range of 1 surfel, of 123), every SH degree
@pytest.mark.parametrize("n,views,degree", [(2_000_000, 2, 0), (2_000_385, 3, 1), (2_000_123, 2, 2), (2_000_001, 4, 3)])
def test_views_equal_single_view_calls(cuda, n, views, degree):
    import torch
    from paper_2411_00771_amd import raster
    rng = np.random.default_rng(views)
    gen = torch.Generator(device=cuda).manual_seed(n)
    rand = lambda *s: torch.rand(s, device=cuda, generator=gen)
    mean = 6 * rand(3, n) - 3  # most surfels outside a view, some in several; the last one in front in all
    mean[2] = mean[2] * 0.6 + 1.0
    mean[:, -1] = torch.tensor([0.0, 0.0, -1.4])
    quat = torch.randn(4, n, device=cuda, generator=gen)
    p = raster.Params(mean, -5.5 + rand(2, n), quat, torch.randn(n, device=cuda, generator=gen),
                      rand(n, (degree + 1) ** 2, 3) - 0.3, degree)
    W, H = 96, 80
    cams = [scenes.tiny_camera(W, H, fov_deg=30.0 + 8 * v, dist=float(rng.uniform(1.8, 4.0))) for v in range(views)]
    eng = raster.Engine(n, W, H, views, capacity=1 << 20)
    arr = eng.cams(cams)
    eng.fit_capacity(p, arr)
    eng.forward(p, arr)
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
    for k in ("mean", "log_scale", "quat", "opacity_logit", "sh"):
        a, b = getattr(g, k).cpu().numpy(), getattr(ref, k).cpu().numpy()
        assert np.abs(b[..., -1] if k != "sh" else b[-1]).max() > 0
        grad_close(k, a, b, rel=1e-4)
