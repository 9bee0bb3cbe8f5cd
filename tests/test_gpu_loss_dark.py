"""The photometric loss keeps its relative precision on dark images and on images that differ by little."""
import pytest

pytestmark = pytest.mark.gpu


def _window(x, torch):
    g = torch.exp(-torch.arange(-5, 6, device=x.device, dtype=torch.float64) ** 2 / 4.5)
    g = g / g.sum()
    for dim, pad in ((-1, (5, 5, 0, 0)), (-2, (0, 0, 5, 5))):
        p = torch.nn.functional.pad(x, pad)
        x = sum(g[k] * p.narrow(dim, k, x.shape[dim]) for k in range(11))
    return x


def _losses(img, tgt, torch):
    """(L1, SSIM gradient of 0.2 (1 - SSIM)) per view in float64."""
    x, y = img.double().requires_grad_(True), tgt.double()
    mx, my = _window(x, torch), _window(y, torch)
    sxx, syy = _window(x * x, torch) - mx * mx, _window(y * y, torch) - my * my
    sxy = _window(x * y, torch) - mx * my
    ssim = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
    ds = torch.autograd.grad((0.2 * (1 - ssim.mean((1, 2, 3)))).sum(), x)[0]
    return (x - y).abs().mean((1, 2, 3)).detach(), ds


# ragged sizes (strips of other heights, a last column of one pixel); values up to 'top'
@pytest.mark.parametrize("W,H", [(65, 33), (317, 203), (640, 400)])
@pytest.mark.parametrize("top,bound", [(0.2, 6e-6), (0.03, 2e-6), (0.004, 2e-6), (1e-4, 2e-6)])
def test_dark_images(cuda, W, H, top, bound):
    import torch
    from paper_2411_00771_amd import raster
    gen = torch.Generator(device=cuda).manual_seed(W)
    low = torch.rand((2, 3, max(2, H // 20), max(2, W // 20)), device=cuda, generator=gen)
    tgt = (0.9 * top * torch.nn.functional.interpolate(low, size=(H, W), mode="bilinear")).contiguous()
    img = (tgt + 0.1 * top * torch.rand(tgt.shape, device=cuda, generator=gen)).contiguous()
    eng = raster.Engine(1, W, H, 2, capacity=64)
    lv = eng.loss(tgt, img=img).double()
    l1, ds = _losses(img, tgt, torch)
    # the L1 value is a float64 sum of differences, each rounded once, and is rounded itself: 2^-24 each
    assert float(((lv[:, 1] - l1) / l1).abs().max()) <= 2 * 2.0 ** -24
    # the moments of 22 taps (a few roundings of 2^-24 of their size, random sign) cancel by at most top^2 against
    # the variances' 9e-4 + variance: a factor of about 8 at 0.2, none below
    assert float((eng.d_img_ssim - ds).norm() / ds.norm()) <= bound


def test_bright_and_mid_images_keep_theirs(cuda):
    """Strips of bright, of mid-grey and of dark values, and strips of several, in one image."""
    import torch
    from paper_2411_00771_amd import raster
    W, H = 640, 400
    gen = torch.Generator(device=cuda).manual_seed(3)
    low = torch.rand((1, 3, 20, 32), device=cuda, generator=gen)
    base = 0.1 * torch.nn.functional.interpolate(low, size=(H, W), mode="bilinear")
    noise = torch.rand(base.shape, device=cuda, generator=gen)
    band = (torch.arange(H, device=cuda) % 160 < 80).float()[:, None]
    # one value range each; the moments about zero would give 2e-5 and more in the first two (measured 6.9e-5, 2.8e-5)
    for offset, bound in ((0.9, 6e-5), (0.45, 2.5e-5)):
        tgt = (base + offset).contiguous()
        img = (tgt + 0.01 * noise).contiguous()
        eng = raster.Engine(1, W, H, 1, capacity=64)
        eng.loss(tgt, img=img)
        _, ds = _losses(img, tgt, torch)
        assert float((eng.d_img_ssim - ds).norm() / ds.norm()) <= bound, offset
    tgt = (band * (base + 0.6) + (1 - band) * 0.1 * base).contiguous()
    img = (tgt + 0.01 * noise * (0.1 + band)).contiguous()
    eng = raster.Engine(1, W, H, 1, capacity=64)
    eng.loss(tgt, img=img)
    _, ds = _losses(img, tgt, torch)
    assert float((eng.d_img_ssim - ds).norm() / ds.norm()) <= 3e-5
