"""The photometric loss over image sizes whose launches take different strip heights (4 to 128 output rows), against
the same formulas in float64 torch."""
import pytest

pytestmark = pytest.mark.gpu


def _window(x, torch):
    g = torch.exp(-torch.arange(-5, 6, device=x.device, dtype=torch.float64) ** 2 / 4.5)
    g = g / g.sum()
    for dim, pad in ((-1, (5, 5, 0, 0)), (-2, (0, 0, 5, 5))):
        p = torch.nn.functional.pad(x, pad)
        x = sum(g[k] * p.narrow(dim, k, x.shape[dim]) for k in range(11))
    return x


# strips of 4 rows with a last one of 1 row, a lone row, one strip per SIMD, two, several, and the tallest
@pytest.mark.parametrize("W,H,V", [(64, 5, 1), (65, 1, 2), (63, 127, 1), (317, 203, 1), (1280, 720, 1), (1600, 1066, 1),
                                   (1237, 823, 3), (640, 1300, 9)])
def test_loss_matches_float64(cuda, W, H, V):
    import torch
    from paper_2411_00771_amd import raster
    gen = torch.Generator(device=cuda).manual_seed(W + H)
    low = torch.rand((V, 3, max(2, H // 20), max(2, W // 20)), device=cuda, generator=gen)
    tgt = torch.nn.functional.interpolate(low, size=(H, W), mode="bilinear").contiguous()
    img = (tgt + 0.1 * torch.rand(tgt.shape, device=cuda, generator=gen)).contiguous()
    eng = raster.Engine(16, W, H, V, capacity=1 << 10)
    lv = eng.loss(tgt, img=img).double()
    x, y = img.double().requires_grad_(True), tgt.double()
    mx, my = _window(x, torch), _window(y, torch)
    sxx, syy = _window(x * x, torch) - mx * mx, _window(y * y, torch) - my * my
    sxy = _window(x * y, torch) - mx * my
    ssim = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
    ssim, l1 = ssim.mean((1, 2, 3)), (x - y).abs().mean((1, 2, 3))
    ds = torch.autograd.grad((0.2 * (1 - ssim)).sum(), x, retain_graph=True)[0]
    dt = ds + torch.autograd.grad((0.8 * l1).sum(), x)[0]
    ssim, l1 = ssim.detach(), l1.detach()
    # float32 variances: the moments (up to 1.2) cancel against the squared means to about 2^-24 * 4 of 1, next to
    # C2 = 9e-4 and variances of 1e-3 in the denominators: 3e-4 relative at worst; the mean over the image averages
    assert float((lv[:, 1] - l1).abs().max()) <= 1e-6 and float((lv[:, 2] - ssim).abs().max()) <= 1e-5
    assert float((eng.d_img_ssim - ds).abs().max() / ds.abs().max()) <= 1e-3
    assert float((eng.d_img - dt).abs().max() / dt.abs().max()) <= 1e-3
    assert float((eng.d_img_ssim - ds).norm() / ds.norm()) <= 3e-4
