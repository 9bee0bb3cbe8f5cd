"""Several views of one thread's surfel project bit for bit like one view at a time."""
import numpy as np
import pytest

from paper_2411_00771_amd import scenes

pytestmark = pytest.mark.gpu


def _compact(p, n, degree, gen, cuda):
    import torch
    from paper_2411_00771_amd import storage
    K = (degree + 1) ** 2
    nf = n // 2
    code = torch.randint(0, 97, (n - nf,), device=cuda, generator=gen).to(torch.int16)  # 90 codewords: some invalid
    return storage.CompactParams(p.mean, p.log_scale.half(), p.quat.half(), p.opacity_logit.half(),
                                 p.sh[:nf].half().contiguous(), code,
                                 torch.rand(90, K, 3, device=cuda, generator=gen).half(), nf, degree)


# 2 and 3 views per thread with a shorter last slice, all views of a launch, one launch of 32 and a second of 1
@pytest.mark.parametrize("n,views,degree,compact", [(600_001, 3, 0, False), (600_001, 5, 2, True),
                                                    (1_048_700, 3, 3, False), (1_048_700, 4, 1, True),
                                                    (300_000, 33, 0, False)])
def test_views_equal_single_views(cuda, n, views, degree, compact):
    import torch
    from paper_2411_00771_amd import raster
    gen = torch.Generator(device=cuda).manual_seed(n + views)
    rand = lambda *s: torch.rand(s, device=cuda, generator=gen)
    p = raster.Params(6 * rand(3, n) - 3, -5.5 + rand(2, n), torch.randn(4, n, device=cuda, generator=gen),
                      3 * torch.randn(n, device=cuda, generator=gen), rand(n, (degree + 1) ** 2, 3) - 0.3, degree)
    p.quat[:, ::1001] = 0.0  # degenerate and non-finite surfels
    p.mean[1, ::997] = float("nan")
    p.log_scale[0, ::991] = 200.0
    if compact:
        p = _compact(p, n, degree, gen, cuda)
    rng = np.random.default_rng(views)
    W, H = 96, 80
    cams = [scenes.tiny_camera(W, H, fov_deg=30.0 + v, dist=float(rng.uniform(1.8, 4.0))) for v in range(views)]
    eng = raster.Engine(n, W, H, views, capacity=1 << 10, backward=False, images=False)
    eng.project(p, eng.cams(cams))
    one = raster.Engine(n, W, H, 1, capacity=1 << 10, backward=False, images=False)
    for v, cam in enumerate(cams):
        one.project(p, one.cams([cam]))
        torch.cuda.synchronize()
        s = slice(v * n, (v + 1) * n)
        vis = (one.flags[:n] & 1).bool()
        assert bool(vis.any()) and not bool(vis.all())
        assert torch.equal(eng.flags[s], one.flags[:n])
        assert torch.equal(eng.radius[s].view(torch.int32), one.radius[:n].view(torch.int32))
        assert torch.equal(eng.rect.view(-1)[4 * v * n:4 * (v + 1) * n], one.rect.view(-1)[:4 * n])
        a = eng.rec.view(views * n, -1)[s][vis].view(torch.int32)
        assert torch.equal(a, one.rec.view(n, -1)[vis].view(torch.int32))
