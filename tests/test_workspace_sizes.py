"""A workspace sized for an engine's largest call serves its smaller ones: no query asks for more at fewer tiles,
fewer views or a smaller image."""
import random

import pytest

from paper_2411_00771_amd import _lib


@pytest.mark.parametrize("capacity", [0, 8, 5000, 1 << 20, 5_000_000])
@pytest.mark.parametrize("views", [1, 4, 40])
def test_bin_sort_workspace_grows_with_tiles(capacity, views):
    need = _lib.lib().cgv2_bin_sort_workspace
    tiles = [1, 2, 64, 102, 103, 512, 513, 1024, 1025, 1200, 4095, 4096, 4097, 5000, 8160, 8192, 8193, 32400]
    sizes = [need(capacity, views, t, 30_000) for t in tiles]
    assert sizes == sorted(sizes)
    for t in tiles:
        assert need(capacity, 1, t, 30_000) <= need(capacity, views, t, 30_000)


def test_bin_sort_workspace_random_pairs():
    need = _lib.lib().cgv2_bin_sort_workspace
    rng = random.Random(5)
    for _ in range(20000):
        capacity, tiles, v = int(2 ** rng.uniform(0, 24)), int(2 ** rng.uniform(0, 15)), rng.randrange(1, 9)
        fewer = rng.randrange(1, tiles + 1)
        assert need(capacity, v, fewer, 1000) <= need(capacity, v, tiles, 1000), (capacity, v, fewer, tiles)


def test_loss_workspace_random_pairs():
    need = _lib.lib().cgv2_loss_workspace
    rng = random.Random(6)
    for _ in range(60000):
        w, h, v = int(2 ** rng.uniform(0, 12)), int(2 ** rng.uniform(0, 12)), rng.randrange(1, 9)
        w2, h2, v2 = (max(1, x - rng.randrange(4)) for x in (w, h, v))
        assert need(w2, h2, v2) <= need(w, h, v), (w, h, v, w2, h2, v2)


@pytest.mark.gpu
@pytest.mark.parametrize("width,height", [(640, 480), (1024, 1008), (64, 48)])
def test_smaller_image_on_a_larger_engine(cuda, width, height):
    """An engine of 8,160 tiles renders 1,200, 4,032 and 12 as an engine of that size does."""
    import torch
    from paper_2411_00771_amd import raster, scenes
    sc = scenes.tiny_scene(4, 6000)
    params = raster.Params.from_scene(sc)
    cam = scenes.tiny_camera(width, height)
    big = raster.Engine(sc.n, 1920, 1080, capacity=1 << 20)
    one = raster.Engine(sc.n, width, height, capacity=1 << 20)
    big.forward(params, big.cams([cam], exact=False))
    one.forward(params, one.cams([cam]))
    torch.cuda.synchronize()
    assert not big.overflowed() and float(one.alpha.max()) > 0
    for name in ("rgb", "depth", "alpha"):
        got, ref = big.image(name, width, height), getattr(one, name)[0]
        assert torch.equal(got.view(torch.int32), ref.contiguous().view(torch.int32)), name
