"""Staging of views whose surfels cover a tile or two each (a surfel per lane, counters column by column, several
counters per tile below 4,096 tiles): the lists equal the oracle's, on either side of every rule's edge."""
import numpy as np
import pytest

import oracle
from paper_2411_00771_amd import scenes
from tests.helpers import compare_lists, fetch_bins, fetch_proj, gpu_forward

pytestmark = pytest.mark.gpu


def _scene(n, n_mid, n_big):
    """Surfels inside the view, most under a tile; n_mid of 9-256 tiles and n_big of more than 256."""
    rng = np.random.default_rng(n)
    sc = scenes.tiny_scene(n, n, sh_degree=0)
    sc.mean[:] = (sc.mean * 0.45).astype(np.float32)
    sc.log_scale[:] = rng.uniform(np.log(2e-4), np.log(1.5e-3), sc.log_scale.shape).astype(np.float32)
    sc.opacity_logit[:] = rng.uniform(0.0, 2.0, n).astype(np.float32)
    sel = rng.permutation(n)
    sc.log_scale[:, sel[:n_mid]] = np.log(rng.uniform(0.03, 0.1, (2, n_mid))).astype(np.float32)
    sc.log_scale[:, sel[n_mid:n_mid + n_big]] = np.log(rng.uniform(0.3, 0.8, (2, n_big))).astype(np.float32)
    return sc


# n: one short of the rule, at it, a short last run, and a last run of one surfel; tiles: 750 and 4,092 (eight
# counters each), 4,290 (one), 8,930 (scanned by several workgroups)
@pytest.mark.parametrize("n,W,H,views,mid,big", [(32767, 480, 400, 1, 300, 5), (32768, 480, 400, 1, 300, 5),
                                                (33025, 1056, 992, 1, 0, 0), (40001, 1056, 1040, 1, 200, 8),
                                                (33000, 1520, 1504, 1, 300, 3), (65537, 480, 400, 2, 500, 9),
                                                (34000, 96, 96, 1, 33, 0)])
def test_small_rect_lists_bit_exact(cuda, n, W, H, views, mid, big):
    sc = _scene(n, mid, big)
    cams = [scenes.tiny_camera(W, H, dist=3.0 + 0.3 * v) for v in range(views)]
    eng, _, _ = gpu_forward(sc, cams, capacity=1 << 20)
    assert eng.status.item() == 0
    vis, needed = int(eng.visible_start[-1].item()), int(eng.needed.item())
    assert vis == n * views and needed <= 6 * vis
    ranges, ids = fetch_bins(eng)
    P = fetch_proj(eng)
    total = 0
    for v, cam in enumerate(cams):
        po = oracle.project(sc, cam)
        a = ranges[v * eng.tiles:(v + 1) * eng.tiles + 1]
        r = compare_lists(a - a[0], ids[a[0]:a[-1]], po, cam, P=P, v=v, max_excluded=40)
        assert r["surfels"] <= 8
        total += r["rect_total"]
        tiles = np.prod(po["tile_rect"].astype(np.int64)[:, 2:] - po["tile_rect"].astype(np.int64)[:, :2], axis=1)
        if W >= 480:
            assert ((tiles > 8) & (tiles <= 256)).sum() >= mid // 2 and (tiles > 256).sum() >= big // 2
    assert abs(needed - total) <= 16  # rounding ties of a rect edge


def test_small_rects_overflow_and_rerun(cuda):
    """Too small a capacity: nothing is staged, the need is reported; the rerun's lists are the first run's."""
    import torch
    sc = _scene(33000, 100, 2)
    cam = scenes.tiny_camera(480, 400)
    eng, params, cs = gpu_forward(sc, [cam], capacity=1 << 18)
    assert eng.status.item() == 0
    ref = fetch_bins(eng)
    need = int(eng.needed.item())
    eng.set_capacity(need - 1)
    eng.bin_sort(cs)
    torch.cuda.synchronize()
    assert eng.status.item() == 1 and int(eng.needed.item()) == need
    eng.set_capacity(need)
    eng.status.zero_()
    eng.bin_sort(cs)
    torch.cuda.synchronize()
    got = fetch_bins(eng)
    assert eng.status.item() == 0 and np.array_equal(ref[0], got[0]) and np.array_equal(ref[1], got[1])
