"""Visible frequencies at the edges of the point boxes (128 points a wave, 512 to 4,096 a workgroup) and of the slices
of views, near oblique cameras, and with points that have no position."""
import numpy as np
import pytest

from oracle import visibility as ovis
from paper_2411_00771_amd import scenes

pytestmark = pytest.mark.gpu


def _counts(P, cams, rho, rf):
    import torch
    from paper_2411_00771_amd import crop
    pt = torch.from_numpy(np.ascontiguousarray(P, np.float32)).cuda()
    return crop.visibility_count(pt, cams, rho, rf).cpu().numpy().view(np.uint32).astype(np.int64)


def _scene(m, views, seed=11):
    city = scenes.make_city(seed, L=300.0, n_boxes=20)
    P = scenes.city_points(seed + 1, m, city)
    # low oblique cameras: their camera planes cut the city
    return P[:, scenes.morton_order(P)], scenes.aerial_cameras(seed + 2, city, count=views, width=320, height=240,
                                                               alt=(20.0, 60.0))


def _check(P, cams, rho, rf):
    ref, frag = ovis.visibility_count(P, cams, rho, rf)
    got = _counts(P, cams, rho, rf)
    assert np.array_equal(got[frag == 0], ref[frag == 0])
    assert np.all(np.abs(got - ref) <= frag)


# a lane short of and past a wave's box and a workgroup's, one and several slices of 64 views, more points per
# workgroup (from 2,048 * 1,024 points); rho small (the pixel disc is the larger reach), between, and large
@pytest.mark.parametrize("rf", [2.1213, 0.5, 0.2])
@pytest.mark.parametrize("m,views,rho", [(127, 1, 0.4), (129, 64, 3.0), (511, 65, 0.02), (513, 130, 0.4),
                                         (4097, 70, 0.4), (2_100_003, 3, 0.4)])
def test_counts_at_box_and_slice_edges(cuda, m, views, rho, rf):
    P, cams = _scene(m, views)
    _check(P, cams, rho, rf)


@pytest.mark.parametrize("rf", [2.1213, 0.2])
def test_points_without_a_position(cuda, rf):
    P, cams = _scene(5000, 40)
    ref, frag = ovis.visibility_count(P, cams, 0.4, rf)
    Q = np.repeat(P, 2, axis=1)
    bad = np.ones(Q.shape[1], bool)
    bad[::2] = False
    rng = np.random.default_rng(2)
    Q[rng.integers(0, 3, bad.sum()), np.flatnonzero(bad)] = np.nan
    got = _counts(Q, cams, 0.4, rf)
    assert not got[bad].any()  # no view sees a point whose coordinate is NaN
    assert np.array_equal(got[~bad][frag == 0], ref[frag == 0])
    Q[:, bad] = P
    Q[0, np.flatnonzero(bad)[::3]] = np.inf  # a point at infinity leaves its box's other points as they are
    got = _counts(Q, cams, 0.4, rf)
    assert np.array_equal(got[~bad][frag == 0], ref[frag == 0])


@pytest.mark.parametrize("m", [1, 63, 255, 257, 2047, 2049, 70_001])
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
def test_crop_volume_keeps_the_order(cuda, m, share):
    import torch
    from paper_2411_00771_amd import crop
    rng = np.random.default_rng(m)
    P = rng.uniform(-50, 50, (3, m)).astype(np.float32)
    cnt = (rng.random(m) < share) * 3
    T = np.array([[0.6, -0.8, 0, 5.0], [0.8, 0.6, 0, -2.0], [0, 0, 1.0, -10.0]])
    keep, ground, (h0, h1) = crop.crop_volume(torch.from_numpy(P).cuda(),
                                              torch.from_numpy(cnt.astype(np.int32)).cuda(), 2, T)
    rk, rg, rh0, rh1 = ovis.crop_volume(P, cnt, 2, T)
    assert np.array_equal(keep.cpu().numpy().astype(bool), rk)
    # sums of four products of at most 50 in FP64, in another order
    assert ground.shape == rg.shape and np.allclose(ground.cpu().numpy(), rg, rtol=0, atol=8 * 50 * 2.0 ** -52)
    if rk.any():
        assert abs(h0 - rh0) <= 8 * 50 * 2.0 ** -52 and abs(h1 - rh1) <= 8 * 50 * 2.0 ** -52
    else:
        assert np.isnan(h0) and np.isnan(h1)
