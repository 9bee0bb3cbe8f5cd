"""The camera array filled by fields equals the cameras one by one."""
import types

import numpy as np
import pytest

from paper_2411_00771_amd import _lib, scenes


def _cameras(n):
    return scenes.aerial_cameras(3, scenes.make_city(2, L=300.0, n_boxes=4), count=n, width=97, height=33)


def _one_by_one(cams):
    return b"".join(bytes(_lib.camera_struct(c)) for c in cams)


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 70])
def test_array_equals_structs(n):
    assert bytes(_lib.camera_array(_cameras(max(n, 1))[:n])) == _one_by_one(_cameras(max(n, 1))[:n])


def _as(c, **kw):
    d = dict(width=c.width, height=c.height, fx=c.fx, fy=c.fy, cx=c.cx, cy=c.cy, R=c.R, t=c.t, znear=c.znear, bg=c.bg)
    return types.SimpleNamespace(**{**d, **kw})


@pytest.mark.parametrize("change", [
    lambda c, k: dict(R=c.R.astype(np.float32), t=list(c.t)),
    lambda c, k: dict(R=c.R.reshape(-1), t=c.t.reshape(3, 1), width=float(c.width)),
    lambda c, k: dict(bg=(0.1, 0.2, 0.3, 1.0) if k % 2 else (0.1, 0.2, 0.3)),  # does not stack
    lambda c, k: dict(t=np.append(c.t, 1.0)),  # the first three count
    lambda c, k: dict(fx=1e39, cx=float("nan"), width=(1 << 32) + 5),
])
def test_fields_of_other_forms(change):
    cams = [_as(c, **change(c, k)) for k, c in enumerate(_cameras(6))]
    assert bytes(_lib.camera_array(cams)) == _one_by_one(cams)


def test_bad_cameras_raise_as_one_by_one():
    cams = _cameras(5)
    cams[3] = _as(cams[3], R=np.zeros(8))
    with pytest.raises(IndexError):
        _lib.camera_array(cams)
    cams[3] = types.SimpleNamespace(width=1)
    with pytest.raises(AttributeError):
        _lib.camera_array(cams)
