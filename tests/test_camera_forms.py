"""Cameras whose fields are of unusual forms are taken, or refused, by the array as they are one by one."""
import types

import numpy as np
import pytest

from paper_2411_00771_amd import _lib, scenes


def _cameras(change, n=6):
    cams = scenes.aerial_cameras(3, scenes.make_city(2, L=300.0, n_boxes=4), count=n, width=97, height=33)
    out = []
    for c in cams:
        d = {f: getattr(c, f) for f in ("width", "height", "fx", "fy", "cx", "cy", "R", "t", "znear", "bg")}
        d.update(change(c))
        out.append(types.SimpleNamespace(**d))
    return out


def _tensor(x, **kw):
    import torch
    return torch.tensor(x, **kw)


@pytest.mark.parametrize("change", [
    lambda c: dict(fx=_tensor(c.fx, requires_grad=True), bg=_tensor([0.1, 0.2, 0.3], requires_grad=True)),
    lambda c: dict(R=_tensor(c.R), t=_tensor(c.t), znear=_tensor(0.3)),
    lambda c: dict(bg=[np.float32(0.1), True, "0.5"], cx=b"12.5"),
    lambda c: dict(bg={0: 0.1, 1: 0.2, 2: 0.3}),
    lambda c: dict(width=-3, height=(1 << 70) + 7),
])
def test_taken_as_one_by_one(change):
    cams = _cameras(change)
    assert bytes(_lib.camera_array(cams)) == b"".join(bytes(_lib.camera_struct(c)) for c in cams)


@pytest.mark.parametrize("change", [
    lambda c: dict(fx=None), lambda c: dict(znear=None), lambda c: dict(bg=(0.1, None, 0.3)), lambda c: dict(bg=None),
    lambda c: dict(R=None), lambda c: dict(bg=(0.1, 0.2)), lambda c: dict(cx="left"), lambda c: dict(t=[1j, 0, 0]),
])
def test_refused_as_one_by_one(change):
    cams = _cameras(change)
    with pytest.raises(Exception) as one:
        _lib.camera_struct(cams[0])
    with pytest.raises(one.type):
        _lib.camera_array(cams)
