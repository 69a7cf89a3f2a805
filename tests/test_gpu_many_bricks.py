"""Rays taken through more bricks than a wavefront tests at a time (64), and fronts of
many bricks: the bits of one lane per ray, front after front."""
import numpy as np
import pytest

import synth
from test_gpu_gather import _both, _opaque, _views

pytestmark = pytest.mark.gpu


# 63, 64, 65 and 1040 bricks; images of one pixel column, inside a tile and past one
@pytest.mark.parametrize("dims,brick", [((50, 41, 62), (49, 2, 20)), ((65, 17, 33), (4, 16, 8)), ((66, 14, 61), (5, 13, 12)),
                                        ((50, 41, 62), (5, 5, 5))])
@pytest.mark.parametrize("image", [(1, 30), (7, 9), (70, 45)])
@pytest.mark.parametrize("eye", [0.0, 300.0])
@pytest.mark.parametrize("mc", [0, 4])
def test_through_all_bricks(dims, brick, image, eye, mc):
    import torch

    def low(vmin, vmax):
        return synth.tf_noise_suppress(vmin, vmax, thresh=2.0, amax=0.6)
    mask = np.linspace(1, 0.2, dims[2]).astype(np.float32)
    for views in (_views(1, eye), _views(3, eye) + [(np.eye(3), eye)]):
        for m in (None, mask):
            x, y = _both(dims, image, lambda vr: vr.grid_spec(brick, macrocell=mc), views, low if mc else _opaque, mask=m,
                         ert_scope=1, tau=0.95, shows=image == (70, 45))
            assert torch.equal(x, y)


# several perspective views whose fronts are few and large
def test_perspective_fronts():
    import torch
    x, y = _both((300, 280, 290), (300, 280), lambda vr: vr.grid_spec((150,) * 3), _views(2, 700.0), _opaque, ert_scope=1,
                 tau=0.95)
    assert torch.equal(x, y)
