"""Footprint-cell march: cells numbered along either axis, rays spread over the
LDS banks, window rows known to the compiler or not, channel masks: the same
bits as one lane per ray stepping through its samples (VR_MARCH=gather)."""
import numpy as np
import pytest

import synth
from test_gpu_gather import _both, _opaque, _ramp, _views

pytestmark = pytest.mark.gpu


# rays 1.6 and 3.7 voxels apart: cells of few rows, numbered along g, and of many
@pytest.mark.parametrize("image", [(430, 400), (180, 190)])
@pytest.mark.parametrize("edge", [128, 333])
@pytest.mark.parametrize("eye", [0.0, 1800.0])
@pytest.mark.parametrize("masked", [False, True])
def test_cells(image, edge, eye, masked):
    import torch
    dims = (500, 380, 401)
    mask = np.random.default_rng(1).uniform(0, 1, dims[2]).astype(np.float32) if masked else None
    # the slab axis is axis 2 in some of these views and axis 3 in others
    views = _views(3, eye) + [(np.eye(3), eye)]
    for tf, mode, tau in ((_ramp, 0, 0.99), (_opaque, 0, 0.9), (_ramp, 1, 0.99)):
        x, y = _both(dims, image, lambda vr: vr.grid_spec((edge,) * 3, twin=edge == 128), views, tf, mask=mask,
                     mode=mode, tau=tau)
        assert torch.equal(x, y)


# the stop test 1 - T >= tau as a bound on T, at thresholds that are no float
@pytest.mark.parametrize("tau", [1e-9, 0.1, 0.3333333, 0.9999999, 0.99999999, 1.0])
def test_stop_threshold(tau):
    import torch
    dims = (400, 380, 390)
    x, y = _both(dims, (300, 280), lambda vr: vr.grid_spec((128,) * 3), _views(2), _opaque, tau=tau, shows=False)
    assert torch.equal(x, y)
