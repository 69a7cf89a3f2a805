"""The walk from macrocell to macrocell at the ends of its ranges: steps so small that
a macrocell holds more samples than an int counts, and macrocells far along a long
axis."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_more_samples_than_an_int(capfd):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    os.environ["VR_DEBUG_PLAN"] = "1"
    try:
        ctx = vr.vr_create(0)
    finally:
        del os.environ["VR_DEBUG_PLAN"]
    # two macrocells of 1024 side by side along axis 1, the first clear; rays along
    # axis 3, 29 voxels long: 7e7 samples each, 2.5e9 to the macrocells' far plane
    dims, step = (1500, 20, 30), 4e-7
    a = torch.zeros(dims[::-1], device="cuda")
    a[:, :, 1025:] = 1.0
    tf = synth.tf_colour(16)
    tf[:, 3] = np.where(np.arange(16) < 8, 0.0, 0.5)
    h = vr.vr_volume_create(ctx, a, dims)
    vr.vr_volume_brick(h, vr.grid_spec((2000, 2000, 2000), macrocell=1024))
    vr.vr_tf_set(ctx, tf, 0.0, 1.0)
    out = torch.full((1, 5, 60, 4), 7.0, device="cuda")
    vr.vr_render(ctx, h, [vr.make_view(np.eye(3), 60, 5, extent=1500.0)], vr.make_params(step=step, tau=0.9), out)
    torch.cuda.synchronize()
    assert "skip 1" in capfd.readouterr().err
    x = (np.arange(60) + 0.5) / 60 * 1500.0 - 0.5
    alpha = out[0, :, :, 3].cpu().numpy()
    hit = np.abs(alpha).max(axis=1) > 0  # rows inside the box
    assert hit.any()
    assert (alpha[hit][:, x < 1020] == 0.0).all()
    assert (alpha[hit][:, (x > 1030) & (x < 1499)] == 0.9375).all()  # four samples of opacity 1/2
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
