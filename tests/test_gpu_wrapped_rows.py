"""Wrapped volumes narrower than a window's row: the caller's array has nothing
readable behind it, so the march that stages whole rows is left to volumes held
by the library, and the images are the same."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _debug_context(vr, **env):
    env = {"VR_DEBUG_PLAN": "1", **env}
    os.environ.update(env)
    try:
        return vr.vr_create(0)
    finally:
        for k in env:
            del os.environ[k]


def test_narrow_wrapped_volume(capfd):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    dims, (W, H) = (24, 8000, 400), (9000, 32)
    # image x along axis 2, image y along axis 1
    R = np.array([[0.0, 1.0, 0.0], [-1.0, 0.0, 0.0], [0.0, 0.0, 1.0]]) @ synth.rot_axis(3, 0.2)
    ctx = _debug_context(vr)
    a = torch.rand(dims[::-1], generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    tf = synth.tf_colour(64)
    tf[:, 3] = np.linspace(0, 0.02, 64)
    vr.vr_tf_set(ctx, tf, 0.0, 1.0)
    images = {}
    for kind in ("held", "wrapped", "bricked", "saved"):
        h = vr.vr_volume_create(ctx, a, dims) if kind == "held" else vr.vr_volume_wrap(ctx, a, dims)
        if kind == "bricked":
            vr.vr_volume_brick(h, vr.grid_spec((100, 10000, 1000)))
        out = torch.full((1, H, W, 4), 7.0, device="cuda")
        capfd.readouterr()
        st = vr.vr_render(ctx, h, [vr.make_view(R, W, H, extent=8000.0)], vr.make_params(tau=2.0), out,
                          save=kind == "saved")
        torch.cuda.synchronize()
        said = capfd.readouterr().err
        assert ("cells axis" in said) == (kind == "held"), said
        assert "saved by cells" not in said
        if st:
            vr.vr_state_destroy(st)
        images[kind] = out
        vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
    assert float(images["held"].abs().max()) > 0
    for kind in ("wrapped", "bricked", "saved"):
        assert torch.equal(images[kind], images["held"])
