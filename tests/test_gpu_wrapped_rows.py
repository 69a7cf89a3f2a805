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


@pytest.mark.parametrize("materialize", [False, True])
def test_ragged_corner_brick(materialize, capfd):
    """A corner brick narrower than a row, in a volume that is not: its rows start in the
    brick before it and end with the array, so cells take wrapped volumes too."""
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    dims, (W, H) = (300, 140, 180), (161, 150)
    ctx, plain = _debug_context(vr, VR_MARCH="ring"), _debug_context(vr, VR_MARCH="gather")
    a = torch.rand(dims[::-1], generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    tf = synth.tf_colour(64)
    tf[:, 3] = np.linspace(0, 0.05, 64)
    images = []
    # (bricks of 70 voxels, the last 20 wide, ghosts included 21; perspective cells too)
    for kind, c in (("held", ctx), ("wrapped", ctx), ("gathers", plain)):
        vr.vr_tf_set(c, tf, 0.0, 1.0)
        h = vr.vr_volume_create(c, a, dims) if kind == "held" else vr.vr_volume_wrap(c, a, dims)
        vr.vr_volume_brick(h, vr.grid_spec((70, 70, 90), materialize=materialize))
        views = [vr.make_view(R, W, H, eye_dist=e) for R, e in
                 zip(synth.random_views(4, 5), (0.0, 0.0, 900.0, 900.0))]
        out = torch.full((4, H, W, 4), 7.0, device="cuda")
        capfd.readouterr()
        for v in range(4):
            vr.vr_render(c, h, views[v:v + 1], vr.make_params(tau=2.0), out[v])
        torch.cuda.synchronize()
        said = capfd.readouterr().err
        if c is ctx:
            assert "gathers" not in said and said.count("cells axis") >= 2, said
        images.append(out)
        vr.vr_volume_destroy(h)
    assert float(images[0].abs().max()) > 0
    assert torch.equal(images[0], images[1]) and torch.equal(images[0], images[2])
    for c in (ctx, plain):
        vr.vr_destroy(c)
