"""A step so small that a ray could have 2^24 samples in a brick: not marched by the
footprint cells, whose count of samples is a float (the plan is looked at, and the
images are those of one lane per ray)."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eye", [0.0, 100.0])
@pytest.mark.parametrize("scope", [0, 1])
def test_no_cells(eye, scope, capfd):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    # opaque at once: a ray takes a few of its 25 million samples
    dims, step = (40, 36, 38), 2.6e-6
    a = torch.full(dims[::-1], 0.5, device="cuda")
    tf = synth.tf_colour(16)
    tf[:, 3] = 0.5
    images = []
    for env in ({"VR_MARCH": "ring", "VR_DEBUG_PLAN": "1"}, {"VR_MARCH": "gather"}):
        os.environ.update(env)
        try:
            ctx = vr.vr_create(0)
        finally:
            for k in env:
                del os.environ[k]
        h = vr.vr_volume_create(ctx, a, dims)
        vr.vr_volume_brick(h, vr.grid_spec((100, 100, 100)))
        vr.vr_tf_set(ctx, tf, 0.0, 1.0)
        views = [vr.make_view(R, 30, 28, eye_dist=eye) for R in synth.random_views(2, 3)]
        for tau, few in ((0.9, step), (0.9, 0.5)):
            out = torch.full((2, 28, 30, 4), 7.0, device="cuda")
            capfd.readouterr()
            vr.vr_render(ctx, h, views, vr.make_params(step=few, tau=tau, ert_scope=scope), out)
            torch.cuda.synchronize()
            said = capfd.readouterr().err
            if env["VR_MARCH"] == "ring":
                # (perspective fronts of whole-ray termination: never cells)
                assert ("cells" in said) == (few == 0.5 and not (eye and scope)), said
            images.append(out)
        vr.vr_volume_destroy(h)
        vr.vr_destroy(ctx)
    assert float(images[0].abs().max()) > 0
    assert torch.equal(images[0], images[2]) and torch.equal(images[1], images[3])
