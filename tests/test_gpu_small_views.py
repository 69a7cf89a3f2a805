"""Views of a few thousand samples: the fixed cost of a view by footprint cells is
part of their estimate, so gathers march them -- masked, unmasked and maximum
intensity projection -- with the bits of the cells."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _context(vr, **env):
    env["VR_DEBUG_PLAN"] = "1"
    os.environ.update(env)
    try:
        return vr.vr_create(0)
    finally:
        for k in env:
            del os.environ[k]


@pytest.mark.parametrize("dims,image,nv,step", [((24, 23, 14), (21, 29), 1, 0.25), ((14, 13, 32), (28, 33), 2, 1.0),
                                                ((14, 215, 12), (149, 171), 2, 0.5)])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("masked", [False, True])
def test_gathers_take_small_views(dims, image, nv, step, mode, masked, capfd):
    import torch
    import paper_1008_0135_amd as vr
    a = torch.from_numpy(synth.cube(*dims, seed=4, n_sources=4, sigma_range=(1.5, 4.0))).cuda()
    mask = np.linspace(0.2, 1.0, dims[2], dtype=np.float32) if masked else None
    got = []
    for c, gathers in ((_context(vr), nv), (_context(vr, VR_MARCH="ring"), 0)):
        h = vr.vr_volume_create(c, a, dims)
        vr.vr_tf_set(c, synth.tf_colour(64), float(a.min()), float(a.max()))
        vr.vr_mask_set(c, mask)
        out = torch.full((nv, image[1], image[0], 4), 7.0, device="cuda")
        capfd.readouterr()
        vr.vr_render(c, h, [vr.make_view(R, *image) for R in synth.random_views(nv, 9)],
                     vr.make_params(step=step, tau=0.95, mode=mode), out)
        torch.cuda.synchronize()
        said = capfd.readouterr().err
        assert said.count("gathers lanes") == gathers, said
        got.append(out)
        vr.vr_volume_destroy(h)
        vr.vr_destroy(c)
    assert torch.equal(*got)
