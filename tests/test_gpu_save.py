"""The checkpointing forward by footprint cells and by gathers, and the adjoint
with one and with several workgroups per tile: the image bit for bit that of
the plain render, the gradients those of the sample-segment adjoint (the march
VR_MARCH=gather selects) to 1e-3 of each entry, floor 1e-3 max|g|: the bound of
the other gradient tests."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _step(dims, image, nviews, tau, mode=None):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    if mode:
        os.environ["VR_MARCH"] = mode
    try:
        ctx = vr.vr_create(0)
    finally:
        os.environ.pop("VR_MARCH", None)
    W, H = image
    vol = torch.from_numpy(synth.cube(*dims, seed=6, n_sources=3)).cuda()
    h = vr.vr_volume_wrap(ctx, vol, dims)
    tf = synth.tf_colour(64)
    tf[:, 3] = np.linspace(0, 0.2, 64)
    vr.vr_tf_set(ctx, tf, float(vol.min()), float(vol.max()))
    views = [vr.make_view(R, W, H) for R in synth.random_views(nviews, 4)]
    p = vr.make_params(tau=tau, ess=0)
    plain, out = (torch.full((nviews, H, W, 4), 7.0, device="cuda") for _ in range(2))
    vr.vr_render(ctx, h, views, p, plain)
    st = vr.vr_render(ctx, h, views, p, out, save=True)
    gout = torch.from_numpy(np.random.default_rng(8).normal(0, 1, (nviews, H, W, 4)).astype(np.float32)).cuda()
    gtf, gvol = torch.empty((64, 4), device="cuda"), torch.empty_like(vol)
    vr.vr_render_backward(ctx, h, st, gout, gtf, gvol)
    torch.cuda.synchronize()
    ring = vr.vr_state_info(st, 0)[0]
    vr.vr_state_destroy(st)
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
    return plain, out, gtf, gvol, ring


# gathers with several workgroups per tile, with one, footprint cells, and rays
# too far apart for windows
@pytest.mark.parametrize("dims,image,nviews", [((61, 83, 72), (100, 92), 2), ((5, 9, 40), (17, 12), 1),
                                               ((60, 64, 50), (420, 400), 2), ((300, 200, 260), (384, 380), 3),
                                               ((80, 82, 238), (21, 23), 3)])
@pytest.mark.parametrize("tau", [2.0, 0.9])
def test_save(dims, image, nviews, tau):
    import torch
    plain, out, gtf, gvol, ring = _step(dims, image, nviews, tau)
    _, _, rtf, rvol, segments = _step(dims, image, nviews, tau, "gather")
    assert ring and not segments
    assert torch.equal(plain, out)
    for g, r in ((gtf, rtf), (gvol, rvol)):
        g, r = g.double(), r.double()
        scale = r.abs().clamp(min=1e-3 * float(r.abs().max()))
        assert float(((g - r).abs() / scale).max()) <= 1e-3
