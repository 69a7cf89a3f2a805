"""vr_render_backward has waited for its stream when it returns, whatever the
table: its caller may read the gradients from any stream, or free what it passed."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("amax", [0.1, 0.5])  # division by 1 - a, replay
@pytest.mark.parametrize("nviews", [1, 4])
def test_stream_is_idle(amax, nviews):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    ctx = vr.vr_create(0)
    dims = (256, 240, 250)
    a = torch.from_numpy(synth.cube(*dims, seed=6, n_sources=3)).cuda()
    h = vr.vr_volume_wrap(ctx, a, dims)
    tf = synth.tf_colour(64)
    tf[:, 3] = np.linspace(0, amax, 64)
    vr.vr_tf_set(ctx, tf, float(a.min()), float(a.max()))
    out, gout = (torch.ones((nviews, 320, 320, 4), device="cuda") for _ in range(2))
    gtf, gvol = torch.empty((64, 4), device="cuda"), torch.empty_like(a)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    st = vr.vr_render(ctx, h, [vr.make_view(R, 320, 320) for R in synth.random_views(nviews, 4)],
                      vr.make_params(tau=2.0, ess=0), out, stream=s, save=True)
    vr.vr_render_backward(ctx, h, st, gout, gtf, gvol, stream=s)
    idle = s.query()
    torch.cuda.synchronize()
    vr.vr_state_destroy(st)
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
    assert idle
