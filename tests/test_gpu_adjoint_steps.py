"""The adjoint where a ray's next sample lies beyond the next group of cell
layers: groups in which a ray has no sample still hold its transmittance, since
the group in front of them ends there.  Gradients against the FP64 oracle (the
bound of the other gradient tests) and, for the forward by footprint cells with
pixels past a cell's 64th, against the sample-segment adjoint."""
import os

import numpy as np
import pytest

import synth
from test_gpu_adjoint_tiles import _check, _table, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,step", [(32, 4.0), (1, 2.0), (32, 7.5), (4, 3.0), (32, 3.0)])
@pytest.mark.parametrize("amax,tau", [(0.2, 2.0), (0.2, 0.7), (0.6, 2.0)])
@pytest.mark.parametrize("dims", [(24, 20, 28), (70, 60, 100)])
def test_skipped_groups(ctx, K, step, amax, tau, dims):  # noqa: F811
    views = synth.random_views(2, 9) + [np.eye(3) @ synth.rot_axis(3, 10.0)]
    _check(ctx, dims, (33, 30), views, _table(32, amax), tau=tau, K=K, step=step)


@pytest.mark.parametrize("step", [0.5, 4.0])
def test_skipped_groups_past_the_cells(step, capfd):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    dims, (W, H) = (300, 200, 260), (384, 380)
    a = torch.from_numpy(synth.cube(*dims, seed=6, n_sources=3)).cuda()
    views = [vr.make_view(R, W, H) for R in synth.random_views(3, 4)]
    gout = torch.from_numpy(np.random.default_rng(8).normal(0, 1, (3, H, W, 4)).astype(np.float32)).cuda()
    grads = []
    for env in ({"VR_MARCH": "ring", "VR_FOOT_RAYS": "64", "VR_FOOT_MAXPX": "4096"}, {"VR_MARCH": "gather"}):
        env["VR_DEBUG_PLAN"] = "1"
        os.environ.update(env)
        try:
            c = vr.vr_create(0)
        finally:
            for k in env:
                del os.environ[k]
        h = vr.vr_volume_wrap(c, a, dims)
        vr.vr_tf_set(c, _table(64, 0.03), float(a.min()), float(a.max()))  # (taken by division)
        out = torch.empty((3, H, W, 4), device="cuda")
        capfd.readouterr()
        st = vr.vr_render(c, h, views, vr.make_params(step=step, tau=2.0, ess=0), out, save=True)
        assert capfd.readouterr().err.count("saved by cells") == (3 if env["VR_MARCH"] == "ring" else 0)
        gtf, gvol = torch.empty((64, 4), device="cuda"), torch.empty_like(a)
        vr.vr_render_backward(c, h, st, gout, gtf, gvol)
        torch.cuda.synchronize()
        vr.vr_state_destroy(st)
        vr.vr_volume_destroy(h)
        vr.vr_destroy(c)
        grads.append((gtf, gvol))
    for g, r in zip(*grads):
        g, r = g.double(), r.double()
        scale = r.abs().clamp(min=1e-3 * float(r.abs().max()))
        assert float(((g - r).abs() / scale).max()) <= 1e-3
