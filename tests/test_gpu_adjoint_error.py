"""How far the gradients are from 64 bits for tables that change fast, where the
rounding of a sample's position shows.  Views saved by gathers, in parts and not:
their checkpoints and sums are of the adjoint's own samples, so that what is left is
the storage of T and of the voxel gradients in single precision (2^-24 each, a few
terms an entry): a root mean square of 5e-7 of the gradient's.  Views saved by
footprint cells, whose checkpoints are the image's transmittance: no further off than
the sample-segment adjoint, which replays from that."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M = 256
S = np.linspace(0, 1, M)
TABLES = {"ramp": 0.25 * S, "bump": 0.2 * np.exp(-((S - 0.5) / 0.2) ** 2), "step": np.where(S > 0.4, 0.2, 0.0),
          "opaque step": np.where(S > 0.4, 0.6, 0.0)}


def _errors(march, dims, image, kind, alpha, colours, capfd):
    import oracle
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    env = {"VR_DEBUG_PLAN": "1"}
    if march:
        env["VR_MARCH"] = march
    os.environ.update(env)
    try:
        ctx = vr.vr_create(0)
    finally:
        for k in env:
            del os.environ[k]
    W, H = image
    rng = np.random.default_rng(1)
    vol = rng.standard_normal(dims[::-1]).astype(np.float32) if kind == "noise" else \
        synth.cube(*dims, seed=6, n_sources=4, sigma_range=(1.5, 4.0))
    tf = synth.tf_colour(M)
    if colours == "random":
        tf[:, :3] = rng.uniform(0, 1, (M, 3))
    tf[:, 3] = TABLES[alpha]
    vmin, vmax = float(vol.min()), float(vol.max())
    views = synth.random_views(1, 7)
    gout = rng.normal(0, 1, (1, H, W, 4)).astype(np.float32)
    a = torch.from_numpy(vol).cuda()
    h = vr.vr_volume_create(ctx, a, dims)
    vr.vr_tf_set(ctx, tf, vmin, vmax)
    out = torch.empty((1, H, W, 4), device="cuda")
    capfd.readouterr()
    st = vr.vr_render(ctx, h, [vr.make_view(R, W, H) for R in views], vr.make_params(tau=2.0, ess=0), out, save=True)
    said = capfd.readouterr().err
    gtf, gvol = torch.empty((M, 4), device="cuda"), torch.empty_like(a)
    vr.vr_render_backward(ctx, h, st, torch.from_numpy(gout).cuda(), gtf, gvol)
    torch.cuda.synchronize()
    vr.vr_state_destroy(st)
    vr.vr_volume_destroy(h)
    vr.vr_destroy(ctx)
    rtf, rvol, _ = oracle.render_grad(vol, tf, views[0], W, H, gout[0].astype(np.float64), vmin, vmax, tau=2.0)
    return said, [float(np.sqrt(((g.cpu().numpy() - r) ** 2).mean() / (r ** 2).mean())) for g, r in ((gtf, rtf), (gvol, rvol))]


@pytest.mark.parametrize("alpha", list(TABLES))
@pytest.mark.parametrize("colours", ["smooth", "random"])
@pytest.mark.parametrize("kind", ["noise", "sources"])
@pytest.mark.parametrize("image,parts", [((60, 50), True), ((400, 380), False)])
def test_gathers(alpha, colours, kind, image, parts, capfd):
    said, err = _errors(None, (96, 90, 100) if parts else (60, 64, 50), image, kind, alpha, colours, capfd)
    assert "saved by gathers" in said and ("1 parts" not in said or "11 parts" in said) == parts, said
    assert max(err) <= 5e-7, err


@pytest.mark.parametrize("alpha", ["ramp", "bump"])
@pytest.mark.parametrize("kind", ["noise", "sources"])
def test_cells(alpha, kind, capfd):
    said, err = _errors("ring", (96, 90, 100), (120, 110), kind, alpha, "smooth", capfd)
    assert "saved by cells" in said
    _, ref = _errors("gather", (96, 90, 100), (120, 110), kind, alpha, "smooth", capfd)
    for e, r in zip(err, ref):
        assert e <= 1.5 * r + 1e-7, (err, ref)
