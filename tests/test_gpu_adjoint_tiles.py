"""The ring adjoint at the edges of its tiles and groups, and on both sides of
the opacity above which it replays a group instead of dividing by 1 - a:
table and voxel gradients against the FP64 oracle's exact gradient, relative
error <= 1e-3 with the scale floor 1e-3 max|g| (the bound of the other gradient
tests; what limits both sides of the line is the forward's single-precision
transmittance)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    c = vr.vr_create(0)
    yield c
    vr.vr_destroy(c)


def _check(ctx, dims, image, views, tf, tau=2.0, K=32, step=0.5, seed=6):
    import oracle
    import torch
    import paper_1008_0135_amd as vr
    W, H = image
    vol = synth.cube(*dims, seed=seed, n_sources=3, sigma_range=(2.0, 4.0), band=False)
    vmin, vmax = float(vol.min()) - 0.5, float(vol.max()) + 0.5
    gout = np.random.default_rng(8).normal(0, 1, (len(views), H, W, 4))
    if tau < 1:
        # rays that may stop one sample apart on the two sides get no gradient
        ref = oracle.render(vol, tf, views, W, H, vmin, vmax, tau=tau, step=step)
        gout[(ref["flags"] & oracle.FLAG_ERT) != 0] = 0.0
    dvol = torch.from_numpy(vol).cuda()
    h = vr.vr_volume_wrap(ctx, dvol, dims)
    vr.vr_tf_set(ctx, tf, vmin, vmax)
    out = torch.empty((len(views), H, W, 4), device="cuda")
    p = vr.make_params(step=step, tau=tau, ckpt_K=K, ess=0)
    st = vr.vr_render(ctx, h, [vr.make_view(R, W, H) for R in views], p, out, save=True)
    # the ring layout, unless a tile's rays span so many voxels that its windows do not fit
    assert vr.vr_state_info(st, 0)[0] or max(dims) > 4 * min(image)
    gtf, gvol = torch.empty((tf.shape[0], 4), device="cuda"), torch.empty_like(dvol)
    vr.vr_render_backward(ctx, h, st, torch.from_numpy(gout.astype(np.float32)).cuda(), gtf, gvol)
    torch.cuda.synchronize()
    vr.vr_state_destroy(st)
    vr.vr_volume_destroy(h)
    gout = gout.astype(np.float32).astype(np.float64)
    otf, ovol = np.zeros((tf.shape[0], 4)), np.zeros(vol.shape)
    for j, R in enumerate(views):
        a, b, _ = oracle.render_grad(vol, tf, R, W, H, gout[j], vmin, vmax, tau=tau, step=step)
        otf += a
        ovol += b
    for g, ref in ((gtf, otf), (gvol, ovol)):
        g = g.cpu().numpy().astype(np.float64)
        scale = max(1e-3 * float(np.abs(ref).max()), 1e-30)
        assert float((np.abs(g - ref) / np.maximum(np.abs(ref), scale)).max()) <= 1e-3


def _table(M, amax):
    tf = synth.tf_colour(M)
    tf[:, 3] = np.linspace(0, amax, M, dtype=np.float32)
    return tf


# images below, at and past a tile of 8 x 8 rays
@pytest.mark.parametrize("image", [(1, 1), (8, 8), (9, 23)])
@pytest.mark.parametrize("dims", [(12, 11, 13), (40, 33, 50)])
@pytest.mark.parametrize("amax", [0.25, 0.26])  # division up to 1/4, replay above
def test_tiles_and_opacity(ctx, image, dims, amax):
    _check(ctx, dims, image, synth.random_views(2, 4), _table(32, amax))


def test_smallest_table(ctx):
    _check(ctx, (20, 18, 22), (30, 28), synth.random_views(1, 4), _table(2, 0.1))


def test_opaque_entries(ctx):
    # opacity 1: nothing behind such a sample counts (T = 0 exactly)
    tf = _table(32, 0.3)
    tf[20:, 3] = 1.0
    _check(ctx, (24, 20, 28), (33, 30), synth.random_views(2, 9), tf)


# groups of one layer to the cap, samples per layer from 1 to many (step 0.1);
# early termination inside a group
@pytest.mark.parametrize("K,step", [(1, 0.5), (32, 2.0), (32, 0.1)])
@pytest.mark.parametrize("amax,tau", [(0.2, 2.0), (0.2, 0.9), (0.6, 0.9)])
def test_groups(ctx, K, step, amax, tau):
    _check(ctx, (24, 20, 28), (33, 30), synth.random_views(2, 9), _table(32, amax), tau=tau, K=K, step=step)


def test_views_along_the_axes(ctx):
    # along +-axis 2 and 3: rays on voxel planes, both marching directions
    views = [np.eye(3), synth.rot_axis(1, 180.0), synth.rot_axis(1, 90.0), synth.rot_axis(1, -90.0)]
    _check(ctx, (20, 22, 24), (16, 18), [v @ synth.rot_axis(3, 10.0) for v in views], _table(32, 0.1))
