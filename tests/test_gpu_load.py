"""Opening volumes: copy and range in one pass, brick and macrocell ranges, the
permuted copy's ranges taken from the source's, and memory of destroyed
volumes used again."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    c = vr.vr_create(0)
    yield c
    vr.vr_destroy(c)


def _ranges(vr, h):
    return [(b.slo[:], b.shi[:], b.vmin, b.vmax) for b in vr.vr_volume_brick_info(h)]


def _check(vr, h, a, edge):
    assert vr.vr_volume_minmax(h) == (a.min(), a.max())
    for slo, shi, mn, mx in _ranges(vr, h):
        part = a[slo[2]:shi[2] + 1, slo[1]:shi[1] + 1, slo[0]:shi[0] + 1]
        assert (mn, mx) == (part.min(), part.max())
    e, cnt, mm = vr.vr_volume_macrocell_info(h)
    assert e == edge
    n3, n2, n1 = a.shape
    for m in np.ndindex(cnt[2], cnt[1], cnt[0]):
        z, y, x = (slice(k * e, min((k + 1) * e, n - 1) + 1) for k, n in zip(m, (n3, n2, n1)))
        assert tuple(mm[m]) == (a[z, y, x].min(), a[z, y, x].max())


# 2: the smallest axis; 257, 1030: rows longer than a workgroup; 33, 131: past the transpose tiles
@pytest.mark.parametrize("dims", [(2, 3, 2), (33, 131, 9), (257, 40, 21), (64, 64, 64), (1030, 17, 5)])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("split", [False, True])
def test_ranges(ctx, dims, offset, split):
    import torch
    import paper_1008_0135_amd as vr
    n = dims[0] * dims[1] * dims[2]
    flat = torch.randn(n + 4, generator=torch.Generator().manual_seed(n)).cuda()
    src = flat[offset:offset + n]  # offset 1: not 16-byte aligned
    a = src.cpu().numpy().reshape(dims[2], dims[1], dims[0])
    h = vr.vr_volume_create(ctx, src, dims)
    spec = vr.kd_spec(2, macrocell=4, twin=True) if split else vr.grid_spec((20, 7, 3), macrocell=4, twin=True)
    vr.vr_volume_brick(h, spec)
    _check(vr, h, a, 4)
    vr.vr_volume_destroy(h)


def test_nonfinite_in_the_tail(ctx):
    import torch
    import paper_1008_0135_amd as vr
    x = torch.zeros(5 * 7 * 3, device="cuda")
    x[-1] = float("nan")  # past the last whole group of four
    with pytest.raises(vr.VRError):
        vr.vr_volume_create(ctx, x, (5, 7, 3))


@pytest.mark.parametrize("split", [False, True])
def test_skipping_in_the_permuted_copy(ctx, split):
    """A view along axis 1 rendered from the permuted copy, whose brick and
    macrocell ranges are the source's permuted, against the unskipped render of
    the same copy: skipped samples add nothing."""
    import torch
    import paper_1008_0135_amd as vr
    dims = (70, 90, 55)
    a = synth.cube(*dims, seed=9, n_sources=3)
    h = vr.vr_volume_create(ctx, torch.from_numpy(a).cuda(), dims)
    opt = dict(macrocell=8, twin=True)
    vr.vr_volume_brick(h, vr.kd_spec(5, **opt) if split else vr.grid_spec((24, 40, 16), **opt))
    vr.vr_tf_set(ctx, synth.tf_noise_suppress(float(a.min()), float(a.max())))
    R = synth.rot_axis(2, 80.0) @ synth.rot_axis(3, 10.0)
    assert abs(R[2][0]) > 0.9
    out = torch.empty((2, 1, 96, 96, 4), device="cuda")
    for ess in (0, 1):
        vr.vr_render(ctx, h, [vr.make_view(R, 96, 96)], vr.make_params(ess=ess), out[ess])
    torch.cuda.synchronize()
    assert float(out[0].abs().max()) > 0.0
    assert torch.equal(out[0], out[1])
    vr.vr_volume_destroy(h)


def test_memory_used_again():
    """Volumes of changing sizes through two contexts, opened and closed in
    turn: each holds its own voxels, whatever block it was given."""
    import torch
    import paper_1008_0135_amd as vr
    ctxs = [vr.vr_create(0), vr.vr_create(0)]
    rng = np.random.default_rng(3)
    live = []
    for i in range(24):
        dims = tuple(int(v) for v in rng.integers(20, 140, 3))
        a = rng.standard_normal(dims[::-1]).astype(np.float32) + i
        h = vr.vr_volume_create(ctxs[i % 2], torch.from_numpy(a).cuda(), dims)
        vr.vr_volume_brick(h, vr.grid_spec((64, 64, 64), macrocell=16, twin=True, materialize=i % 3 == 0))
        live.append((h, a))
        if len(live) > 3:
            h, a = live.pop(int(rng.integers(len(live))))
            _check(vr, h, a, 16)
            vr.vr_volume_destroy(h)
    for h, a in live:
        _check(vr, h, a, 16)
        vr.vr_volume_destroy(h)
    for c in ctxs:
        vr.vr_destroy(c)
