"""Tuned occupancies of the batched launch in VR_TUNE_CACHE: a limit that was written
for a grid of resident workgroups does not cap the launch of a workgroup per item,
the launch without a limit is the default the tuner compares with, and a limit
written now is read back."""
import os

import pytest

import synth

pytestmark = pytest.mark.gpu


def test_occupancy_entries(tmp_path):
    import torch
    torch.cuda.init()
    import paper_1008_0135_amd as vr
    cache = tmp_path / "tune"

    def context():
        os.environ["VR_TUNE_CACHE"] = str(cache)
        try:
            return vr.vr_create(0)
        finally:
            del os.environ["VR_TUNE_CACHE"]

    def retune(c):
        """Any tuning writes what the context has read."""
        os.environ["VR_TUNE_CACHE"] = str(cache)
        try:
            h = vr.vr_volume_create(c, synth.cube(20, 22, 24, seed=1, n_sources=2, sigma_range=(1.5, 3.0)), (20, 22, 24))
            vr.vr_tf_set(c, synth.tf_ramp(32))
            vr.vr_autotune(c, h, vr.make_view(synth.rot_axis(1, 20.0), 40, 30), vr.make_params())
            vr.vr_volume_destroy(h)
        finally:
            del os.environ["VR_TUNE_CACHE"]
        return [line.split()[:2] for line in cache.read_text().splitlines() if line.startswith("batch/waves")]

    cache.write_text("batch/waves_per_cu 8 0 0 0\n")
    c = context()
    assert retune(c) == []
    vr.vr_destroy(c)
    cache.write_text("batch/waves_at_most 4 0 0 0\n")
    c = context()
    assert retune(c) == [["batch/waves_at_most", "4"]]
    h = vr.vr_volume_create(c, synth.cube(60, 62, 64, seed=1, n_sources=2, sigma_range=(1.5, 3.0)), (60, 62, 64))
    t = torch.from_numpy(synth.tf_ramp(32)).cuda()
    outs = [torch.empty((90, 100, 4), device="cuda") for _ in range(8)]
    reqs = [vr.make_request(h, R, 100, 90, t, 0.0, 0.0, o) for R, o in zip(synth.random_views(8, 2), outs)]
    res, batch = vr.vr_autotune_batch(c, reqs, vr.make_params())
    assert res.ms <= res.ms_default and res.waves_per_cu in (2, 4, 8, 16, 32)
    assert (res.ms == res.ms_default) == (res.waves_per_cu == 32)
    assert retune(c) == [["batch/waves_at_most", str(res.waves_per_cu)]]
    torch.cuda.synchronize()
    vr.vr_batch_destroy(batch)
    vr.vr_volume_destroy(h)
    vr.vr_destroy(c)
