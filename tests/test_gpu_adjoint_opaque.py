"""Rays that become opaque with early termination off: the transmittance falls far
below the rounding of 1, the gradients stay finite and those of the FP64 oracle
(relative error <= 1e-3, scale floor 1e-3 max|g|: the bound of the other gradient
tests).  The images are small, so that several workgroups share a tile, each
starting behind what lies in front of its part."""
import numpy as np
import pytest

import synth
from test_gpu_adjoint_tiles import _check, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


# one opacity for every sample, on both sides of the line of the replay; a ray of
# 270 samples is left with (1 - a)^270: 1e-7 to 1e-270
@pytest.mark.parametrize("alpha", [0.06, 0.1, 0.15, 0.25, 0.3, 0.6, 0.9])
def test_opaque_rays(ctx, alpha):  # noqa: F811
    tf = synth.tf_colour(32)
    tf[:, 3] = alpha
    _check(ctx, (70, 60, 100), (24, 20), synth.random_views(2, 4), tf)


def test_opaque_layer(ctx):  # noqa: F811
    # opacities from 0 to 0.95: rays stop mattering at different depths
    tf = synth.tf_colour(32)
    tf[:, 3] = np.linspace(0, 0.95, 32)
    _check(ctx, (70, 60, 100), (24, 20), synth.random_views(2, 5), tf)
