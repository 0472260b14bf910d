"""FWHM of peaks below zero (images in dB, for instance): such a peak lies below its own
half, so both crossings are sought between the peak and its neighbours, and at the
image's edge, where a neighbour is missing, the width is NaN. Elsewhere the float64
oracle's figures; the pixel values and crossings are exact in float32, so the only
roundings are the pixel step's and the product's, 6e-8 each: relative 1e-6."""

import math

import numpy as np
import pytest

from cases import geom
from oracle import metrics as om

pytestmark = pytest.mark.gpu

NX, NZ = 70, 90


@pytest.mark.parametrize("ix", [0, 1, 30, NX - 2, NX - 1])
@pytest.mark.parametrize("iz", [0, 1, 40, NZ - 2, NZ - 1])
def test_negative_peak(ix, iz):
    import torch
    from paper_2311_00482_amd import resolution_metrics
    g = geom(nx=NX, nz=NZ, x_min=-NX * 0.05e-3, x_max=NX * 0.05e-3, z_min=5e-3,
             z_max=5e-3 + NZ * 0.1e-3)
    x, z = np.arange(NX)[:, None] - ix, np.arange(NZ)[None, :] - iz
    env = (-2.0 ** np.minimum(np.abs(x) + np.abs(z), 20)).astype(np.float32)
    target = (-NX * 0.05e-3 + (ix + 0.5) * 0.1e-3, 5e-3 + (iz + 0.5) * 0.1e-3, 0.23e-3)
    got = resolution_metrics(g, torch.from_numpy(env).cuda(), [target])[0]
    assert (got["ix"], got["iz"], got["peak"]) == (ix, iz, -1.0)
    for k, at, n, line, step in (("fwhm_x", ix, NX, env[:, iz], g.dx),
                                 ("fwhm_z", iz, NZ, env[ix], g.dz)):
        if 0 < at < n - 1:
            assert got[k] == pytest.approx(om._half_width(line, at, -0.5) * step, rel=1e-6), k
        else:
            assert math.isnan(got[k]), k
