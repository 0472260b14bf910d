"""GPU image metrics on regions of awkward sizes: discs of many columns and depth
runs, clipped at the image's edges, of a few pixels and off the image, with NaN
around them, and points whose half level lies more than one wavefront's 64 pixels
away or past the image's edge, against the float64 oracle metrics on the same image.
Statistics are float32 sums over at most 70 000 pixels in 512 partial sums: relative
1e-5."""

import math

import numpy as np
import pytest

from cases import geom
from metric_checks import _split
from oracle import metrics as om

pytestmark = pytest.mark.gpu


def _grid(nx, nz):
    return geom(nx=nx, nz=nz, x_min=-nx * 0.05e-3, x_max=nx * 0.05e-3, z_min=5e-3,
                z_max=5e-3 + nz * 0.1e-3)


def _disc(g, ix, iz, r):
    """A disc of radius r pixels around pixel (ix, iz) of _grid's 0.1 mm pixels."""
    x0, z0 = -g.nx * 0.05e-3, 5e-3
    return x0 + (ix + 0.5) * 0.1e-3, z0 + (iz + 0.5) * 0.1e-3, r * 0.1e-3


@pytest.mark.parametrize("nx, nz, inner, outer", [
    (321, 401, (150.31, 200.27, 139.53), (160.1, 190.7, 149.41)),  # five depth runs
    (257, 130, (0.2, 60.1, 31.77), (255.7, 65.3, 32.21)),        # at the left, at the right
    (97, 65, (48.3, 0.4, 40.13), (48.1, 63.8, 63.87)),           # at the top, at the bottom
    (64, 64, (30.2, 30.1, 0.73), (40.4, 30.3, 1.61)),            # one pixel, a few
    (40, 700, (20.3, 350.2, 400.3), (20.3, 350.2, 331.9)),       # taller than the image is wide
])
def test_contrast_regions(nx, nz, inner, outer):
    import torch
    from paper_2311_00482_amd import contrast_metrics
    g = _grid(nx, nz)
    env = np.random.default_rng(nx * 1000 + nz).rayleigh(20.0, (nx, nz)).astype(np.float32)
    cyst = (_disc(g, *inner), _disc(g, *outer))
    for disc in cyst:
        assert not _split(g, disc)[1].any()  # every pixel is decided alike
    out = ~(_split(g, cyst[0])[0] | _split(g, cyst[1])[0])
    env[out] = np.nan  # no pixel outside the discs may count
    got = contrast_metrics(g, torch.from_numpy(env).cuda(), [cyst])[0]
    ref = om.contrast(g, env, *cyst)
    assert (got["n_in"], got["n_out"]) == (ref["n_in"], ref["n_out"])
    for k in ("mu_in", "mu_out", "sigma_in", "sigma_out"):
        assert got[k] == pytest.approx(ref[k], rel=1e-5), k
    # both discs show the same speckle, so the difference of their means cancels: the
    # figures formed from the statistics are held to the statistics returned
    mi, mo, si, so = (got[k] for k in ("mu_in", "mu_out", "sigma_in", "sigma_out"))
    assert got["cr_db"] == pytest.approx(20.0 * math.log10(mi / mo), abs=1e-5)
    assert got["cnr"] == pytest.approx((mi - mo) / math.sqrt(0.5 * (si * si + so * so)), rel=1e-5)


def test_contrast_off_the_image():
    import torch
    from paper_2311_00482_amd import contrast_metrics
    g = _grid(64, 80)
    env = torch.rand(64, 80, device="cuda") + 1.0
    got = contrast_metrics(g, env, [(_disc(g, 500, 40, 9.3), _disc(g, 30, 40, 9.3))])[0]
    assert got["n_in"] == 0 and got["n_out"] > 0
    assert math.isnan(got["mu_in"]) and math.isnan(got["cr_db"]) and math.isnan(got["cnr"])


@pytest.mark.parametrize("ix, iz, sx, sz", [
    (200, 190, 90.0, 100.0),  # half level past several runs of 64 pixels, every way
    (200, 190, 54.35, 54.4),  # next to the 64th pixel
    (3, 190, 40.0, 9.0),      # the left half level is past the edge
    (200, 397, 9.0, 40.0),    # the lower half level is past the edge
    (0, 0, 1.5, 1.5),
])
def test_resolution_walks(ix, iz, sx, sz):
    import torch
    from paper_2311_00482_amd import resolution_metrics
    g = _grid(401, 400)
    x, z = np.arange(401)[:, None] - ix, np.arange(400)[None, :] - iz
    env = (100.0 * np.exp(-(x / sx) ** 2 - (z / sz) ** 2)).astype(np.float32)
    target = _disc(g, ix + 0.21, iz + 0.13, 2.6)
    got = resolution_metrics(g, torch.from_numpy(env).cuda(), [target])[0]
    ref = om.resolution(g, env, target)
    assert (got["ix"], got["iz"]) == (ref["ix"], ref["iz"]) == (ix, iz)
    assert got["peak"] == ref["peak"]
    for k in ("fwhm_x", "fwhm_z"):
        if math.isnan(ref[k]):
            assert math.isnan(got[k]), k
        else:
            assert got[k] == pytest.approx(ref[k], rel=1e-5), k
