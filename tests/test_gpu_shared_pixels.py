"""GPU parity of single-frame plans whose wavefronts share a pixel's channels (two,
four or eight to a pixel, with one lane group and with several): whole images
against the FP64 oracle at the 1e-5 bar. The plan's block size shows how many
share; channel counts leave the last of them with fewer channels."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5

FINE = dict(x_min=-1.5e-3, x_max=1.5e-3, z_min=3e-3, z_max=6e-3)
CASES = [
    # name, mode, angles, channels, geometry, wavefronts per pixel
    ("das_1a", "das", 1, 37, dict(nx=33, nz=60, **FINE), 8),
    ("das_1a_boxcar", "das", 1, 64, dict(nx=33, nz=60, apod="boxcar", **FINE), 8),
    ("das_few_channels", "das", 1, 9, dict(nx=33, nz=60, **FINE), 2),
    ("das_9a", "das", 9, 41, dict(nx=29, nz=50, **FINE), 8),
    ("das_32a_sums_in_lds", "das", 32, 33, dict(nx=17, nz=30, **FINE), 8),
    ("das_2_per_pixel", "das", 1, 24, dict(nx=300, nz=400, x_min=-4e-3, x_max=4e-3, z_min=3e-3,
                                           z_max=12e-3), 2),
    ("das_coarse_lane_groups", "das", 1, 64, dict(nx=40, nz=12, x_min=-9e-3, x_max=9e-3,
                                                  z_min=3e-3, z_max=12e-3), 2),
    ("dmas_1a", "dmas", 1, 39, dict(nx=33, nz=60, **FINE), 4),
    ("dmas_7a", "dmas", 7, 39, dict(nx=33, nz=60, **FINE), 4),
    ("pdas_5a", "pdas", 5, 39, dict(nx=33, nz=60, **FINE), 4),
    ("iqdas_1a", "iqdas", 1, 39, dict(nx=33, nz=60, n_samples=512, **FINE), 8),
    ("iqdas_11a", "iqdas", 11, 38, dict(nx=33, nz=60, n_samples=512, **FINE), 2),
    ("bbdmas_3a", "bbdmas", 3, 39, dict(nx=33, nz=60, n_samples=512, **FINE), 8),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_shared_pixels(case):
    import torch
    from paper_2311_00482_amd import beamform, describe_plan, iq_demodulate
    name, mode, n, channels, kw, least = case
    g = geom(angles_deg=tuple(np.linspace(-9.0, 8.0, n)) if n > 1 else (2.0,),
             n_channels=channels, **kw)
    p = describe_plan(g, mode, -1)
    share = p["threads_per_block"] // (64 * p["wz"] * p["wx"])
    assert share >= least, p
    rf = rand_rf(g, 700 + n + channels)
    dev = torch.from_numpy(rf).cuda()
    iq = mode in ("iqdas", "bbdmas")
    want = ("rf", "imag", "env", "log") if iq else ("rf",)
    src = iq_demodulate(g, dev) if iq else dev
    out = beamform(g, src, mode, -1, want=want)
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    if iq:
        got = got + 1j * out["imag"].cpu().numpy()
        ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1,
                                 parallel=True)
        env = np.abs(ref)
        assert np.abs(out["env"].cpu().numpy() - env).max() <= TOL32 * env.max()
        assert float(out["log"].max()) == 0.0  # the frame maximum comes from every tile
    else:
        ref = oracle.beamform(g, rf, mode, -1)["rf"]
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max(), name
