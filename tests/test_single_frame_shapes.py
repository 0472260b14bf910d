"""The library's own launch shapes of single frames: how many wavefronts share a pixel's
channels and how large the tiles are, at sizes on either side of the limits (the shapes
that were measured faster there), and GPU parity of a launch large enough for the
register-bound kernels of 13 to 16 angles that share pixels."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

TOL32 = 1e-5


def _plan(mode, n, channels, nx, nz, **kw):
    from paper_2311_00482_amd import describe_plan
    width = min(channels * 0.3e-3, nx * 0.5e-3)
    g = geom(angles_deg=tuple(np.linspace(-8.0, 8.0, n)) if n > 1 else (2.0,), nx=nx, nz=nz,
             n_channels=channels, n_samples=2048, x_min=-0.5 * width, x_max=0.5 * width,
             z_min=5e-3, z_max=5e-3 + nz * 60e-6, f_number=1.5, **kw)
    p = describe_plan(g, mode, -1)
    share = p["threads_per_block"] // (64 * p["wz"] * p["wx"])
    return p, share


@pytest.mark.parametrize("mode, n, channels, nx, nz, share", [
    ("das", 1, 128, 128, 128, 8),   # a block of eight wavefronts for each compute unit
    ("das", 1, 128, 130, 150, 4),
    ("das", 1, 64, 300, 300, 2),
    ("das", 1, 64, 512, 400, 1),
    ("das", 3, 16, 300, 400, 1),    # too few channels to share
    ("das", 3, 48, 512, 512, 1),    # windows that leave room for four blocks
    ("das", 11, 128, 128, 256, 8),
    ("das", 11, 64, 300, 400, 4),
    ("das", 11, 128, 384, 384, 2),
    ("das", 14, 16, 800, 700, 1),   # registers leave no room for more wavefronts
    ("dmas", 3, 16, 512, 512, 1),   # every sharing wavefront would fill a table
    ("pdas", 5, 32, 700, 600, 1),
    ("iqdas", 11, 32, 128, 256, 1),
    ("iqdas", 24, 64, 130, 150, 1),
    ("iqdas", 5, 128, 130, 150, 4),
    ("iqdas", 5, 62, 722, 90, 2),   # more wavefronts than lane groups are good for
    ("bbdmas", 11, 90, 210, 420, 2),
    ("bbdmas", 11, 90, 500, 300, 2),
    ("iqdas", 5, 40, 500, 300, 1),  # past them, too few channels
    ("iqdas", 11, 105, 42, 768, 1),  # the wavefronts past the grid's edge count: lane groups
])
def test_sharing(mode, n, channels, nx, nz, share):
    p, got = _plan(mode, n, channels, nx, nz)
    assert got == share, p
    assert got * p["wz"] * p["wx"] > 1, p


@pytest.mark.parametrize("mode, n, channels, nx, nz, pixels", [
    ("dmas", 5, 128, 128, 128, 32),   # halves of these stage the same windows twice as often
    ("pdas", 3, 128, 200, 150, 64),
    ("dmas", 11, 32, 128, 256, 128),
    ("dmas", 3, 32, 512, 400, 256),
])
def test_root_tiles(mode, n, channels, nx, nz, pixels):
    p, share = _plan(mode, n, channels, nx, nz)
    assert share == 1
    assert 64 // p["cpw"] * p["wz"] * p["wx"] == pixels, p


def _long_windows(nx, nz):
    # windows that fill the LDS and leave the default tile no room
    return geom(angles_deg=(2.0,), nx=nx, nz=nz, n_channels=121, n_samples=2400, x_min=-18e-3,
                x_max=18e-3, z_min=8e-3, z_max=8e-3 + nz * 90e-6, f_number=1.0)


def test_no_block_of_two_wavefronts():
    from paper_2311_00482_amd import describe_plan
    p = describe_plan(_long_windows(190, 900), "das", -1)
    assert p["lds_bytes"] > 40 * 1024 and p["wz"] * p["wx"] == 2, p
    assert p["threads_per_block"] == 4 * 64, p


@pytest.mark.gpu
def test_parity_long_windows():
    import torch
    from paper_2311_00482_amd import beamform
    g = _long_windows(190, 900)
    rf = rand_rf(g, 91)
    out = beamform(g, torch.from_numpy(rf).cuda(), "das", -1, want=("rf",))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    pix = np.random.default_rng(9).integers(0, g.nx * g.nz, 30000)
    pix[:4] = [0, g.nz - 1, (g.nx - 1) * g.nz, g.nx * g.nz - 1]
    ref = oracle.das(g, rf, -1, pix=pix, parallel=True)
    assert np.abs(got.reshape(-1)[pix] - ref).max() <= TOL32 * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("mode, n, nx, nz", [("iqdas", 5, 362, 181), ("bbdmas", 3, 402, 301)])
def test_parity_two_share_iq(mode, n, nx, nz):
    import torch
    from paper_2311_00482_amd import beamform, describe_plan, iq_demodulate
    g = geom(angles_deg=tuple(np.linspace(-8.0, 7.0, n)), nx=nx, nz=nz, n_channels=49,
             n_samples=1024, x_min=-7e-3, x_max=7e-3, z_min=4e-3, z_max=4e-3 + nz * 50e-6,
             f_number=1.5)
    p = describe_plan(g, mode, -1)
    assert p["threads_per_block"] == 2 * 64 * p["wz"] * p["wx"] and p["cpw"] == 1, p
    rf = rand_rf(g, 92 + n)
    iq = iq_demodulate(g, torch.from_numpy(rf).cuda())
    out = beamform(g, iq, mode, -1, want=("rf", "imag"))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64) + 1j * out["imag"].cpu().numpy()
    ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1,
                             parallel=True)
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [13, 14, 16])
def test_many_shared_tiles(n):
    import torch
    from paper_2311_00482_amd import beamform, describe_plan
    g = geom(angles_deg=tuple(np.linspace(-9.0, 8.0, n)), nx=702, nz=577, n_channels=33,
             n_samples=1200, x_min=-4.9e-3, x_max=4.9e-3, z_min=3e-3, z_max=26e-3)
    p = describe_plan(g, "das", -1)
    assert p["threads_per_block"] == 2 * 64 * p["wz"] * p["wx"], p
    assert p["tiles_z"] * p["tiles_x"] >= 1536, p
    rf = rand_rf(g, 70 + n)
    out = beamform(g, torch.from_numpy(rf).cuda(), "das", -1, want=("rf",))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    pix = np.random.default_rng(n).integers(0, g.nx * g.nz, 6000)
    pix[:4] = [0, g.nz - 1, (g.nx - 1) * g.nz, g.nx * g.nz - 1]
    ref = oracle.das(g, rf, -1, pix=pix, parallel=True)
    assert np.abs(got.reshape(-1)[pix] - ref).max() <= TOL32 * np.abs(ref).max()
