"""GPU parity of the exactly unrolled kernels over the angle counts: 17..32 angles
of the RF modes and 2..16 of the IQ modes (with 17, the first count of their
predicated kernel), whole images against the FP64 oracle at the 1e-5 bar, with
one lane group per wavefront and with several."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def _geometry(n, **kw):
    return geom(angles_deg=tuple(np.linspace(-12.0, 11.0, n)), nx=9, nz=37, n_channels=9,
                x_min=-0.6e-3, x_max=0.6e-3, z_max=6e-3, **kw)


def _image(g, rf, mode, tile):
    import torch
    from paper_2311_00482_amd import Tile, beamform
    want = ("rf", "imag") if mode in ("iqdas", "bbdmas") else ("rf",)
    out = beamform(g, rf, mode, -1, tile=Tile(*tile), want=want)
    torch.cuda.synchronize()
    img = out["rf"].cpu().numpy().astype(np.float64)
    return img + 1j * out["imag"].cpu().numpy() if len(want) > 1 else img


@pytest.mark.parametrize("tile", [(1, 8, 1, 1, 0), (4, 4, 1, 2, 4)], ids=["cpw1", "cpw4"])
@pytest.mark.parametrize("mode", ["das", "dmas", "pdas"])
@pytest.mark.parametrize("n", [17, 18, 21, 25, 28, 31, 32])
def test_rf_modes(mode, n, tile):
    import torch
    g = _geometry(n)
    rf = rand_rf(g, 400 + n)
    got = _image(g, torch.from_numpy(rf).cuda(), mode, tile)
    ref = oracle.beamform(g, rf, mode, -1)["rf"]
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()


@pytest.mark.parametrize("tile", [(1, 8, 1, 1, 0), (4, 4, 1, 2, 4)], ids=["cpw1", "cpw4"])
@pytest.mark.parametrize("mode", ["iqdas", "bbdmas"])
@pytest.mark.parametrize("n", [2, 3, 4, 6, 7, 8, 9, 10, 12, 13, 14, 15, 16, 17])
def test_iq_modes(mode, n, tile):
    import torch
    from paper_2311_00482_amd import iq_demodulate
    g = _geometry(n, n_samples=512)
    rf = rand_rf(g, 500 + n)
    iq = iq_demodulate(g, torch.from_numpy(rf).cuda())
    got = _image(g, iq, mode, tile)
    ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1)
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()
