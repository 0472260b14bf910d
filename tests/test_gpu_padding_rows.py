"""Lane groups whose channels do not divide a tile's aperture read the channels past it
and drop them: NaN there must not reach the image, which matches the FP64 oracle of the
records without them at the 1e-5 bar."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.mark.parametrize("tile", [(2, 8, 1, 2, 0), (4, 4, 2, 2, 8), (8, 4, 1, 2, 0), (16, 2, 1, 4, 16)])
@pytest.mark.parametrize("mode, n", [("das", 1), ("das", 3), ("dmas", 2), ("pdas", 5),
                                     ("iqdas", 3), ("bbdmas", 2)])
def test_channels_past_the_aperture(mode, n, tile):
    import torch
    from paper_2311_00482_amd import Tile, beamform, iq_demodulate
    g = geom(angles_deg=tuple(np.linspace(-6.0, 5.0, n)) if n > 1 else (1.0,), n_channels=41,
             nx=14, nz=45, x_min=-0.5e-3, x_max=0.5e-3, z_min=3e-3, z_max=5.5e-3, n_samples=512)
    rf = rand_rf(g, 40 + n)
    iq = mode in ("iqdas", "bbdmas")
    src = torch.from_numpy(rf).cuda()
    if iq:
        src = iq_demodulate(g, src)
    far = torch.from_numpy(np.abs(np.asarray(g.elem_x)) > 3.0e-3).cuda()
    assert 16 <= int(far.sum()) <= 24
    src[:, far] = float("nan")
    out = beamform(g, src, mode, -1, tile=Tile(*tile), want=("rf", "imag") if iq else ("rf",))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    if iq:
        got = got + 1j * out["imag"].cpu().numpy()
        ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1)
    else:
        ref = oracle.beamform(g, rf, mode, -1)["rf"]
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()
