"""GPU parity of IQ frames of 17 to 32 angles (one predicated kernel for all of them):
whole images against the FP64 oracle at the 1e-5 bar, with one lane group per wavefront,
with several, and with the library's own shape, whose LDS stays within a block's 64 KB
also where wavefronts share a pixel and add 2 x 32 sums there."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.mark.parametrize("tile", [None, (1, 8, 1, 1, 0), (4, 4, 1, 2, 4)],
                         ids=["own", "cpw1", "cpw4"])
@pytest.mark.parametrize("mode", ["iqdas", "bbdmas"])
@pytest.mark.parametrize("n, channels", [(17, 70), (24, 38), (32, 9), (32, 70)])
def test_many_angles(n, channels, mode, tile):
    import torch
    from paper_2311_00482_amd import Tile, beamform, describe_plan, iq_demodulate
    g = geom(angles_deg=tuple(np.linspace(-12.0, 11.0, n)), nx=19, nz=37, n_channels=channels,
             n_samples=512, x_min=-0.9e-3, x_max=0.9e-3, z_max=6e-3)
    rf = rand_rf(g, 600 + n)
    t = Tile(*tile) if tile else None
    assert describe_plan(g, mode, -1, t)["lds_bytes"] <= 64 * 1024
    iq = iq_demodulate(g, torch.from_numpy(rf).cuda())
    out = beamform(g, iq, mode, -1, want=("rf", "imag"), tile=t)
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64) + 1j * out["imag"].cpu().numpy()
    ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1,
                             parallel=True)
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()
