"""GPU parity of the root modes' kernels of several lane groups at 12 to 16 angles, which
differ between blocks of up to four wavefronts and of more: whole images against the FP64
oracle at the 1e-5 bar."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.mark.parametrize("tile", [(4, 4, 1, 2, 4), (2, 4, 2, 2, 2), (4, 4, 2, 4, 4)],
                         ids=["2waves", "4waves", "8waves"])
@pytest.mark.parametrize("mode", ["dmas", "pdas"])
@pytest.mark.parametrize("n", [11, 12, 14, 16, 17])
def test_blocks_of_few_and_of_many_wavefronts(n, mode, tile):
    import torch
    from paper_2311_00482_amd import Tile, beamform
    g = geom(angles_deg=tuple(np.linspace(-12.0, 11.0, n)), nx=21, nz=45, n_channels=11,
             x_min=-0.9e-3, x_max=0.9e-3, z_max=6e-3)
    rf = rand_rf(g, 800 + n)
    out = beamform(g, torch.from_numpy(rf).cuda(), mode, -1, tile=Tile(*tile), want=("rf",))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    ref = oracle.beamform(g, rf, mode, -1)["rf"]
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()
