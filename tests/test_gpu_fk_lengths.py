"""GPU parity of the f-k migrations at every record length (2 to 4096 samples: rows of
one thread up to 512, several rows to a block below 512) and every padded array length
(4 to 1024 for Lu's method, 4 to 512 for Stolt's), with odd channel counts (the last
row of two traces holds one) and two angles, against the FP64 oracle; the bar is the
other f-k tests': max |gpu - oracle| / max |oracle| <= 1e-5 of the complex image."""

import numpy as np
import pytest

from oracle import fk

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5
LENGTHS = [(2, 2), (4, 3), (8, 5), (16, 9), (32, 17), (64, 33), (128, 65), (256, 131), (512, 256),
           (1024, 7), (2048, 21), (4096, 37), (512, 2), (256, 4)]


@pytest.mark.parametrize("method", ["stolt", "lu"])
@pytest.mark.parametrize("samples, channels", LENGTHS)
def test_fk_lengths(samples, channels, method):
    import torch
    from paper_2311_00482_amd import fk_migrate
    depth = 0.7 * samples * 38.5e-6
    g = geom(n_channels=channels, n_samples=samples, angles_deg=(-4.0, 3.0), nx=21, nz=37,
             x_min=-channels * 0.1e-3, x_max=channels * 0.1e-3, z_min=0.05 * depth, z_max=depth)
    rf = rand_rf(g, samples + channels, "f32", white=samples < 64)
    out = fk_migrate(g, torch.from_numpy(rf).cuda(), -1, want=("rf", "imag"), method=method)
    got = out["rf"].cpu().numpy().astype(np.float64) + 1j * out["imag"].cpu().numpy()
    ref = fk.fk_migrate(g, rf.astype(np.float64), -1, method=method)
    peak = np.abs(ref).max()
    assert peak > 0
    assert np.abs(got - ref).max() <= TOL32 * peak
