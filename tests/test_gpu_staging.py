"""GPU parity of the window staging where its wide loads and its channel table
change path: odd record lengths and start addresses of 16-bit storage, records
that begin or end inside a window, and launch shapes whose LDS holds the
channel table only in parts. Whole images against the FP64 oracle at 1e-5; the
storage's own values are the oracle's input, so no storage error enters."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def _rel(got, ref):
    return np.abs(got - ref).max() / np.abs(ref).max()


def _store(g, seed, dtype, offset):
    """Seeded records of dtype, `offset` elements into their allocation."""
    import torch
    host = torch.from_numpy(rand_rf(g, seed, "i16" if dtype == "int16" else "f32"))
    host = host.to(getattr(torch, dtype))
    buf = torch.zeros(host.numel() + offset + 8, dtype=host.dtype, device="cuda")
    rf = buf[offset:offset + host.numel()].view(host.shape)
    rf.copy_(host)
    return rf, host.to(torch.float64).numpy()


@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("dtype", ["int16", "float16", "float32"])
@pytest.mark.parametrize("samples", [151, 152, 27])
def test_record_lengths_and_addresses(dtype, samples, offset):
    import torch
    from paper_2311_00482_amd import beamform
    # delays of 10 to 330 samples: records of 151 end inside the windows, records
    # of 27 start and end inside one (the first pixel rows reach delay 0)
    g = geom(n_samples=samples, angles_deg=(-4.0, 0.0, 5.0), nx=19, nz=70,
             z_min=0.0 if samples == 27 else 1e-3, z_max=1e-3 if samples == 27 else 8e-3,
             x_min=-1e-3, x_max=1e-3, n_channels=11)
    rf, host = _store(g, samples, dtype, offset)
    for mode in ("das", "pdas"):
        out = beamform(g, rf, mode, -1, want=("rf",))["rf"]
        torch.cuda.synchronize()
        ref = oracle.beamform(g, host, mode, -1)["rf"]
        assert _rel(out.cpu().numpy(), ref) <= TOL32, mode


TABLE = [
    # mode, angles, tile: windows that leave no room for a 256-channel table
    ("das", 32, (4, 8, 1, 1, 4)),
    ("das", 32, (1, 8, 1, 1, 4)),
    ("iqdas", 16, (4, 8, 1, 1, 4)),
    ("bbdmas", 15, (1, 8, 1, 1, 4)),
]


@pytest.mark.parametrize("mode,n,tile", TABLE, ids=[f"{m}{n}_cpw{t[0]}" for m, n, t in TABLE])
def test_channel_table_in_parts(mode, n, tile):
    import torch
    from paper_2311_00482_amd import Tile, beamform, describe_plan, iq_demodulate
    g = geom(n_channels=255, n_samples=1024, angles_deg=tuple(np.linspace(-9.0, 8.0, n)), nx=9,
             nz=21, x_min=-0.4e-3, x_max=0.4e-3, z_min=20e-3, z_max=25.4e-3, f_number=0.4)
    lds = describe_plan(g, mode, -1, Tile(*tile))["lds_bytes"]
    assert 64 * 1024 - 255 * 20 < lds <= 64 * 1024  # no room left for 255 channels' entries
    rf = rand_rf(g, 600 + n)
    dev = torch.from_numpy(rf).cuda()
    iq = mode in ("iqdas", "bbdmas")
    out = beamform(g, iq_demodulate(g, dev) if iq else dev, mode, -1, tile=Tile(*tile),
                   want=("rf", "imag") if iq else ("rf",))
    torch.cuda.synchronize()
    got = out["rf"].cpu().numpy().astype(np.float64)
    if iq:
        got = got + 1j * out["imag"].cpu().numpy()
        ref = oracle.iq_beamform(g, oracle.iq_demodulate(g, rf.astype(np.float64)), mode, -1,
                                 parallel=True)
    else:
        ref = oracle.beamform(g, rf, mode, -1)["rf"]
    assert _rel(got, ref) <= TOL32
