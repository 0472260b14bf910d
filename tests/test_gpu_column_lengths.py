"""GPU parity of the register FFTs at every length they take: the depth
post-processing of columns of 2..4096 samples (with and without the band-pass, a
column count that leaves the last block partly empty, and the same columns
through a batch) and the demodulation of records of 2..4096 samples at every
decimation. Against the FP64 oracle at the 1e-5 bar; the log image to 0.1 dB
where it is at least -40 dB."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def _rel(got, ref):
    m = np.abs(ref).max()
    return np.abs(got - ref).max() / m if m > 0 else np.abs(got).max()


@pytest.mark.parametrize("bandpass", [False, True], ids=["plain", "band"])
@pytest.mark.parametrize("log2nz", range(1, 13))
def test_columns(log2nz, bandpass):
    import torch
    from paper_2311_00482_amd import Batch, FrameSpec, alloc_outputs, beamform
    nz = 1 << log2nz
    z = nz * 25e-6 if bandpass else 20e-3
    g = geom(nx=19, nz=nz, n_channels=6, n_samples=3000, z_min=4e-3, z_max=4e-3 + z,
             x_min=-1e-3, x_max=1e-3)
    rf = rand_rf(g, 30 + log2nz)
    dev = torch.from_numpy(rf).cuda()
    want = ("rf", "env", "log") + (("filtered",) if bandpass else ())
    out = beamform(g, dev, "das", 0, want=want, bandpass=bandpass)
    batched = alloc_outputs(g, want, "cuda")
    batch = Batch([FrameSpec(g, dev, "das", 0, batched, bandpass)])
    batch.launch()
    torch.cuda.synchronize()
    ref = oracle.beamform(g, rf, "das", 0, bandpass=bandpass)
    for name in want:
        for planes in (out, batched):
            got = planes[name].cpu().numpy().astype(np.float64)
            if name != "log":
                assert _rel(got, ref[name]) <= TOL32, name
            else:
                m = ref["log"] >= -40.0
                assert not m.any() or np.abs(got[m] - ref["log"][m]).max() <= 0.1
    batch.close()


@pytest.mark.parametrize("D", [1, 2, 4, 8])
@pytest.mark.parametrize("log2ns", range(1, 13))
def test_records(log2ns, D):
    import torch
    from paper_2311_00482_amd import GeometryArg, iq_demodulate
    ns = 1 << log2ns
    if ns < 2 * D:
        pytest.skip("a decimated record holds at least two samples")
    g = geom(n_samples=ns, angles_deg=(-5.0, 1.0, 4.0), n_channels=7)
    rf = rand_rf(g, 60 + log2ns, white=ns < 32)
    iq = iq_demodulate(GeometryArg(g, iq_decimation=D), torch.from_numpy(rf).cuda())
    torch.cuda.synchronize()
    ref = oracle.iq_demodulate(g, rf.astype(np.float64), decimation=D)
    got = iq.cpu().numpy().astype(np.complex128)
    assert got.shape == ref.shape
    assert _rel(got, ref) <= TOL32
