"""Decimated demodulation where both edges of the kept band fall on DFT bins and
rounding keeps them both: n_samples / D + 1 bins, two of which are the same bin of
the decimated spectrum. White records (so that the edge bins carry as much as any
other) against the FP64 oracle at the 1e-5 bar, one row per wavefront, several, and
rows of several wavefronts."""

import numpy as np
import pytest

import oracle

from cases import geom, rand_rf

TOL32 = 1e-5

CASES = [  # fs, f0 / fs, D
    (62.5e6 / 3, 20 / 64, 4),
    (1e8 / 3, 20 / 64, 4),
    (62.5e6 / 3, 16 / 64, 8),
]


@pytest.mark.parametrize("fs, ratio, D", CASES)
@pytest.mark.parametrize("log2ns", [4, 6, 9, 10, 11, 12])
def test_the_rule_keeps_both_edges(fs, ratio, D, log2ns):
    ns = 1 << log2ns
    kept = np.flatnonzero(oracle.band_keep(ns, fs, fs * ratio, D))
    assert len(kept) == ns // D + 1 and kept[-1] - kept[0] == ns // D


@pytest.mark.gpu
@pytest.mark.parametrize("fs, ratio, D", CASES)
@pytest.mark.parametrize("log2ns", [4, 6, 9, 10, 11, 12])
def test_records_with_both_edges(fs, ratio, D, log2ns):
    import torch
    from paper_2311_00482_amd import GeometryArg, iq_demodulate
    g = geom(n_samples=1 << log2ns, n_channels=7, angles_deg=(-5.0, 4.0), fs=fs, f0=fs * ratio)
    rf = rand_rf(g, 90 + log2ns, white=True)
    iq = iq_demodulate(GeometryArg(g, iq_decimation=D), torch.from_numpy(rf).cuda())
    torch.cuda.synchronize()
    ref = oracle.iq_demodulate(g, rf.astype(np.float64), decimation=D)
    got = iq.cpu().numpy().astype(np.complex128)
    assert got.shape == ref.shape
    assert np.abs(got - ref).max() <= TOL32 * np.abs(ref).max()
