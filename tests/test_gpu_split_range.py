"""Range of the FP32 Legendre products that run as three BF16 parts per factor: the
same accuracy at every magnitude that FP32 holds, against the FP64 oracle.

TOL: the kernels reach 2e-7 .. 7e-7 relative l2; leaving out any one of the six partial
products gives 2.5e-6 and more (random operands), and so does a lost low part."""
import numpy as np
import pytest
import torch

from oracle import sht
from paper_2510_01785_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1.5e-6


@pytest.fixture(scope="module")
def shtx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as m
    return m


def rel_l2(got, ref):
    """Per channel, the largest."""
    return max(float(np.linalg.norm(g - r) / np.linalg.norm(r)) for g, r in zip(got, ref))


def analysis(shtx, maps, lmax):
    """Unit-weight analysis (spectra of the maps' own magnitude), and the oracle's."""
    nside = shtx.nside_of(maps.shape[1])
    got = shtx.alm2map_backward_raw(torch.tensor(maps, device="cuda"), lmax, torch.complex64)
    return got.cpu().numpy().astype(np.complex128), sht.alm2map_backward(maps.astype(np.float64), lmax, nside)


def synthesis(shtx, alm, nside, lmax):
    got = shtx.alm2map_raw(torch.tensor(alm, device="cuda"), nside, lmax)
    return got.cpu().numpy().astype(np.float64), sht.alm2map(alm.astype(np.complex128), nside, lmax)


# one and two groups of 16 channels per wave (two from 257 ring pairs), one- and two-wave workgroups
@pytest.mark.parametrize("nside,lmax,batch", [(64, 127, 6), (64, 150, 20), (256, 300, 20), (1024, 140, 5)])
@pytest.mark.parametrize("exponent", [0, 90, -60, -116, -122])
def test_magnitudes(shtx, nside, lmax, batch, exponent):
    print("\n[case] 2^%d nside=%d lmax=%d B=%d" % (exponent, nside, lmax, batch), flush=True)
    s = np.float32(2.0 ** exponent)
    x = synth.white_map(nside + lmax, batch, 12 * nside * nside).astype(np.float32) * s
    a = synth.random_alm(nside + lmax, batch, lmax).astype(np.complex64) * s
    for got, ref in (analysis(shtx, x, lmax), synthesis(shtx, a, nside, lmax)):
        err = rel_l2(got * 2.0 ** -exponent, ref * 2.0 ** -exponent)
        print("rel l2 %.2e" % err, flush=True)
        assert err <= TOL


def test_magnitudes_by_channel(shtx):
    """Channels of one call, each of its own magnitude."""
    nside, lmax, batch = 64, 130, 21
    print("\n[case] a magnitude per channel", flush=True)
    s = np.array([2.0 ** e for e in (0, -122, -30, 90, -45)], dtype=np.float32)[np.arange(batch) % 5][:, None]
    x = synth.white_map(3, batch, 12 * nside * nside).astype(np.float32) * s
    a = synth.random_alm(4, batch, lmax).astype(np.complex64) * s
    for got, ref in (analysis(shtx, x, lmax), synthesis(shtx, a, nside, lmax)):
        assert rel_l2(got / s.astype(np.float64), ref / s.astype(np.float64)) <= TOL


# tiny values first, then ordinary ones, and the other way round: along the rings
# (north to equator) in the analysis, along l in the synthesis
@pytest.mark.parametrize("first,then", [(-116, 0), (0, -116), (-116, -45), (-45, 60)])
def test_magnitude_changes(shtx, first, then):
    nside, lmax, batch = 128, 200, 5
    print("\n[case] 2^%d, then 2^%d" % (first, then), flush=True)
    x = synth.white_map(5, batch, 12 * nside * nside).astype(np.float32)
    a = synth.random_alm(6, batch, lmax).astype(np.complex64)
    ls, _ = synth.lm_arrays(lmax)
    cap = 2 * nside * (nside - 1)
    x[:, :cap] *= np.float32(2.0 ** first)
    x[:, -cap:] *= np.float32(2.0 ** first)
    x[:, cap:-cap] *= np.float32(2.0 ** then)
    a *= np.where(ls < 60, np.float32(2.0 ** first), np.float32(2.0 ** then))
    for got, ref in (analysis(shtx, x, lmax), synthesis(shtx, a, nside, lmax)):
        big = 2.0 ** max(first, then)
        assert rel_l2(got / big, ref / big) <= TOL


def test_largest_spectra(shtx):
    """A ring spectrum just below the largest FP32 value (ring weight 2), whose BF16
    rounding is infinite, in the last channel."""
    nside, lmax, batch = 16, 20, 5
    print("\n[case] spectra below 2^128", flush=True)
    r = 10  # ring number, 4 r pixels from pixel 2 r (r - 1) on
    x = np.zeros((batch, 12 * nside * nside), dtype=np.float32)
    x[:, 2 * r * (r - 1):2 * r * (r + 1)] = 1.0
    x[-1] *= np.float32(2.0 ** 127 * (1 - 2.0 ** -11) / (4 * r))
    w = np.full(2 * nside, 2.0)
    got = shtx.map2alm_weighted_raw(torch.tensor(x, device="cuda"), lmax, torch.tensor(w)).cpu().numpy()
    # (the oracle's ring weights are one per ring, mirrored here)
    ref = sht.map2alm(x.astype(np.float64), lmax, nside, ring_weights=np.full(4 * nside - 1, 2.0))
    assert np.isfinite(got).all()
    big = np.abs(ref).max(axis=1, keepdims=True)
    assert rel_l2(got.astype(np.complex128) / big, ref / big) <= TOL
