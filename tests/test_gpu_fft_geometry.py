"""Workgroup shapes of the ring FFT (threads, channels per workgroup, slices of
unequal width) at sizes on both sides of their rules: both directions against
the FP64 oracle at the transforms' tolerances."""
import numpy as np
import pytest
import torch

from oracle import sht
from paper_2510_01785_amd import synth

pytestmark = pytest.mark.gpu
TOL = {torch.float64: 1e-12, torch.float32: 1e-5}


# one channel per workgroup (few channels), two and four (many), slices of unequal
# width (3 + 2); 128, 256 and 512 threads; Nside 256 at 8 and 9 channels, FP64
# Nside 512 at 1 and 4
@pytest.mark.parametrize("nside,lmax,batch,dtype", [
    (1, 2, 3, torch.float32), (2, 5, 40, torch.float64), (16, 40, 64, torch.float32), (32, 65, 70, torch.float32),
    (32, 40, 33, torch.float64), (64, 70, 2, torch.float32), (64, 90, 33, torch.float32), (64, 70, 9, torch.float64),
    (128, 129, 1, torch.float32), (128, 140, 5, torch.float32), (128, 130, 17, torch.float64),
    (256, 260, 1, torch.float32), (256, 257, 8, torch.float32), (256, 257, 9, torch.float32),
    (256, 258, 5, torch.float64), (512, 80, 5, torch.float32), (512, 90, 1, torch.float64),
    (512, 60, 4, torch.float64)])
def test_ring_fft_shapes(nside, lmax, batch, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    print("\n[case] ring FFT nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    x = torch.tensor(synth.white_map(nside + batch, batch, 12 * nside * nside), dtype=dtype)
    a = shtx.map2alm_raw(x.cuda(), lmax)
    ref = sht.map2alm(x.double().numpy(), lmax, nside)
    got = a.cpu().numpy()
    assert np.linalg.norm(got - ref) <= TOL[dtype] * np.linalg.norm(ref)
    f = shtx.alm2map_raw(a, nside, lmax).cpu().numpy()
    ref = sht.alm2map(got.astype(np.complex128), nside, lmax)
    assert np.linalg.norm(f - ref) <= TOL[dtype] * np.linalg.norm(ref)


# ring lengths 4 i of every odd radix, alone, squared and mixed, with odd and even
# power-of-two parts; the first lengths past the direct radices
_RINGS = [1, 3, 5, 7, 9, 11, 13, 17, 19, 23, 27, 29, 31, 46, 121, 125, 169, 242, 289, 343, 361, 368, 391, 437, 529, 676,
          729, 768, 874, 899, 945, 969, 1000, 1001, 1008, 1012, 1021, 1024]


# A map that is zero off one ring: alm[l, m] is the ring's Fourier sum at m times a
# factor (weight, phase, Legendre value) that does not depend on the ring's pixels, so
# against a unit pixel's alm the ratio is the DFT.
@pytest.mark.parametrize("batch,dtype", [(2, torch.float64), (5, torch.float64), (2, torch.float32), (7, torch.float32)])
def test_ring_lengths_by_radix(batch, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    nside, lmax = 1024, 2100  # |m| past every frequency of every cap ring
    m = torch.tensor(np.repeat(np.arange(lmax + 1), lmax + 1 - np.arange(lmax + 1)), device="cuda")
    gen = torch.Generator().manual_seed(batch)
    for r in _RINGS:
        n = 4 * r
        print("\n[case] ring length %d B=%d %s" % (n, batch, dtype), flush=True)
        x = torch.zeros(batch, 12 * nside * nside, dtype=dtype, device="cuda")
        ring = torch.randn(batch, n, generator=gen).to(dtype)
        ring[0] = 0
        ring[0, 0] = 1
        x[:, 2 * r * (r - 1):2 * r * (r + 1)] = ring.cuda()
        a = shtx.map2alm_raw(x, lmax).to(torch.complex128)
        dft = torch.tensor(np.fft.fft(ring.double().numpy(), axis=1)).cuda()[:, m % n]
        err = torch.linalg.norm(a - a[:1] * dft, dim=1)
        assert (err <= TOL[dtype] * n ** 0.5 * torch.linalg.norm(a[0])).all(), r
        del x, a, dft, err
