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
