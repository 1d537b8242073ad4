"""Which pixels a NaN coefficient reaches: all of every ring where its lambda counts,
none of a ring that has no lambda of its order, no other channel.  Every synthesis kernel."""
import numpy as np
import pytest
import torch

from oracle import geometry, sht
from oracle.legendre import lambda_table
from paper_2510_01785_amd import synth

pytestmark = pytest.mark.gpu


# vector ALUs and matrix cores; orders that most, some and few rings have
@pytest.mark.parametrize("dtype,batch", [(torch.complex64, 2), (torch.complex64, 5), (torch.complex128, 1),
                                         (torch.complex128, 6)])
@pytest.mark.parametrize("l,m", [(150, 140), (380, 200), (383, 383)])
def test_nan_coefficient(dtype, batch, l, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    nside, lmax = 128, 383
    print("\n[case] NaN a_%d,%d, B=%d %s" % (l, m, batch, dtype), flush=True)
    alm = torch.tensor(synth.random_alm(l + m, batch, lmax)).to(dtype)
    alm[-1, geometry.alm_index(l, m, lmax)] = complex("nan+nanj")
    f = shtx.alm2map_raw(alm.cuda(), nside, lmax).cpu().numpy()
    g = geometry.ring_geometry(nside)
    lam = np.abs(lambda_table(lmax, m, g["z"], g["sth"]))
    # (the kernels' threshold applies to lambda over a factor in 0.1 .. 1)
    ring = np.repeat(np.arange(4 * nside - 1), g["n"])
    reached = (lam[l - m] > 2.0 ** -60)[ring]
    past = (lam.max(axis=0) < 2.0 ** -68)[ring]
    assert reached.any() and past.any()
    assert np.isnan(f[-1][reached]).all() and np.isfinite(f[-1][past]).all()
    tol = 1e-5 if dtype == torch.complex64 else 1e-12
    if batch > 1:
        ref = sht.alm2map(alm[:-1].numpy().astype(np.complex128), nside, lmax)
        assert np.linalg.norm(f[:-1] - ref) <= tol * np.linalg.norm(ref)
    # where the order has no lambda, the pixels are those without the coefficient
    alm[-1, geometry.alm_index(l, m, lmax)] = 0
    ref = sht.alm2map(alm[-1:].numpy().astype(np.complex128), nside, lmax)[0]
    assert np.abs(f[-1] - ref)[past].max() <= 10 * tol * np.abs(ref).max()
