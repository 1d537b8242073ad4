"""The coefficient layout pass of the synthesis (1 .. 4 channels by registers, more
through tiles of 16 channels): numbers of coefficients around its blocks and channel
counts around its slices, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import sht

pytestmark = pytest.mark.gpu
TOL = {torch.complex128: 1e-12, torch.complex64: 1e-5}


# coefficients: 1, 253 and 276 (blocks of 256), 1035 (of 4 x 256)
@pytest.mark.parametrize("lmax", [0, 21, 22, 44])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_coefficient_blocks(lmax, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    rng = np.random.default_rng(lmax)
    n = (lmax + 1) * (lmax + 2) // 2
    for batch in (1, 2, 3, 4, 5, 6, 15, 16, 17, 31, 33, 64):
        print("\n[case] layout lmax=%d B=%d %s" % (lmax, batch, dtype), flush=True)
        a = torch.tensor(rng.standard_normal((batch, n)) + 1j * rng.standard_normal((batch, n))).to(dtype)
        got = shtx.alm2map_raw(a.cuda(), 16, lmax).cpu().numpy()
        ref = sht.alm2map(a.numpy(), 16, lmax)
        assert np.linalg.norm(got - ref) <= TOL[dtype] * np.linalg.norm(ref), batch
