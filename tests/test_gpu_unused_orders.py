"""Orders past every seed of a ring: the synthesis neither writes nor reads their
spectra, whatever the workspace held; every Legendre kernel, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import sht

pytestmark = pytest.mark.gpu
TOL = {torch.float64: 1e-12, torch.float32: 1e-5}


# vector ALUs with 1, 2 and 4 ring pairs per lane, matrix cores with one group of
# channels and pairs of groups; band limits far above and below the polar rings' orders
@pytest.mark.parametrize("nside,lmax,batch,dtype", [
    (1, 40, 1, torch.float64), (32, 95, 1, torch.float64), (64, 191, 2, torch.float64), (128, 383, 3, torch.float64),
    (256, 300, 1, torch.float64), (128, 383, 8, torch.float64), (64, 70, 20, torch.float64), (32, 95, 1, torch.float32),
    (64, 191, 3, torch.float32), (256, 700, 2, torch.float32), (512, 600, 4, torch.float32),
    (256, 700, 16, torch.float32), (256, 300, 40, torch.float32)])
def test_nan_workspace(nside, lmax, batch, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    from paper_2510_01785_amd import _lib
    print("\n[case] unused orders nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    L = _lib.lib()
    dev = torch.device("cuda", 0)
    code, cdt = (_lib.F64, torch.complex128) if dtype == torch.float64 else (_lib.F32, torch.complex64)
    rng = np.random.default_rng(nside + batch)
    n = (lmax + 1) * (lmax + 2) // 2
    alm = torch.tensor(rng.standard_normal((batch, n)) + 1j * rng.standard_normal((batch, n))).to(cdt)
    x = alm.to(dev)
    tables = shtx.get_tables(nside, lmax, dev)
    nb = L.shtx_workspace_bytes(nside, lmax, batch, code)
    out = []
    for fill in (0.0, float("nan")):
        work = torch.full((nb // 4,), fill, device=dev)
        f = torch.empty(batch, 12 * nside * nside, dtype=dtype, device=dev)
        _lib.check("shtx_alm2map", L.shtx_alm2map(nside, lmax, batch, code, x.data_ptr(), f.data_ptr(),
                                                  tables.data_ptr(), work.data_ptr(), nb,
                                                  torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        out.append(f.cpu())
    assert torch.equal(out[0], out[1])
    ref = sht.alm2map(alm.numpy().astype(np.complex128), nside, lmax)
    assert np.linalg.norm(out[1].numpy() - ref) <= TOL[dtype] * np.linalg.norm(ref)
