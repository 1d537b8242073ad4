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


# chunks of 256 ring pairs whose orders end early (from Nside 256), each analysis
# kernel: vector ALUs, FP32, FP64 and BF16 matrix cores
@pytest.mark.parametrize("nside,lmax,batch,dtype,nested", [
    (256, 767, 1, torch.float64, 0), (512, 300, 2, torch.float64, 0), (256, 500, 3, torch.float64, 0),
    (512, 700, 8, torch.float64, 0), (64, 150, 4, torch.float64, 0), (256, 767, 1, torch.float32, 0),
    (512, 700, 4, torch.float32, 0), (256, 600, 3, torch.float32, 1), (512, 700, 5, torch.float32, 0),
    (256, 767, 20, torch.float32, 0), (1, 30, 6, torch.float32, 0), (512, 700, 5, torch.bfloat16, 0),
    (256, 767, 18, torch.bfloat16, 1), (512, 600, 2, torch.bfloat16, 0)])
def test_nan_workspace_analysis(nside, lmax, batch, dtype, nested):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    from paper_2510_01785_amd import _lib
    print("\n[case] unused orders, analysis nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    L = _lib.lib()
    dev = torch.device("cuda", 0)
    code = {torch.float64: _lib.F64, torch.float32: _lib.F32, torch.bfloat16: _lib.BF16}[dtype]
    gen = torch.Generator().manual_seed(nside + batch)
    x = torch.randn(batch, 12 * nside * nside, generator=gen).to(dtype)
    xd = x.to(dev)
    tables = shtx.get_tables(nside, lmax, dev)
    nb = L.shtx_workspace_bytes(nside, lmax, batch, code)
    fn = L.shtx_map2alm_nested if nested else L.shtx_map2alm
    out = []
    for fill in (0.0, float("nan")):
        work = torch.full((nb // 4,), fill, device=dev)
        a = torch.empty(batch, (lmax + 1) * (lmax + 2) // 2, device=dev,
                        dtype=torch.complex128 if dtype == torch.float64 else torch.complex64)
        _lib.check("analysis", fn(nside, lmax, batch, code, xd.data_ptr(), a.data_ptr(), tables.data_ptr(),
                                  work.data_ptr(), nb, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        out.append(a.cpu())
    assert torch.equal(out[0], out[1])
    if not nested and dtype != torch.bfloat16:
        ref = sht.map2alm(x.double().numpy(), lmax, nside)
        assert np.linalg.norm(out[1].numpy() - ref) <= TOL[dtype] * np.linalg.norm(ref)
