"""Orders past every seed of a chunk of ring pairs are not stored: the entry points that
read those spectra from elsewhere (NESTED maps, stored lambda, the fixed scratch), with
NaN where the spectra go, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import nested, sht

pytestmark = pytest.mark.gpu
# FP32 transforms; BF16 spectra and Legendre values: both factors rounded (2^-9 each),
# with the cancellation allowance of the BF16 contraction's tests
TOL = {torch.float64: 1e-12, torch.float32: 1e-5, torch.bfloat16: 2.5 * 2.0 ** -8}


@pytest.fixture(scope="module")
def shtx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as m
    return m


def maps(nside, batch, dtype):
    return torch.randn(batch, 12 * nside * nside, generator=torch.Generator().manual_seed(nside + batch)).to(dtype)


def check(got, x, lmax, nside):
    ref = sht.map2alm(x.double().numpy(), lmax, nside)
    got = got.cpu().numpy()
    assert np.linalg.norm(got - ref) <= TOL[x.dtype] * np.linalg.norm(ref)


@pytest.mark.parametrize("entry,nside,lmax,batch,dtype", [
    ("map2alm", 512, 700, 5, torch.bfloat16), ("map2alm", 256, 767, 18, torch.bfloat16),
    ("nested", 256, 767, 18, torch.bfloat16), ("nested", 256, 600, 3, torch.float32),
    ("nested", 512, 600, 2, torch.float64), ("stored", 256, 300, 5, torch.bfloat16),
    ("stored", 256, 767, 2, torch.bfloat16)])
def test_workspace(shtx, entry, nside, lmax, batch, dtype):
    from paper_2510_01785_amd import _lib
    print("\n[case] %s nside=%d lmax=%d B=%d %s" % (entry, nside, lmax, batch, dtype), flush=True)
    L = _lib.lib()
    dev = torch.device("cuda", 0)
    code = {torch.float64: _lib.F64, torch.float32: _lib.F32, torch.bfloat16: _lib.BF16}[dtype]
    x = maps(nside, batch, dtype)
    xd = x.to(dev)
    if entry == "nested":  # the RING maps in NESTED order
        x = torch.tensor(nested.nest_to_ring(x.double().numpy(), nside)).to(dtype)
    tables = shtx.get_tables(nside, lmax, dev)
    nb = L.shtx_workspace_bytes(nside, lmax, batch, code)
    work = torch.full((nb // 4,), float("nan"), device=dev)
    a = torch.empty(batch, (lmax + 1) * (lmax + 2) // 2, device=dev,
                    dtype=torch.complex128 if dtype == torch.float64 else torch.complex64)
    lam = [shtx.get_lambda_table(nside, lmax, dev).data_ptr()] if entry == "stored" else []
    fn = {"map2alm": L.shtx_map2alm, "nested": L.shtx_map2alm_nested, "stored": L.shtx_map2alm_stored}[entry]
    _lib.check(entry, fn(nside, lmax, batch, code, xd.data_ptr(), a.data_ptr(), tables.data_ptr(), *lam,
                         work.data_ptr(), nb, torch.cuda.current_stream().cuda_stream))
    check(a, x, lmax, nside)
    shtx.release_lambda_tables()


# a call on NaN maps first leaves NaN spectra in the fixed scratch
@pytest.mark.parametrize("nside,lmax,batch,dtype", [(256, 511, 5, torch.bfloat16), (256, 300, 6, torch.float32),
                                                    (256, 400, 1, torch.float64)])
def test_fixed_scratch(shtx, nside, lmax, batch, dtype):
    from paper_2510_01785_amd import _lib
    print("\n[case] fixed scratch nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    L = _lib.lib()
    dev = torch.device("cuda", 0)

    def call(x, n, l, code, ct):
        xd = x.to(dev)
        a = torch.empty(x.shape[0], (l + 1) * (l + 2) // 2, dtype=ct, device=dev)
        _lib.check("shtx_map2alm_noalloc", L.shtx_map2alm_noalloc(
            n, l, x.shape[0], code, xd.data_ptr(), a.data_ptr(), shtx.get_tables(n, l, dev).data_ptr(),
            torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        return a

    x = maps(nside, batch, dtype)
    # every order of Nside 16 at lmax 15 counts, so all 64 MB (but the last channels') is written
    call(torch.full((8000, 12 * 16 * 16), float("nan")), 16, 15, _lib.F32, torch.complex64)
    check(call(x, nside, lmax, {torch.float64: _lib.F64, torch.float32: _lib.F32, torch.bfloat16: _lib.BF16}[dtype],
               torch.complex128 if dtype == torch.float64 else torch.complex64), x, lmax, nside)
