"""Legendre kernels whose FP32 products run as BF16 partial products on the
matrix cores, at the edges of their tiles: against the FP64 oracle at the FP32
tolerance of the transforms (1e-5 relative l2; the products carry 24 bits)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import sht
from paper_2510_01785_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def shtx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as m
    return m


def rel_l2(got, ref):
    return float(np.linalg.norm((got - ref).ravel()) / np.linalg.norm(ref.ravel()))


# one and two groups of 16 channels per wave, partial groups; columns of m that
# end inside, at and just past a group of 32 l (every m = 0..L is one); fewer,
# as many and more ring pairs than a chunk of 64; band limits below 8
@pytest.mark.parametrize("nside,lmax,batch", [(1, 0, 3), (2, 7, 5), (8, 31, 16), (8, 32, 17), (16, 47, 31),
                                              (32, 63, 32), (32, 64, 33), (64, 101, 48), (64, 191, 3), (128, 130, 7)])
def test_synthesis_edges(shtx, nside, lmax, batch):
    print("\n[case] synthesis nside=%d lmax=%d B=%d" % (nside, lmax, batch), flush=True)
    alm = synth.random_alm(nside + lmax + batch, batch, lmax).astype(np.complex64)
    got = shtx.alm2map_raw(torch.tensor(alm, device="cuda"), nside, lmax).cpu().numpy()
    assert rel_l2(got, sht.alm2map(alm.astype(np.complex128), nside, lmax)) <= TOL


def test_synthesis_reads_nothing_past_the_coefficients(shtx):
    """A workspace full of NaN changes nothing (rows past lmax and channels
    past the batch meet no product), and a NaN channel stays in its channel."""
    from paper_2510_01785_amd import _lib
    nside, lmax, B = 16, 42, 9
    print("\n[case] synthesis, NaN workspace", flush=True)
    alm = torch.tensor(synth.random_alm(5, B, lmax).astype(np.complex64), device="cuda")
    want = shtx.alm2map_raw(alm, nside, lmax)
    L = _lib.lib()
    nb = L.shtx_workspace_bytes(nside, lmax, B, _lib.F32)
    work = torch.full((nb // 4,), float("nan"), device="cuda")
    out = torch.empty_like(want)
    st = L.shtx_alm2map(nside, lmax, B, _lib.F32, alm.data_ptr(), out.data_ptr(),
                        shtx.get_tables(nside, lmax, alm.device).data_ptr(), work.data_ptr(), ctypes.c_size_t(nb),
                        torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert torch.equal(out, want)
    alm[4] = float("nan")
    got = shtx.alm2map_raw(alm, nside, lmax)
    keep = [b for b in range(B) if b != 4]
    assert torch.equal(got[keep], want[keep]) and torch.isnan(got[4]).all()


@pytest.mark.parametrize("scale", [1e-30, 1e30, float(np.finfo(np.float32).max)])
def test_synthesis_coefficient_range(shtx, scale):
    """Small and large coefficients, up to the largest finite one (a_00 alone:
    a constant map below the FP32 limit)."""
    print("\n[case] synthesis, coefficients of %g" % scale, flush=True)
    nside, lmax, B = 16, 40, 5
    alm = np.zeros((B, synth.nalm(lmax)), dtype=np.complex64)
    alm[:, 0] = scale
    if scale < 1e31:
        alm = (synth.random_alm(6, B, lmax) * scale).astype(np.complex64)
    got = shtx.alm2map_raw(torch.tensor(alm, device="cuda"), nside, lmax).cpu().numpy().astype(np.float64)
    ref = sht.alm2map(alm.astype(np.complex128), nside, lmax)
    assert np.isfinite(got).all() and rel_l2(got / scale, ref / scale) <= TOL


# item edges of the analysis: band limits that end inside the first and second
# half of a block of 128 l, a block exactly full and one past it; fewer, as many
# and more ring pairs than a slice of 64, with partial slices per wave; partial
# channel groups
@pytest.mark.parametrize("nside,lmax,batch", [(1, 2, 5), (8, 31, 17), (16, 47, 16), (32, 63, 5), (32, 64, 33),
                                              (64, 127, 6), (64, 128, 16), (128, 301, 5)])
def test_analysis_edges(shtx, nside, lmax, batch):
    print("\n[case] analysis nside=%d lmax=%d B=%d" % (nside, lmax, batch), flush=True)
    maps = synth.white_map(nside + lmax + batch, batch, 12 * nside * nside).astype(np.float32)
    got = shtx.map2alm_raw(torch.tensor(maps, device="cuda"), lmax).cpu().numpy()
    assert rel_l2(got, sht.map2alm(maps.astype(np.float64), lmax, nside)) <= TOL


@pytest.mark.parametrize("nside,lmax,batch", [(64, 150, 5), (256, 300, 16)])
def test_analysis_of_constant_maps(shtx, nside, lmax, batch):
    """A constant map's products repeat from ring to ring and so do their
    roundings: 24 of them (at most 2^-24 each) in the sum over a slice of 64
    rings, then one per slice (8 at Nside 256), 32 x 2^-24 = 1.9e-6 at most."""
    print("\n[case] analysis of constants nside=%d lmax=%d B=%d" % (nside, lmax, batch), flush=True)
    c = (1.2345678 + 0.37 * np.arange(batch)).astype(np.float32)
    maps = np.repeat(c[:, None], 12 * nside * nside, axis=1)
    got = shtx.map2alm_raw(torch.tensor(maps, device="cuda"), lmax).cpu().numpy()
    assert rel_l2(got, sht.map2alm(maps.astype(np.float64), lmax, nside)) <= 2e-6


def test_analysis_keeps_channels_apart(shtx):
    """An infinite and a NaN pixel stay in their channels."""
    print("\n[case] analysis, inf and NaN channels", flush=True)
    nside, lmax, B = 16, 40, 18
    x = torch.tensor(synth.white_map(7, B, 12 * nside * nside).astype(np.float32), device="cuda")
    want = shtx.map2alm_raw(x, lmax)
    x[3, 100] = float("inf")
    x[16, 5] = float("nan")
    got = shtx.map2alm_raw(x, lmax)
    keep = [b for b in range(B) if b not in (3, 16)]
    assert torch.equal(got[keep], want[keep])
    for b in (3, 16):  # (the imaginary parts of m = 0 are written as zero)
        assert (~torch.isfinite(torch.view_as_real(got[b]))).any(dim=1).all()


# the vector-ALU analysis at the edges of its rings per lane and workgroup
# shapes (up to 128, 256, 1024 ring pairs and more), one and two channels,
# against the oracle at the transforms' tolerances
@pytest.mark.parametrize("nside,lmax,batch", [(1, 1, 1), (16, 20, 2), (64, 127, 1), (64, 129, 2), (128, 150, 1),
                                              (128, 260, 2), (256, 300, 1), (512, 513, 3), (1024, 260, 1),
                                              (1024, 140, 2)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_vector_alu_analysis(shtx, monkeypatch, nside, lmax, batch, dtype):
    print("\n[case] vector-ALU analysis nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    monkeypatch.setenv("SHTX_FORCE_VALU", "1")
    x = torch.tensor(synth.white_map(nside + lmax, batch, 12 * nside * nside), dtype=dtype)
    got = shtx.map2alm_raw(x.cuda(), lmax).cpu().numpy()
    ref = sht.map2alm(x.double().numpy(), lmax, nside)
    assert rel_l2(got, ref) <= (1e-12 if dtype == torch.float64 else TOL)


# the vector-ALU synthesis with one, two and four ring pairs per lane (the
# number of waves decides), partial lanes, every channel-group width
@pytest.mark.parametrize("nside,lmax,batch", [(1, 1, 1), (16, 33, 2), (64, 65, 4), (128, 130, 7), (512, 900, 1),
                                              (512, 600, 2), (1024, 520, 4), (1024, 2100, 1)])
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
def test_vector_alu_synthesis(shtx, monkeypatch, nside, lmax, batch, dtype):
    print("\n[case] vector-ALU synthesis nside=%d lmax=%d B=%d %s" % (nside, lmax, batch, dtype), flush=True)
    monkeypatch.setenv("SHTX_FORCE_VALU", "1")
    alm = torch.tensor(synth.gaussian_alm(nside + lmax, batch, lmax, "lp10")).to(dtype)
    got = shtx.alm2map_raw(alm.cuda(), nside, lmax).cpu().numpy()
    ref = sht.alm2map(alm.numpy().astype(np.complex128), nside, lmax)
    assert rel_l2(got, ref) <= (1e-12 if dtype == torch.complex128 else TOL)
