"""The vector-ALU Legendre kernels with more channel groups than a launch has grid
rows (65535), at the smallest transform."""
import numpy as np
import pytest
import torch

from oracle import sht
from paper_2510_01785_amd import synth

pytestmark = pytest.mark.gpu


def test_channel_groups_past_one_grid(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_01785_amd as shtx
    monkeypatch.setenv("SHTX_FORCE_VALU", "1")
    nside, lmax, groups = 1, 1, 65537  # of 2 channels (FP64 both ways, FP32 analysis)
    print("\n[case] %d channels" % (2 * groups), flush=True)
    x = synth.white_map(9, 2, 12).astype(np.float32)
    ref = sht.map2alm(x.astype(np.float64), lmax, nside)
    back = sht.alm2map(ref, nside, lmax)
    for dtype, tol in ((torch.float32, 1e-5), (torch.float64, 1e-12)):
        a = shtx.map2alm_raw(torch.tensor(x).to(dtype).cuda().repeat(groups, 1), lmax)
        f = shtx.alm2map_raw(a, nside, lmax)
        for got, want in ((a, ref), (f, back)):
            d = got.cpu().numpy().reshape((groups,) + want.shape) - want
            assert np.abs(d).max() <= tol * np.abs(want).max()
