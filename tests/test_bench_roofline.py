"""The unit that bench.py prices each Legendre kernel at."""
import pytest

import bench

T = 3_000_000_000  # executed triples


@pytest.mark.parametrize("stage", ["legendre_fwd", "legendre_inv"])
@pytest.mark.parametrize("dtype,batch,nside,bound,peak", [
    ("f32", 16, 1024, "mfma", 2500.0 / 6),  # six BF16 partial products each
    ("f32", 1, 1024, "alu", 157.3), ("f64", 16, 1024, "mfma", 78.6), ("f64", 1, 2048, "alu", 78.6),
    ("bf16", 3, 128, "alu", 78.6),  # FP32 contraction; the FP64 recurrence takes longer
    ("f32", 3, 128, "alu", 78.6)])
def test_unit(stage, dtype, batch, nside, bound, peak):
    got, amount, unit, at = bench.legendre_work(stage, dtype, batch, nside, T)
    assert (got, unit) == (bound, "TFLOP/s") and at == pytest.approx(peak)
    recurrence = bench.on_mfma(stage, dtype, batch, nside) and bound == "alu"
    assert amount == (3.0 * T if recurrence else 4.0 * T * batch)


@pytest.mark.parametrize("batch,bound,peak", [(16, "alu", 78.6), (64, "mfma", 2500.0)])
def test_bf16_analysis(batch, bound, peak):
    got, _, _, at = bench.legendre_work("legendre_fwd", "bf16", batch, 1024, T)
    assert got == bound and at == peak
