"""The long-tap FIR at the edges of its 16-row tiles and 16-tap segments:
element by element against the FP64 oracle, and up to 64 taps bit for bit
against the register window."""
import numpy as np
import pytest

import oracle
from paper_1511_03599_amd import synth
from helpers import c128, say, taps_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T,S,B,dtype", [
    (64, 65, 1, 1, "c64"), (65, 80, 15, 2, "ci16"), (63, 81, 16, 1, "ci8"), (128, 96, 17, 3, "cf16"),
    (1, 79, 33, 1, "c64"), (130, 1024, 5, 1, "ci8"), (96, 112, 1000, 2, "c64"), (77, 95, 31, 1, "cf16")])
def test_long_taps_tile_and_segment_edges(dev, C, T, S, B, dtype):
    """Each component is one float32 accumulator over T products, so its error
    is at most (T + 1) 2^-24 of the sum of the products' magnitudes."""
    from paper_1511_03599_amd import pfb
    say(f"long-tap FIR edges C={C} T={T} S={S} B={B} {dtype}")
    x = synth.noise_stream(B, C, T, S, 2100 + C + T, dtype=dtype).x
    h = synth.random_taps(C, T, 2101)
    y = c128(pfb.Plan(C, T, S, B, dtype, pfb.FIR_ONLY).execute(to_device(x, dev), taps_to_device(h, dev)))
    ref, size = oracle.fir(x, h), oracle.fir(np.abs(x), np.abs(h))
    bound = (T + 1) * 2.0 ** -24
    assert np.all(np.abs(y.real - ref.real) <= bound * size.real)
    assert np.all(np.abs(y.imag - ref.imag) <= bound * size.imag)


@pytest.mark.parametrize("C,T,S,B", [(64, 33, 1, 1), (63, 48, 16, 2), (65, 49, 17, 1), (256, 64, 3000, 1),
                                     (1000, 40, 700, 3), (1, 63, 100, 1)])
@pytest.mark.parametrize("dtype", ["c64", "ci16", "ci8", "cf16"])
def test_33_to_64_taps_equal_the_register_window(dev, C, T, S, B, dtype):
    """Small launches of 33 to 64 taps go through the long-tap FIR; a plain
    plan keeps the register window. Same sums in the same order: same bits."""
    import torch
    from paper_1511_03599_amd import pfb
    say(f"33 to 64 taps C={C} T={T} S={S} B={B} {dtype}")
    x = synth.device_quantised_noise((B, S + T - 1, C), dtype, 2200 + C + T, dev)
    h = taps_to_device(synth.random_taps(C, T, 2201), dev)
    y = pfb.Plan(C, T, S, B, dtype, pfb.FIR_ONLY).execute(x, h)
    assert torch.equal(y, pfb.Plan(C, T, S, B, dtype, pfb.FIR_ONLY | pfb.PLAIN).execute(x, h))


@pytest.mark.parametrize("C,T,before,after", [
    (256, 40, 0, 24),    # register window and blocked kernel: 24 zero taps lead; long-tap FIR: 8
    (256, 64, 0, 0),
    (256, 65, 15, 0),    # long-tap FIR: 15 zero taps follow
    (1000, 90, 6, 0),
])
def test_non_finite_samples_stay_within_the_padded_window(dev, C, T, before, after, tmp_path, monkeypatch):
    """An infinity reaches the spectra whose T rows hold it, and at most those
    whose window holds it under zero taps; the others have the same bits as
    without it, on every path."""
    import torch
    from paper_1511_03599_amd import pfb
    S, r = 400, 200
    say(f"non-finite long taps C={C} T={T}")
    x = synth.device_noise((1, S + T - 1, C), 2300 + C + T, dev)
    h = taps_to_device(synth.random_taps(C, T, 2301), dev)
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    plans = [pfb.Plan(C, T, S, 1, "c64", flags) for flags in (0, pfb.NO_FUSE, pfb.PLAIN)]
    if T <= 64:
        for choice in ("block=1", "block=0 segments=0 fir_sb=64", "block=0 segments=1"):
            cache = tmp_path / "tune.txt"
            cache.write_text(f"{arch} 0 {C} {T} 1 {S} path=1 {choice}\n")
            monkeypatch.setenv("PFB_TUNE_CACHE", str(cache))
            plans.append(pfb.Plan(C, T, S, 1, "c64"))
            monkeypatch.delenv("PFB_TUNE_CACHE")
    bad = x.clone()
    bad[0, r, 7] = float("inf")
    finite = plans[0].execute(x, h)
    for i, plan in enumerate(plans):
        Y = plan.execute(bad, h)[0]
        ok = torch.isfinite(Y.real).all(1) & torch.isfinite(Y.imag).all(1)
        assert not ok[r - T + 1:r + 1].any(), i
        lo, hi = r - T + 1 - before, r + 1 + after
        assert ok[:lo].all() and ok[hi:].all(), i
        assert torch.equal(Y[:lo], finite[0, :lo]) and torch.equal(Y[hi:], finite[0, hi:]), i
