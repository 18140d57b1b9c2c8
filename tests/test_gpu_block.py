"""The blocked forward (FIR and FFT in one launch) against the two-launch
split path, whose oracle parity the other tests pin: sums, radices, twiddles
and order of operations are the same, so the spectra must be the same bits."""
import numpy as np
import pytest

from paper_1511_03599_amd import synth
from helpers import say, taps_to_device, to_device

pytestmark = pytest.mark.gpu


def blocked_plan(pfb, C, T, S, B, dtype, tmp_path, monkeypatch):
    """A plan that runs blocked whatever its size."""
    import torch
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{arch} {pfb.DTYPE_CODES[dtype]} {C} {T} {B} {S} path=1 block=1\n")
    monkeypatch.setenv("PFB_TUNE_CACHE", str(cache))
    plan = pfb.Plan(C, T, S, B, dtype)
    monkeypatch.delenv("PFB_TUNE_CACHE")
    return plan


# block rows (filtered spectra per block): 512, 256, 128, 64, 32 at 32 to 512
# channels, 32, 16, 8, 4 at 1024 to 8192
@pytest.mark.parametrize("C,T,S,B,dtype", [
    (32, 4, 513, 2, "ci16"), (32, 64, 511, 1, "c64"), (64, 3, 256, 3, "ci8"), (64, 17, 300, 1, "cf16"),
    (128, 1, 129, 2, "c64"), (128, 12, 1, 2, "ci8"), (128, 64, 127, 1, "ci16"), (256, 17, 65, 2, "ci8"),
    (256, 64, 64, 1, "cf16"), (512, 32, 33, 2, "c64"), (512, 33, 31, 1, "ci16"), (1024, 20, 33, 2, "c64"),
    (1024, 64, 65, 1, "ci8"), (1024, 32, 31, 3, "cf16"), (2048, 4, 17, 2, "c64"), (2048, 16, 16, 1, "ci8"),
    (2048, 31, 8, 2, "ci16"), (2048, 9, 9, 1, "cf16"), (2048, 32, 7, 1, "c64"), (4096, 16, 8, 2, "c64"),
    (4096, 3, 4, 1, "ci16"), (4096, 13, 5, 3, "ci8"), (4096, 32, 9, 1, "cf16"), (4096, 25, 3, 1, "c64"),
    (8192, 16, 5, 2, "c64"), (8192, 4, 2, 1, "ci8"), (8192, 7, 3, 1, "cf16"), (8192, 2, 4, 2, "ci16"),
    (2048, 16, 16 * 300 + 1, 1, "ci16"), (4096, 16, 8 * 130 + 3, 2, "ci8"), (128, 8, 128 * 520, 1, "c64"),
])
def test_blocked_equals_split(dev, C, T, S, B, dtype, tmp_path, monkeypatch):
    import torch
    from paper_1511_03599_amd import pfb
    say(f"blocked C={C} T={T} S={S} B={B} {dtype}")
    x = synth.device_quantised_noise((B, S + T - 1, C), dtype, 2600 + C + T, dev)
    h = taps_to_device(synth.random_taps(C, T, 2601), dev)
    plan = blocked_plan(pfb, C, T, S, B, dtype, tmp_path, monkeypatch)
    rows = (16384 // C) * (2 if C >= 1024 else 1)
    assert plan.info()["chunk_rows"] == rows
    assert dtype == "c64" or plan.info()["workspace_bytes"] == 0  # complex64 plans own the adjoint's
    Y = plan.execute(x, h)
    ref = pfb.Plan(C, T, S, B, dtype, pfb.NO_FUSE).execute(x, h)
    assert torch.equal(Y, ref)


@pytest.mark.parametrize("C,T", [(64, 12), (2048, 12), (4096, 30)])
def test_blocked_non_finite_samples(dev, C, T, tmp_path, monkeypatch):
    """An infinity and a NaN reach the same spectra as on the split path."""
    import torch
    from paper_1511_03599_amd import pfb
    S = 3 * (16384 // C) + 2 * T + 1  # some spectra stay finite
    say(f"blocked non-finite C={C} T={T} S={S}")
    x = synth.device_noise((1, S + T - 1, C), 2700 + C, dev)
    x[0, S // 2, 5] = float("inf")
    x[0, S - 1, C - 1] = complex(0.0, float("nan"))
    h = taps_to_device(synth.random_taps(C, T, 2701), dev)
    Y = blocked_plan(pfb, C, T, S, 1, "c64", tmp_path, monkeypatch).execute(x, h).cpu().numpy()
    ref = pfb.Plan(C, T, S, 1, "c64", pfb.NO_FUSE).execute(x, h).cpu().numpy()
    assert np.array_equal(Y.view(np.float32), ref.view(np.float32), equal_nan=True)
    assert np.isnan(ref).any() and np.isfinite(ref).any()


@pytest.mark.parametrize("CV,NS,T,S,dtype", [(512, 3, 16, 33, "ci8"), (512, 2, 4, 15, "c64"), (1024, 5, 32, 241, "ci16"),
                                             (2048, 9, 12, 65, "c64"), (4096, 8, 16, 33, "ci8"), (4096, 65, 3, 3, "cf16")])
def test_blocked_subbands_equal_streams(dev, CV, NS, T, S, dtype):
    """Each sub-band and polarisation gives the bits of a split plan run on
    that stream alone (sizes at which the blocked kernel runs)."""
    import torch
    from paper_1511_03599_amd import pfb
    say(f"blocked sub-bands C_V={CV} N_sub={NS} T={T} S={S} {dtype}")
    x = synth.device_quantised_noise((S + T - 1, NS, CV, 2), dtype, 2800 + CV, dev)
    h = taps_to_device(synth.random_taps(CV, T, 2801), dev)
    Y = pfb.VegasPlan(CV, NS, T, S, dtype).execute(x, h)
    plan = pfb.Plan(CV, T, S, 1, dtype, pfb.NO_FUSE)
    for sub in sorted({0, NS // 2, NS - 1}):
        for pol in range(2):
            ref = plan.execute(x[:, sub, :, pol].contiguous()[None], h)
            assert torch.equal(Y[:, sub, :, pol], ref[0]), (sub, pol)


@pytest.mark.parametrize("CV", [512, 1024, 2048, 4096])
@pytest.mark.parametrize("T", [3, 7, 13, 32])
def test_blocked_subbands_every_window_and_type(dev, CV, T):
    """Past the line (112 blocks) in every input type, the last block ragged;
    a blocked sub-band plan has no workspace."""
    import ctypes
    import torch
    from paper_1511_03599_amd import pfb
    NS, rows = 8, 16384 // CV * (2 if CV >= 1024 else 1) // 2
    S = 14 * rows - 1
    h = taps_to_device(synth.random_taps(CV, T, 2851), dev)
    for dtype in ("c64", "ci16", "ci8", "cf16"):
        say(f"blocked sub-bands C_V={CV} T={T} S={S} {dtype}")
        x = synth.device_quantised_noise((S + T - 1, NS, CV, 2), dtype, 2850 + CV + T, dev)
        vegas = pfb.VegasPlan(CV, NS, T, S, dtype)
        info = pfb.PlanInfo()
        pfb.check(pfb.lib().pfb_plan_get_info(vegas._h, ctypes.byref(info)))
        assert info.workspace_bytes == 0
        Y = vegas.execute(x, h)
        plan = pfb.Plan(CV, T, S, 1, dtype, pfb.NO_FUSE)
        for sub in (0, NS - 1):
            for pol in range(2):
                ref = plan.execute(x[:, sub, :, pol].contiguous()[None], h)
                assert torch.equal(Y[:, sub, :, pol], ref[0]), (dtype, sub, pol)
