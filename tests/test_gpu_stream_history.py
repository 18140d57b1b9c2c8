"""Streams cut into calls of fewer, as many and more new spectra than the T-1
carried ones (the headroom and the last rows overlap, touch or are apart), in
rows that are and are not a multiple of 16 bytes."""
import numpy as np
import pytest

from paper_1511_03599_amd import synth
from helpers import say, taps_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T,S,B,dtype,flags", [
    (1024, 16, 14, 2, "ci16", 0), (1024, 16, 15, 2, "ci16", 0), (1024, 16, 16, 1, "c64", 0),
    (3, 5, 3, 2, "ci8", 1), (3, 5, 4, 2, "ci8", 1), (5, 9, 8, 3, "cf16", 1), (64, 2, 1, 3, "ci8", 0),
])
def test_history_rotation(dev, C, T, S, B, dtype, flags):
    import torch
    from paper_1511_03599_amd import pfb
    k = 5
    say(f"history rotation C={C} T={T} S={S} B={B} {dtype} flags={flags}")
    new = synth.device_quantised_noise((B, k * S, C), dtype, 3200 + C, dev)
    h = taps_to_device(synth.random_taps(C, T, 3201), dev)
    full = torch.cat([torch.zeros_like(new[:, :1]).expand(-1, T - 1, *new.shape[2:]), new], dim=1).contiguous()
    ref = pfb.Plan(C, T, k * S, B, dtype, flags).execute(full, h)
    plan = pfb.Plan(C, T, S, B, dtype, flags | pfb.STREAMING)
    buf = plan.stream_buffer(dev)
    for i in range(k):
        buf[:, T - 1:] = new[:, i * S:(i + 1) * S]
        out = plan.execute_stream(buf, h)
        assert torch.equal(out, ref[:, i * S:(i + 1) * S]), i
        # the headroom holds the carried spectra
        assert torch.equal(buf[:, :T - 1], full[:, i * S:i * S + T - 1]), i
