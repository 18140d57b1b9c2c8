"""Tiles and transform schedules of every shape that the size rules give. Fused
tiles: from one transform round (8 or 16 rows) at short streams to 128 rows,
with streams that end inside, at and just past a tile; split adjoint tiles;
mixed-radix schedules and groups."""
import numpy as np
import pytest

import oracle
from paper_1511_03599_amd import synth
from helpers import GH_TOL, GX_TOL, SPEC_TOL, c128, rel_l2, say, taps_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T,S,B,dtype", [
    (1024, 16, 7, 1, "c64"), (1024, 16, 8, 2, "ci16"), (1024, 9, 9, 1, "ci8"), (1024, 4, 2049, 1, "cf16"),
    (1024, 16, 4097, 1, "c64"), (1024, 8, 999, 17, "ci8"), (512, 16, 8, 1, "c64"), (512, 3, 17, 3, "ci16"),
    (512, 12, 8193, 1, "c64"), (512, 8, 100, 300, "ci8"), (256, 8, 16, 1, "cf16"), (256, 16, 33, 2, "c64"),
    (256, 5, 16385, 1, "ci8"),
])
def test_forward_tiles_equal_split(dev, C, T, S, B, dtype):
    import torch
    from paper_1511_03599_amd import pfb
    x = synth.device_quantised_noise((B, S + T - 1, C), dtype, 2900 + C + T, dev)
    h = taps_to_device(synth.random_taps(C, T, 2901), dev)
    plan = pfb.Plan(C, T, S, B, dtype)
    say(f"forward tiles C={C} T={T} S={S} B={B} {dtype}: {plan.info()['fir_rows']} rows")
    assert plan.info()["path"] == "fused"
    ref = pfb.Plan(C, T, S, B, dtype, pfb.NO_FUSE).execute(x, h)
    assert torch.equal(plan.execute(x, h), ref)


@pytest.mark.parametrize("C,T,S,B", [(1024, 16, 17, 1), (1024, 7, 600, 3), (1024, 16, 2000, 1), (512, 16, 1001, 3),
                                     (512, 4, 29, 1), (256, 16, 1, 2), (256, 8, 3000, 2)])
def test_adjoint_tiles(dev, C, T, S, B):
    from paper_1511_03599_amd import pfb
    x = synth.quantise(synth.complex_gaussian((B, S + T - 1, C), 2950 + C), "c64")
    h = synth.random_taps(C, T, 2951)
    gY = synth.quantise(synth.complex_gaussian((B, S, C), 2952), "c64")
    plan = pfb.Plan(C, T, S, B, "c64")
    rows_per_tile = plan.info()["backward_rows"]
    say(f"adjoint tiles C={C} T={T} S={S} B={B}: {rows_per_tile} rows")
    gx, gh = plan.backward(to_device(x, dev), taps_to_device(h, dev), to_device(gY, dev))
    rows = sorted(r for r in {0, 1, T - 1, rows_per_tile - 1, rows_per_tile, 3 * rows_per_tile, S - 1, S + T - 2}
                  if 0 <= r < S + T - 1)
    gx_r = oracle.pfb_adjoint_x_rows(h, gY, rows)
    assert max(rel_l2(c128(gx[b, rows]), gx_r[b]) for b in range(B)) <= GX_TOL
    ch = [0, 1, C // 2, C - 1]
    gh_r = oracle.pfb_adjoint_h_channels(x, gY, T, ch)
    assert rel_l2(gh[:, ch].cpu().numpy().astype(np.float64), gh_r) <= GH_TOL


@pytest.mark.parametrize("C,T,S,B", [(128, 16, 1, 1), (64, 9, 15, 2), (32, 3, 700, 3), (128, 5, 4000, 1), (2048, 17, 33, 2),
                                     (96, 31, 200, 2), (4096, 8, 170, 1), (1000, 12, 90, 1)])
def test_split_adjoint_tiles(dev, C, T, S, B):
    """Tiles of one unrolled block and more, ragged last tiles and channel
    counts that are no multiple of a wave."""
    from paper_1511_03599_amd import pfb
    say(f"split adjoint tiles C={C} T={T} S={S} B={B}")
    x = synth.quantise(synth.complex_gaussian((B, S + T - 1, C), 2970 + C), "c64")
    h = synth.random_taps(C, T, 2971)
    gY = synth.quantise(synth.complex_gaussian((B, S, C), 2972), "c64")
    plan = pfb.Plan(C, T, S, B, "c64")
    assert plan.info()["backward_kind"] == "split"
    gx, gh = plan.backward(to_device(x, dev), taps_to_device(h, dev), to_device(gY, dev))
    gx_r, gh_r = oracle.pfb_adjoint(x, h, gY)
    assert rel_l2(c128(gx), gx_r) <= GX_TOL
    assert rel_l2(gh.cpu().numpy().astype(np.float64), gh_r) <= GH_TOL


# schedules with every radix, every group width (4 lanes to 13 waves) and a
# row count that leaves a block part empty
@pytest.mark.parametrize("C,S", [(36, 7), (45, 70), (50, 3), (54, 65), (63, 5), (162, 33), (240, 17), (280, 9), (6000, 3),
                                 (8000, 2), (8100, 2), (7203, 3)])
def test_mixed_radix_schedules(dev, C, S):
    from paper_1511_03599_amd import pfb
    T, B = 3, 2
    say(f"mixed-radix schedule C={C} S={S}")
    x = synth.quantise(synth.complex_gaussian((B, S + T - 1, C), 2980 + C), "c64")
    h = synth.random_taps(C, T, 2981)
    gY = synth.quantise(synth.complex_gaussian((B, S, C), 2982), "c64")
    plan = pfb.Plan(C, T, S, B, "c64")
    args = (to_device(x, dev), taps_to_device(h, dev))
    assert rel_l2(c128(plan.execute(*args)), oracle.pfb_forward(x, h)) <= SPEC_TOL
    gx, gh = plan.backward(*args, to_device(gY, dev))
    gx_r, gh_r = oracle.pfb_adjoint(x, h, gY)
    assert rel_l2(c128(gx), gx_r) <= GX_TOL
    assert rel_l2(gh.cpu().numpy().astype(np.float64), gh_r) <= GH_TOL


# rows off the sectors: 16-lane groups that store through L2, groups widened
# to a wave; row counts that leave a block part empty
@pytest.mark.parametrize("C,S", [(125, 33), (147, 15), (175, 17), (252, 5), (343, 9), (441, 6)])
def test_mixed_radix_rows_off_the_lines(dev, C, S):
    test_mixed_radix_schedules(dev, C, S)


@pytest.mark.parametrize("T", [3, 9, 13, 16])
@pytest.mark.parametrize("S", [127, 129, 300, 700])
def test_tested_form_of_the_fused_tiles(dev, T, S, tmp_path, monkeypatch):
    """Tiles of 128 rows at 1024 channels (the form that tests its rows) with
    ragged last tiles, padded taps and rows before the stream."""
    import torch
    from paper_1511_03599_amd import pfb
    C, B = 1024, 2
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    h = taps_to_device(synth.random_taps(C, T, 2921), dev)
    for dtype in ("c64", "ci16", "ci8", "cf16"):
        say(f"tested form T={T} S={S} {dtype}")
        cache = tmp_path / f"{dtype}.txt"
        cache.write_text(f"{arch} {pfb.DTYPE_CODES[dtype]} {C} {T} {B} {S} path=0 fused_ws=0 fused_sb=128\n")
        monkeypatch.setenv("PFB_TUNE_CACHE", str(cache))
        plan = pfb.Plan(C, T, S, B, dtype)
        monkeypatch.delenv("PFB_TUNE_CACHE")
        info = plan.info()
        assert info["path"] == "fused" and info["fir_rows"] == 128 and not info["fused_ws"]
        x = synth.device_quantised_noise((B, S + T - 1, C), dtype, 2920 + T + S, dev)
        ref = pfb.Plan(C, T, S, B, dtype, pfb.NO_FUSE).execute(x, h)
        assert torch.equal(plan.execute(x, h), ref), dtype
