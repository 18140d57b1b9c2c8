"""What plans take from a tuning cache and what the tuner writes, on the host
(launches recorded, their times given by the test)."""
import pytest

from hostlib import host_run


def plans_with(tmp_path_factory, tmp_path, lines, code):
    cache = tmp_path / "tune.txt"
    cache.write_text("".join(l + "\n" for l in lines))
    return host_run(tmp_path_factory, code, {"PFB_TUNE_CACHE": str(cache)})


@pytest.mark.parametrize("line,rows", [
    ("gfx950 0 1024 32 1 1900 fir_cpt=1 fir_sb=128", 32),   # another length: its height does not carry over
    ("gfx950 0 1024 32 1 2000 fir_cpt=1", 32),              # no height
    ("gfx950 0 1024 32 1 2000 fir_cpt=1 fir_sb=64", 64),
    ("gfx950 0 1024 31 1 2000 fir_cpt=1 fir_sb=64", 32),    # other taps
    ("gfx950 0 1024 32 1 900000 fir_cpt=1 fir_sb=128", 32),
])
def test_short_launches_keep_short_tiles_beside_an_entry(tmp_path_factory, tmp_path, line, rows):
    got = plans_with(tmp_path_factory, tmp_path, [line], "result = info(plan(1024, 32, 2000, flags=FIR_ONLY)).fir_rows")
    assert got == rows


@pytest.mark.parametrize("line,rows", [
    ("gfx950 0 1024 16 1 900 path=0 fused_ws=0", 16), ("gfx950 0 1024 16 1 900 fir_cpt=2", 16),
    ("gfx950 0 1024 16 1 1000 fir_cpt=1 fir_sb=64", 32), ("gfx950 0 1024 16 1 900 fir_cpt=1 fir_sb=64", 64)])
def test_heights_up_to_16_taps_beside_an_entry(tmp_path_factory, tmp_path, line, rows):
    got = plans_with(tmp_path_factory, tmp_path, [line], "result = info(plan(1024, 16, 900, flags=FIR_ONLY)).fir_rows")
    assert got == rows
