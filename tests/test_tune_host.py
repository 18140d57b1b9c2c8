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


TUNE = """
import os
cache = os.environ["PFB_TUNE_CACHE"]
os.environ.pop("PFB_TUNE_CACHE")
d = Desc({C}, {T}, {S}, 1, {dtype}, {flags})
rt.host_time({kernel!r}.encode(), ctypes.c_float({ms}))
assert L.pfb_tune(ctypes.byref(d), cache.encode()) == 0
events()
libc = ctypes.CDLL(None)
libc.setenv(b"PFB_TUNE_CACHE", cache.encode(), 1)
p = plan({C}, {T}, {S}, 1, {dtype}, {flags})
events()
Y = None if {flags} & FIR_ONLY else A
assert L.pfb_execute(p, A, A, A if {flags} & FIR_ONLY else None, Y, None) == 0
result = dict(launches=events(), line=dict(f.split("=") for f in open(cache).read().split()[6:]), rows=info(p).fir_rows)
"""


def tuned(tmp_path_factory, tmp_path, **kw):
    """Tune with every launch taking 1 ms but those of `kernel`, then what a
    plan with that cache launches."""
    return host_run(tmp_path_factory, TUNE.format(**{"dtype": "C64", "flags": "0", "ms": 0.5, **kw}),
                    {"PFB_TUNE_CACHE": str(tmp_path / "tuned.txt")})


@pytest.mark.parametrize("T,flags", [(33, "FIR_ONLY"), (48, "FIR_ONLY"), (64, "FIR_ONLY"), (48, "NO_FUSE")])
def test_tuner_can_choose_the_long_tap_fir(tmp_path_factory, tmp_path, T, flags):
    got = tuned(tmp_path_factory, tmp_path, C=256, T=T, S=3000, flags=flags, kernel="fir_long_kernel")
    assert "fir_long_kernel" in got["launches"][0][0] and got["line"]["segments"] == "1"
    (tmp_path / "tuned.txt").unlink()
    got = tuned(tmp_path_factory, tmp_path, C=256, T=T, S=3000, flags=flags, kernel="fir_long_kernel", ms=2.0)
    assert "fir_long_kernel" not in got["launches"][0][0] and got["line"]["segments"] == "0"


@pytest.mark.parametrize("line,long", [
    ("gfx950 0 256 48 1 3000 fir_cpt=1 fir_sb=64 segments=0", False),
    ("gfx950 0 256 48 1 3000 fir_cpt=1 segments=1", True),
    ("gfx950 0 256 48 1 3000 fir_cpt=1 fir_sb=64", True),        # written without the choice: the rule
    ("gfx950 0 256 48 1 2900 fir_cpt=1 fir_sb=64 segments=0", True),  # another length: the rule
])
def test_long_tap_fir_beside_an_entry(tmp_path_factory, tmp_path, line, long):
    got = plans_with(tmp_path_factory, tmp_path, [line], """
p = plan(256, 48, 3000, flags=FIR_ONLY)
events()
assert L.pfb_execute(p, A, A, A, None, None) == 0
result = events()[0][0]
""")
    assert ("fir_long_kernel" in got) == long
    plain = plans_with(tmp_path_factory, tmp_path, ["gfx950 0 256 48 1 3000 segments=1"], """
p = plan(256, 48, 3000, flags=FIR_ONLY | PLAIN)
events()
assert L.pfb_execute(p, A, A, A, None, None) == 0
result = events()[0][0]
""")
    assert "fir_long_kernel" not in plain


def test_blocked_choice_keeps_the_timed_fir(tmp_path_factory, tmp_path):
    """Where the blocked kernel wins, the FIR of the other calls is the one
    that was fastest in two launches (all take the same time here: the first
    one timed), not an untimed height."""
    got = tuned(tmp_path_factory, tmp_path, C=256, T=48, S=3000, kernel="block_kernel", ms=0.25)
    assert got["line"]["block"] == "1" and "block_kernel" in got["launches"][0][0]
    assert got["line"]["fir_cpt"] == "1" and got["line"]["fir_sb"] == "16" and got["line"]["segments"] == "0"
    (tmp_path / "tuned.txt").unlink()
    got = tuned(tmp_path_factory, tmp_path, C=4096, T=4, S=3000, kernel="block_kernel", ms=0.25)
    assert got["line"]["block"] == "1" and got["line"]["fir_sb"] == "16"
