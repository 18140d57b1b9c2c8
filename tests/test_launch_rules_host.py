"""The rules that choose kernels, tiles and workspaces, called in the built
library on the host (no device)."""
import ctypes
import os

import pytest

from hostlib import host_run


@pytest.fixture(scope="module")
def L():
    from paper_1511_03599_amd import pfb
    if not os.path.exists(pfb.LIB_PATH):
        pytest.skip("libpfb.so not built")
    return pfb.lib()


class GfftPass(ctypes.Structure):
    _fields_ = [("radix", ctypes.c_int), ("stride", ctypes.c_int), ("magic", ctypes.c_uint32), ("tw", ctypes.c_int)]


class GfftSched(ctypes.Structure):
    _fields_ = [("C", ctypes.c_int), ("npass", ctypes.c_int), ("group", ctypes.c_int),
                ("rows_per_block", ctypes.c_int), ("nt", ctypes.c_bool), ("tw_entries", ctypes.c_int),
                ("passes", GfftPass * 8)]


def test_mixed_radix_groups_write_whole_lines(L):
    """Groups of up to 16 lanes store past L2 only where rows start on sectors or
    the last pass is one step; rows off them have no group of 32 lanes where a
    wave is filled."""
    schedule = L._ZN3pfb13gfft_scheduleEiPNS_9GfftSchedE
    schedule.restype = ctypes.c_bool
    s = GfftSched()
    for C in range(33, 8192):
        if C & (C - 1) == 0 or not schedule(C, ctypes.byref(s)):
            continue
        assert s.group * s.rows_per_block == 256 or (s.group % 64 == 0 and s.rows_per_block == 1), C
        radix = [s.passes[p].radix for p in range(s.npass)]
        assert all(C // r <= s.group * (1 if r > 8 else 16 // r) for r in radix), C
        first, last = C // radix[0], C // radix[-1]
        if s.group <= 16:
            assert s.nt == (s.group == 16 and (C % 8 == 0 or last <= 16)), C
        else:
            assert s.nt and not (s.group == 32 and C % 8 and 35 <= first <= 64), C


@pytest.mark.parametrize("C,T,S,B,rows", [
    # tiles as high as at every size before, or fewer partials: never many
    # more of them than the reduction adds in the time the stream is read in
    (64, 8, 65536, 1, 64), (64, 4, 10000, 4, 64), (128, 16, 65536, 1, 96), (1024, 32, 16384, 1, 192), (1000, 16, 10000, 1, 16)])
def test_tiles_of_the_tap_gradient_alone(tmp_path_factory, C, T, S, B, rows):
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, {B})
events()
assert L.pfb_backward(p, A, A, A, None, A, None) == 0
result = [e for e in events() if "gh_partial" in e[0]]
""")
    assert len(got) >= 1
    waves = B * -(-C // 64) * -(-S // rows)
    assert sum(n for _, n in got) <= -(-waves // 4) + len(got)


@pytest.mark.parametrize("C,T,S,B,dtype,one", [
    (128, 20, 1, 1, "C64", False), (128, 32, 47, 1, "CF16", False), (128, 32, 48, 1, "C64", True),
    (128, 32, 15, 1, "CI8", False), (128, 17, 16, 1, "CI16", True), (128, 17, 5, 20, "C64", True),
    (256, 30, 15, 1, "C64", False), (256, 30, 16, 1, "CI8", True), (64, 32, 8, 1, "CF16", False),
    (32, 32, 1, 1, "C64", True), (128, 16, 1, 1, "C64", True)])
def test_part_of_a_block_at_17_to_32_taps(tmp_path_factory, C, T, S, B, dtype, one):
    """A handful of spectra take the two launches, not a whole block's time."""
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, {B}, {dtype})
events()
assert L.pfb_execute(p, A, A, None, A, None) == 0
result = [e[0] for e in events()]
""")
    assert len(got) == (1 if one else 2) and ("block_kernel" in got[0]) == one


@pytest.mark.parametrize("cus,blocks,one", [(256, 83, False), (256, 84, True), (32, 10, False), (32, 11, True)])
def test_lines_scale_with_the_compute_units(tmp_path_factory, cus, blocks, one):
    """The blocked kernel's lines are in blocks per compute unit (2048
    channels, 16 taps; sub-bands of 1024 channels from 72 for 256), and so is
    a beam's size for a launch of its own (here always the fused one)."""
    got = host_run(tmp_path_factory, f"""
rt.host_cus({cus})
def launches(f):
    events()
    assert f() == 0
    return [e[0] for e in events()]
p = plan(2048, 16, {blocks} * 16)
result = [launches(lambda: L.pfb_execute(p, A, A, None, A, None))]
v = vp()
assert L.pfb_plan_create_vegas(1024, 1, 16, {blocks - 12 if cus == 256 else blocks - 2} * 16, C64, ctypes.byref(v)) == 0
result.append(launches(lambda: L.pfb_execute_vegas(v, A, A, A, None)))
b, P = vp(), vp * 1
assert L.pfb_plan_create_batched(1, ctypes.byref(Desc(1024, 16, {16 * cus - (0 if one else 1)}, 1, C64, 0)), ctypes.byref(b)) == 0
result.append(launches(lambda: L.pfb_execute_batched(b, P(A.value), P(A.value), P(A.value), None)))
""")
    assert (len(got[0]) == 1 and "block_kernel" in got[0][0]) == one
    assert (len(got[1]) == 1 and "block_kernel" in got[1][0]) == one
    assert (len(got[2]) == 1 and "fused_fwd" in got[2][0]) == one


def test_new_buffers_of_a_beam_with_its_own_launch(tmp_path_factory):
    """They need no new pointer table, so no wait for the call before; new
    buffers of a beam of the persistent launch do."""
    got = host_run(tmp_path_factory, """
P = vp * 2
beams = (Desc * 2)(Desc(1024, 16, 4096, 1, C64, 0), Desc(64, 4, 100, 1, C64, 0))
b = vp()
assert L.pfb_plan_create_batched(2, beams, ctypes.byref(b)) == 0
def call(big, small):
    events()
    assert L.pfb_execute_batched(b, P(big, small), P(A.value, A.value), P(big, small), None) == 0
    return [e[0] if e[0] in ("wait", "copy", "graph") else "launch" for e in events()]
a = A.value
result = [call(a, a), call(a, a), call(a + 4096, a), call(a + 4096, a + 4096)]
""")
    first, same, big, small = got
    assert first == ["launch", "copy", "graph"] and same == big == ["launch", "graph"]
    assert small == ["launch", "wait", "copy", "graph"]


@pytest.mark.parametrize("C,T,S,dtype,long", [
    # window and long-tap FIR as measured, us
    (256, 35, 201231, "C64", False),    # 226, 278
    (1024, 33, 25246, "C64", False),    # 116, 128
    (4096, 41, 8410, "C64", False),     # 143, 153
    (8192, 57, 2442, "CI16", False),    # 82, 87
    (256, 64, 55183, "C64", False),     # 69, 94
    (256, 48, 3000, "C64", True),       # 33, 8
    (2048, 48, 14684, "C64", True),     # 129, 107
    (8192, 47, 1599, "C64", True),      # 75, 55
    (2048, 47, 4513, "CI8", True),      # 52, 34
    (4096, 35, 8000, "CF16", True),     # 125, 101 at 7645, int16
    (1000, 64, 56880, "CF16", True),    # 310, 245
])
def test_long_tap_fir_where_it_is_the_faster(tmp_path_factory, C, T, S, dtype, long):
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, 1, {dtype}, FIR_ONLY)
events()
assert L.pfb_execute(p, A, A, A, None, None) == 0
result = events()[0][0]
""")
    assert ("fir_long_kernel" in got) == long


@pytest.mark.parametrize("cus,blocks,groups", [(256, 165, 168), (256, 256, 256), (256, 300, 256), (256, 97, 104),
                                               (304, 301, 304), (60, 57, 57), (60, 300, 60)])
def test_blocked_grids_deal_runs_to_the_xcds(tmp_path_factory, cus, blocks, groups):
    """A multiple of eight workgroups where the compute units allow it."""
    got = host_run(tmp_path_factory, f"""
rt.host_cus({cus})
p = plan(128, 8, {blocks} * 128)
events()
assert L.pfb_execute(p, A, A, None, A, None) == 0
result = events()[0]
""")
    assert "block_kernel" in got[0] and got[1] == groups


@pytest.mark.parametrize("C,T,dtype,blocks,one", [
    # split / blocked time as measured at or beside that count
    (4096, 16, "C64", 92, False),    # 0.85
    (4096, 16, "C64", 100, True),    # 1.02
    (4096, 16, "CI8", 84, True),     # 1.03
    (4096, 32, "C64", 165, True), (4096, 32, "C64", 256, True),
    (4096, 32, "C64", 257, False),   # 0.86
    (4096, 32, "C64", 384, False),   # 0.96
    (4096, 32, "C64", 420, True),
    (4096, 24, "CI16", 300, False), (4096, 24, "CI16", 330, True),
    (8192, 8, "C64", 92, False),     # 0.90
    (8192, 16, "C64", 320, False), (8192, 16, "C64", 344, True), (8192, 16, "CI8", 257, False), (8192, 16, "CI8", 280, True),
    (1024, 32, "CF16", 100, False), (1024, 32, "C64", 84, True),
    (1024, 64, "CI8", 300, False),   # 0.89
    (1024, 64, "CI8", 384, True), (256, 48, "CF16", 300, False), (256, 48, "C64", 280, True)])
def test_blocked_lines(tmp_path_factory, C, T, dtype, blocks, one):
    rows = 16384 // C * (2 if C >= 1024 else 1)
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {blocks * rows}, 1, {dtype})
events()
assert L.pfb_execute(p, A, A, None, A, None) == 0
result = [e[0] for e in events()]
""")
    assert (len(got) == 1 and "block_kernel" in got[0]) == one


@pytest.mark.parametrize("C,T,S,dtype,rows", [
    # tall and short tiles as measured, us
    (2048, 16, 4000, "CI8", 64),     # 16.5, 21.8
    (1024, 32, 8000, "C64", 128),    # 25.4, 32.4
    (1024, 16, 7600, "C64", 32),     # 24.2, 28.7
    (4096, 8, 1000, "CF16", 32),     # 8.1, 8.8
    (1024, 16, 900, "C64", 16),      # 9.0, 6.7
    (1024, 32, 2000, "C64", 32),     # 28, 11
    (1024, 20, 8000, "C64", 32), (1024, 20, 16000, "CF16", 32),
    (1024, 16, 1600, "CI16", 16), (2048, 32, 2000, "CI8", 32)])
def test_short_fir_tiles_for_few_waves(tmp_path_factory, C, T, S, dtype, rows):
    assert host_run(tmp_path_factory, f"result = info(plan({C}, {T}, {S}, 1, {dtype}, FIR_ONLY)).fir_rows") == rows


@pytest.mark.parametrize("C,T,S,B", [(64, 8, 100000, 1), (128, 16, 65536, 1), (32, 4, 1000, 300), (128, 24, 70000, 2),
                                     (64, 50, 90000, 1), (4096, 16, 8192, 2), (96, 16, 300000, 1)])
def test_tap_gradient_sums_are_no_longer_than_before(tmp_path_factory, C, T, S, B):
    """The longest serial sum, of a tile's rows or of a quarter of the
    partials, is no longer than 256-row tiles make it."""
    rows, (both, alone) = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, {B})
def tiles(gx, kernel):
    events()
    assert L.pfb_backward(p, A, A, A, gx, A, None) == 0
    return sum(n for k, n in events() if kernel in k) * 4 // {-(-C // 64)}
result = [info(p).backward_rows, [tiles(A, "gxgh" if {T} <= 32 else "gh_partial"), tiles(None, "gh_partial")]]
""")
    raw = S + T - 1
    most = max(256, B * -(-raw // 256) // 4)
    assert max(both, alone) // 4 <= most * 1.05 + 2
    if T <= 32:
        assert rows <= 256 and B * -(-raw // rows) // 4 <= most
