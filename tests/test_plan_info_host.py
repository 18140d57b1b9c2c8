"""pfb_plan_get_info says what runs (launches recorded on the host)."""
import pytest

from hostlib import host_run


@pytest.mark.parametrize("C,T,S,flags,rows,taps", [
    (256, 48, 3000, "FIR_ONLY", 16, 48), (256, 33, 3000, "NO_FUSE", 16, 48), (300, 49, 5, "FIR_ONLY", 16, 64),
    (256, 65, 100, "0", 16, 80), (1000, 1024, 100, "FIR_ONLY", 16, 1024), (256, 48, 3000, "FIR_ONLY | PLAIN", 256, 64),
    (1024, 32, 2000, "FIR_ONLY", 32, 32)])
def test_fir_rows_and_padded_taps(tmp_path_factory, C, T, S, flags, rows, taps):
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, flags={flags})
events()
fir_only = ({flags}) & FIR_ONLY
assert L.pfb_execute(p, A, A, A if fir_only else None, None if fir_only else A, None) == 0
i = info(p)
result = [events()[0], i.fir_rows, i.padded_taps, i.fir_cpt]
""")
    (kernel, groups), fir_rows, padded, cpt = got
    assert (fir_rows, padded) == (rows, taps)
    assert groups == -(-(-(-S // fir_rows)) * -(-C // (64 * cpt)) // 4)
    assert ("fir_long_kernel" in kernel) == (rows == 16)


@pytest.mark.parametrize("C,T,S,B", [(128, 16, 4000, 3), (4096, 16, 8192, 2), (1024, 32, 16384, 1), (96, 5, 30, 1),
                                     (1024, 40, 3000, 1)])
def test_backward_rows_of_the_split_adjoint(tmp_path_factory, C, T, S, B):
    got = host_run(tmp_path_factory, f"""
p = plan({C}, {T}, {S}, {B})
events()
assert L.pfb_backward(p, A, A, A, A, A, None) == 0
result = [[e for e in events() if "gxgh" in e[0] or "fir_kernel" in e[0]], info(p).backward_rows]
""")
    (((kernel, groups),), rows) = got
    assert ("gxgh" in kernel) == (T <= 32)
    assert groups == -(-(B * -(-(S + T - 1) // rows) * -(-C // 64)) // 4)
