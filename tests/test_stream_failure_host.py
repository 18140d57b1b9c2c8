"""A streaming call whose filter bank does not launch leaves the carried
spectra as they were (launches on the host; the streaming copies run there)."""
import pytest

from hostlib import host_run


@pytest.mark.parametrize("C,T,S,B,flags,kernel", [
    (256, 4, 8, 2, "0", "fused_fwd"), (256, 4, 2, 2, "0", "fused_fwd"), (64, 5, 4, 1, "0", "block_kernel"),
    (48, 3, 7, 3, "NO_FUSE", "gfft_kernel"), (3, 4, 5, 2, "FIR_ONLY", "fir_kernel"), (64, 70, 69, 1, "0", "fir_long")])
def test_failed_launch_keeps_the_carried_spectra(tmp_path_factory, C, T, S, B, flags, kernel):
    got = host_run(tmp_path_factory, f"""
C, T, S, B = {C}, {T}, {S}, {B}
p = plan(C, T, S, B, CF16, STREAMING | {flags})
n = B * (S + T - 1) * C
raw = ctypes.create_string_buffer(n * 4 + 64)
addr = (ctypes.addressof(raw) + 15) // 16 * 16
x = (ctypes.c_uint32 * n).from_address(addr)
fir = {flags} & FIR_ONLY
def call(first):
    for i in range(n):
        x[i] = first + i
    return L.pfb_execute_stream(p, vp(addr), A, A if fir else None, None if fir else A, None)
def headroom():
    return [x[(b * (S + T - 1) + r) * C] for b in range(B) for r in range(T - 1)]
result = [call(1000), headroom()]
rt.host_fail(b"{kernel}")
result += [call(1000000)]
L.pfb_last_error.restype = ctypes.c_char_p
result += [L.pfb_last_error().decode()]
rt.host_fail(b"")
result += [call(2000000), headroom(), call(3000000), headroom()]
""")
    ok, head0, failed, why, ok2, head2, ok3, head3 = got
    rows = S + T - 1
    assert (ok, ok2, ok3, failed) == (0, 0, 0, 4) and "launch" in why
    assert head0 == [0] * (B * (T - 1))

    def carried(first, before):
        """The last T-1 rows of the call that began with `first` (its headroom
        rows held `before`)."""
        out = []
        for b in range(B):
            all_rows = before[b * (T - 1):(b + 1) * (T - 1)] + [first + (b * rows + r) * C for r in range(T - 1, rows)]
            out += all_rows[-(T - 1):]
        return out
    assert head2 == carried(1000, head0)
    assert head3 == carried(2000000, head2)
