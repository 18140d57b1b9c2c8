"""libpfb.so over the host runtime of host_hip.cpp, in a process of its own
(no torch, no device): host_run(code) runs `code` after PRELUDE and returns
what it assigned to `result`."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1511_03599_amd", "libpfb.so")
ROCM = "/opt/rocm/include"

PRELUDE = '''
import ctypes, json, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
rt.host_events.restype = ctypes.c_char_p
rt.host_allocated.restype = ctypes.c_size_t
rt.host_time.argtypes = [ctypes.c_char_p, ctypes.c_float]
vp, i64 = ctypes.c_void_p, ctypes.c_int64
for f in ("pfb_execute", "pfb_execute_stream"):
    getattr(L, f).argtypes = [vp] * 6
L.pfb_backward.argtypes = [vp] * 7
L.pfb_execute_batched.argtypes = [vp] * 5
L.pfb_execute_vegas.argtypes = [vp] * 5
C64, CI16, CI8, CF16 = range(4)
FIR_ONLY, NO_FUSE, PLAIN, STREAMING = 1, 4, 8, 16

class Desc(ctypes.Structure):
    _fields_ = [("channels", ctypes.c_int32), ("taps", ctypes.c_int32), ("spectra", i64), ("batch", ctypes.c_int32),
                ("dtype", ctypes.c_int32), ("flags", ctypes.c_uint32)]

class Info(ctypes.Structure):
    _fields_ = [("path", ctypes.c_int32), ("fir_rows", ctypes.c_int32), ("fir_cpt", ctypes.c_int32),
                ("padded_taps", ctypes.c_int32), ("workspace_bytes", i64), ("chunk_rows", i64),
                ("backward_fused", ctypes.c_int32), ("fused_ws", ctypes.c_int32), ("backward_rows", ctypes.c_int32)]

def plan(C, T, S, B=1, dtype=C64, flags=0):
    h = vp()
    assert L.pfb_plan_create(ctypes.byref(Desc(C, T, S, B, dtype, flags)), ctypes.byref(h)) == 0
    return h

def info(h):
    i = Info()
    assert L.pfb_plan_get_info(h, ctypes.byref(i)) == 0
    return i

def events():
    """What the library did since the last call: (kernel, workgroups), or
    the name of a wait, a copy or a graph launch."""
    out = []
    for line in rt.host_events().decode().splitlines():
        f = line.split()
        out.append((f[1], int(f[2])) if f[0] == "launch" else (f[0], 0))
    return out

A = vp(1 << 20)  # a device address that nothing follows
'''


def host_run(tmp_path_factory, code: str, env: dict | None = None):
    if not os.path.exists(LIB):
        pytest.skip("libpfb.so not built")
    so = os.path.join(tmp_path_factory.getbasetemp(), "host_hip.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM,
                        os.path.join(HERE, "host_hip.cpp"), "-o", so], check=True)
    full = {k: v for k, v in os.environ.items() if k != "PFB_TUNE_CACHE"}
    r = subprocess.run([sys.executable, "-c", PRELUDE + code + "\nprint(json.dumps(result))", so, LIB],
                       env={**full, **(env or {})}, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.splitlines()[-1])
