"""A sine-transform set-up that finds no host memory for its tables returns a status:
no C++ exception crosses the C entry (no GPU: it ends before any HIP call)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, resource, sys
from paper_1208_4247_amd import capi
L = ctypes.CDLL(capi.LIB_PATH)
L.gmg_dst_setup.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p,
                            ctypes.POINTER(ctypes.c_size_t), ctypes.c_void_p,
                            ctypes.POINTER(ctypes.c_void_p)]
libc = ctypes.CDLL(None)
libc.malloc.restype = ctypes.c_void_p
libc.malloc.argtypes = [ctypes.c_size_t]
n, h = ctypes.c_size_t(0), ctypes.c_void_p()
assert L.gmg_dst_setup(2, 12, None, ctypes.byref(n), None, None) == 0
held = 0
pages = int(open("/proc/self/statm").read().split()[0])
resource.setrlimit(resource.RLIMIT_AS, (pages * 4096, resource.RLIM_INFINITY))
while libc.malloc(160000) and held < 4096:  # (the tables take 163848 bytes)
    held += 1
s = L.gmg_dst_setup(2, 12, 4096, ctypes.byref(n), None, ctypes.byref(h))
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
assert held < 4096 and h.value is None
print("status", s)
"""


def test_no_memory_is_a_status():
    from paper_1208_4247_amd import build, capi

    if not os.path.exists(capi.LIB_PATH):
        build.build()
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, timeout=120,
                       cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["status", str(capi.GMG_ERR_HIP)]
