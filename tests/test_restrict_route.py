"""The full weighting of a right-hand side itself (no iterate) is refused, before
any launch, together with a stop test or a table of problems, which its kernel
does not know."""
import ctypes

import pytest

HIP_ERROR_INVALID_VALUE = 1


class RestrictArgs(ctypes.Structure):
    _fields_ = [("u", ctypes.c_void_p), ("f", ctypes.c_void_p), ("fc", ctypes.c_void_p),
                ("active", ctypes.c_void_p), ("m", ctypes.c_int), ("mc", ctypes.c_int),
                ("inv_h2", ctypes.c_double), ("fin_partials", ctypes.c_void_p),
                ("fin_n", ctypes.c_int), ("fin_state", ctypes.c_void_p)]


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("what", ["partials", "state", "table", "entries"])
def test_no_iterate_with_stop_test_or_table(dim, what):
    import os

    from paper_1208_4247_amd import build, capi

    if not os.path.exists(capi.LIB_PATH):
        build.build()
    fn = getattr(ctypes.CDLL(capi.LIB_PATH), "_ZN3gmg15launch_restrictIdEE10hipError_tiNS_12"
                 "RestrictArgsIT_EEP12ihipStream_tPKS4_i")
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_int, RestrictArgs, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int]
    buf = ctypes.create_string_buffer(4096)  # (host memory: never launched with)
    at = ctypes.addressof(buf)
    a = RestrictArgs(u=None, f=at, fc=at + 2048, m=7, mc=3, inv_h2=64.0)
    if what == "partials":
        a.fin_partials = at
    elif what == "state":
        a.fin_state = at
    assert fn(dim, a, None, at if what == "table" else None, 2 if what == "entries" else 1) == \
        HIP_ERROR_INVALID_VALUE
