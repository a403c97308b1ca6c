"""Every LDS access of the red-black passes lies inside the workgroup's
allocation, for every tile and form, lanes past the tile included (the host
mirrors the kernel's farthest indices; no GPU)."""
import ctypes

import pytest

PROLONG, NORM_IN, RESTRICT = 2, 4, 16
MAX_LDS = 160 * 1024


@pytest.fixture(scope="module")
def lib():
    from paper_1208_4247_amd import build, capi
    import os

    if not os.path.exists(capi.LIB_PATH):
        build.build()
    L = ctypes.CDLL(capi.LIB_PATH)
    slack = getattr(L, "_ZN3gmg17rb_pass_lds_slackEiiiim")
    slack.restype = ctypes.c_long
    slack.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t]
    fits = getattr(L, "_ZN3gmg12rb_pass_fitsEiiiim")
    fits.restype = ctypes.c_bool
    fits.argtypes = slack.argtypes
    return L, slack, fits


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("stages", [2, 3, 4])
@pytest.mark.parametrize("elem", [4, 8])
def test_accesses_stay_inside(lib, dim, stages, elem):
    L, slack, fits = lib
    ran = 0
    for v in range(L.gmg_tile_variant_count(dim, 0, stages)):
        for flags in (0, PROLONG, NORM_IN, RESTRICT, RESTRICT | NORM_IN, RESTRICT | PROLONG):
            if fits(dim, stages, v, flags, elem):
                assert slack(dim, stages, v, flags, elem) >= 0, (v, flags)
                ran += 1
    assert ran >= 6
