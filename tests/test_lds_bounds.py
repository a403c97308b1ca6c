"""Every LDS access of the smoothing passes lies inside the workgroup's
allocation, for every tile and form, lanes past the tile included (the host
mirrors the kernel's farthest indices; no GPU)."""
import ctypes

import pytest

PROLONG, NORM_IN, RESTRICT = 2, 4, 16


@pytest.fixture(scope="module")
def lib():
    from paper_1208_4247_amd import build, capi
    import os

    if not os.path.exists(capi.LIB_PATH):
        build.build()
    L = ctypes.CDLL(capi.LIB_PATH)

    def fn(name, result, ints):
        f = getattr(L, name)
        f.restype = result
        f.argtypes = [ctypes.c_int] * ints + [ctypes.c_size_t]
        return f

    return dict(count=L.gmg_tile_variant_count,
                slack=fn("_ZN3gmg17rb_pass_lds_slackEiiiim", ctypes.c_long, 4),
                fits=fn("_ZN3gmg12rb_pass_fitsEiiiim", ctypes.c_bool, 4),
                wj_slack=fn("_ZN3gmg17wj_pass_lds_slackEiiiim", ctypes.c_long, 4),
                wj_folds=fn("_ZN3gmg13wj_pass_foldsEiiim", ctypes.c_bool, 3))


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("stages", [2, 3, 4])
@pytest.mark.parametrize("elem", [4, 8])
def test_red_black(lib, dim, stages, elem):
    ran = 0
    for v in range(lib["count"](dim, 0, stages)):
        for flags in (0, PROLONG, NORM_IN, RESTRICT, RESTRICT | NORM_IN, RESTRICT | PROLONG):
            if lib["fits"](dim, stages, v, flags, elem):
                assert lib["slack"](dim, stages, v, flags, elem) >= 0, (v, flags)
                ran += 1
    assert ran >= 6


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("stages", [1, 2])
@pytest.mark.parametrize("elem", [4, 8])
def test_jacobi(lib, dim, stages, elem):
    for v in range(lib["count"](dim, 1, stages)):
        for flags in (0, PROLONG, RESTRICT, RESTRICT | PROLONG):
            if not flags & RESTRICT or lib["wj_folds"](dim, stages, v, elem):
                assert lib["wj_slack"](dim, stages, v, flags, elem) >= 0, (v, flags)
