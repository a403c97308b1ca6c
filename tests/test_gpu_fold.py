"""The restriction folded into the last pre-smoothing pass, tile by tile: the
profile says that a set tile runs the folded form exactly where it fits, and
the bits are those of the separate restriction."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu

PROLONG, NORM_IN, RESTRICT = 2, 4, 16


def _lib():
    from paper_1208_4247_amd import capi

    return capi, capi.lib()


def _folds(dim, stages, v, smoother, prec, form=NORM_IN):
    """The library's own rule: whether the tile runs the form with the fold."""
    capi, _ = _lib()
    L = ctypes.CDLL(capi.LIB_PATH)
    name = "_ZN3gmg13wj_pass_foldsEiiim" if smoother == "wj" else "_ZN3gmg12rb_pass_fitsEiiiim"
    fn = getattr(L, name)
    fn.restype = ctypes.c_bool
    args = [dim, stages, v] + ([] if smoother == "wj" else [form | RESTRICT])
    fn.argtypes = [ctypes.c_int] * len(args) + [ctypes.c_size_t]
    return fn(*args, 8 if prec == "fp64" else 4)


def _solve(plan, f, cycles):
    u = torch.zeros_like(f)
    plan.solve(u, f, rtol=1e-30, maxit=cycles)
    return u.cpu().numpy()


@pytest.mark.parametrize("dim,L,smoother,stages", [
    (3, 6, "rbgs", 2), (3, 7, "rbgs", 2), (3, 6, "rbgs", 4), (3, 7, "rbgs", 4), (2, 7, "rbgs", 2),
    (2, 8, "rbgs", 4), (3, 6, "wj", 2), (3, 7, "wj", 2), (2, 7, "wj", 2)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_every_tile_folds_where_it_fits(dim, L, smoother, stages, prec):
    capi, lib = _lib()
    nu1 = stages if smoother == "wj" else stages // 2  # one pass
    kw = dict(nu1=nu1, nu2=1, smoother=smoother, precision=prec)
    if prec == "mixed":
        kw["inner_cycles"] = 2
    f = torch.from_numpy(wl.rhs_uniform(dim, (1 << L) - 1, seed=840 + L)).cuda()
    base = capi.GMG_PROFILE | capi.GMG_NO_CROSS_CYCLE
    from paper_1208_4247_amd.solver import Plan

    ref = Plan(dim, L, flags=base | capi.GMG_NO_FUSED_RESTRICT, **kw)
    want = _solve(ref, f, 2)
    apart = ref.profile()["resid_restrict_l0"]["launches"]
    assert apart > 0
    folded = 0
    for v in range(lib.gmg_tile_variant_count(dim, 1 if smoother == "wj" else 0, stages)):
        for tz in (0, 5, 16):
            plan = Plan(dim, L, flags=base, **kw)
            plan.set_tile(0, stages, v, tz)
            assert np.array_equal(_solve(plan, f, 2), want), (v, tz)
            fold = _folds(dim, stages, v, smoother, prec)
            assert plan.profile()["resid_restrict_l0"]["launches"] == (0 if fold else apart), (v, tz)
            folded += fold
    assert folded > 0


@pytest.mark.parametrize("dim,L", [(3, 6), (3, 7), (2, 8)])
@pytest.mark.parametrize("nu", [(1, 1), (2, 1)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_every_three_stage_tile_runs_as_set(dim, L, nu, prec):
    capi, lib = _lib()
    from paper_1208_4247_amd.solver import Plan

    kw = dict(nu1=nu[0], nu2=nu[1], precision=prec)
    if prec == "mixed":
        kw["inner_cycles"] = 4
    cycles = 4 if prec == "fp64" else 1
    f = torch.from_numpy(wl.rhs_uniform(dim, (1 << L) - 1, seed=850 + L)).cuda()
    want = _solve(Plan(dim, L, flags=capi.GMG_NO_CROSS_CYCLE | capi.GMG_NO_FUSED_RESTRICT, **kw),
                  f, cycles)
    form = NORM_IN if nu[0] > 1 else PROLONG
    folded = 0
    for v in range(lib.gmg_tile_variant_count(dim, 0, 3)):
        for tz in (0, 5, 16):
            plan = Plan(dim, L, flags=capi.GMG_PROFILE, **kw)
            plan.set_tile(0, 2 * nu[0], 0, 8)  # the first cycle's pass
            try:
                plan.set_tile(0, 3, v, tz)
            except capi.GmgError:
                continue  # runs neither form
            tile = plan.get_tile(0, 2)
            assert tile[:2] == (3, v)
            assert np.array_equal(_solve(plan, f, cycles), want), (v, tz)
            assert plan.get_tile(0, 2) == tile
            apart = plan.profile()["resid_restrict_l0"]["launches"]
            fold = _folds(dim, 3, v, "rbgs", prec, form)
            # the first cycle may restrict apart, the three after it do not
            assert apart <= 1 if fold else apart >= 3, (v, tz, apart)
            folded += fold
    assert folded > 0


@pytest.mark.parametrize("smoother,nu1,problems", [
    ("wj", 2, [(2, 8), (2, 9), (3, 8), (2, 8)]), ("rbgs", 1, [(2, 7), (2, 9), (3, 8), (2, 8)])])
def test_batches_fold_by_default(smoother, nu1, problems):
    capi, _ = _lib()
    from paper_1208_4247_amd.solver import BatchPlan

    fs = [torch.from_numpy(wl.rhs_uniform(d, (1 << L) - 1, seed=860 + i)).cuda()
          for i, (d, L) in enumerate(problems)]
    out, apart = [], []
    for flags in (0, capi.GMG_NO_FUSED_RESTRICT):
        plan = BatchPlan(problems, smoother=smoother, nu1=nu1, nu2=1, flags=flags | capi.GMG_PROFILE)
        us = [torch.zeros_like(f) for f in fs]
        plan.solve(us, fs, rtol=1e-30, maxit=2)
        apart.append(plan.profile()["resid_restrict_coarse"]["launches"])  # (every level's)
        out.append([u.cpu().numpy() for u in us])
    # three sizes of 255 up, in at least the two cycles
    assert apart[0] <= apart[1] - 6
    for a, b in zip(*out):
        assert np.array_equal(a, b)
