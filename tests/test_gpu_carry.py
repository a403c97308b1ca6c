"""Repeated cycles of red-black V(nu1 >= 2, nu2) solves leave out the red
half-sweep that the cycle before them ended with (its values are a fixed point
of that half-sweep): the same iterates bit for bit as the plain schedule, and
the oracle's solve to 1e-12 (1e-15 to 1e-14 from the order of the transfers'
sums, so 1e-12 leaves two orders of magnitude)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


def _mods():
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    return capi, Plan


def _dev(a):
    return torch.from_numpy(a).cuda()


def _solve(plan, f, **kw):
    u = torch.zeros_like(f)
    st, it, rel = plan.solve(u, f, **kw)
    return st, it, rel, u.cpu().numpy()


@pytest.mark.parametrize("dim,L,nu", [(2, 2, (2, 2)), (2, 7, (2, 2)), (2, 10, (3, 1)),
                                      (3, 2, (2, 1)), (3, 5, (2, 2)), (3, 6, (4, 2)),
                                      (3, 7, (2, 3)), (3, 7, (3, 3))])
@pytest.mark.parametrize("tune", [False, True])
def test_repeated_cycles_bitwise_and_oracle(dim, L, nu, tune):
    c, Plan = _mods()
    f = wl.rhs_uniform(dim, (1 << L) - 1, seed=301)
    fd = _dev(f)
    flags = c.GMG_AUTOTUNE if tune else 0
    kw = dict(rtol=1e-9, maxit=40)
    a = _solve(Plan(dim, L, nu1=nu[0], nu2=nu[1], flags=flags), fd, **kw)
    b = _solve(Plan(dim, L, nu1=nu[0], nu2=nu[1], flags=flags | c.GMG_NO_CROSS_CYCLE), fd, **kw)
    assert a[:2] == b[:2] and np.array_equal(a[3], b[3])
    assert abs(a[2] - b[2]) <= 1e-12 * b[2]  # the partial sums' order only
    u_ref, it_ref, _, st_ref, _ = oracle.solve(f, nu1=nu[0], nu2=nu[1], **kw)
    assert (a[0], a[1]) == (st_ref, it_ref)
    assert np.linalg.norm(a[3] - u_ref) <= 1e-12 * np.linalg.norm(u_ref)


@pytest.mark.parametrize("dim,L,nu1", [(3, 6, 2), (3, 7, 2), (2, 8, 2), (3, 6, 3)])
def test_repeated_cycles_every_tile_bitwise(dim, L, nu1):
    c, Plan = _mods()
    fd = _dev(wl.rhs_uniform(dim, (1 << L) - 1, seed=302))
    ref = _solve(Plan(dim, L, nu1=nu1, flags=c.GMG_NO_CROSS_CYCLE), fd, rtol=1e-6)
    ran = 0
    for flags in (0, c.GMG_NO_FUSED_RESTRICT):
        for v in range(c.lib().gmg_tile_variant_count(dim, 0, 3)):
            for tz in (0, 5, 16):
                plan = Plan(dim, L, nu1=nu1, flags=flags)
                plan.set_tile(0, 4, 1, 8)  # two sweeps per pass
                try:
                    plan.set_tile(0, 3, v, tz)
                except c.GmgError:
                    continue  # the tile does not run this form
                assert plan.get_tile(0, 2)[:2] == (3, v)
                got = _solve(plan, fd, rtol=1e-6)
                assert got[:2] == ref[:2] and np.array_equal(got[3], ref[3]), (flags, v, tz)
                ran += 1
    assert ran >= 6


def test_repeated_cycles_maxit_and_resume():
    c, Plan = _mods()
    f = wl.rhs_uniform(3, 31, seed=303)
    fd = _dev(f)
    plan = Plan(3, 5)
    full = _solve(plan, fd, rtol=1e-10)
    for maxit in (1, 2, 3):
        st, it, _, u = _solve(plan, fd, rtol=1e-10, maxit=maxit)
        want = np.zeros_like(f)
        for _ in range(maxit):
            want = oracle.vcycle(want, f, 2, 2)
        assert (st, it) == (1, maxit)
        assert np.linalg.norm(u - want) <= 1e-12 * np.linalg.norm(want)
    # an iterate that no cycle of this solve produced: the first cycle relaxes
    # every colour
    ud = torch.zeros_like(fd)
    plan.solve(ud, fd, rtol=1e-10, maxit=3)
    st, it, _ = plan.solve(ud, fd, rtol=1e-10, res0=oracle.norm2(f))
    assert (st, it) == (0, full[1] - 3) and np.array_equal(ud.cpu().numpy(), full[3])


@pytest.mark.parametrize("dim,L,inner", [(3, 6, 1), (3, 6, 4), (2, 8, 3)])
def test_mixed_inner_cycles_repeat_bitwise(dim, L, inner):
    c, Plan = _mods()
    f = wl.rhs_uniform(dim, (1 << L) - 1, seed=304)
    kw = dict(precision="mixed", inner_cycles=inner)
    a = _solve(Plan(dim, L, **kw), _dev(f), rtol=1e-9)
    b = _solve(Plan(dim, L, flags=c.GMG_NO_CROSS_CYCLE, **kw), _dev(f), rtol=1e-9)
    assert a[:2] == b[:2] and a[0] == 0 and np.array_equal(a[3], b[3])
