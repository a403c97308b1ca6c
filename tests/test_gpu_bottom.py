"""The one-workgroup bottom kernel on every hierarchy it holds (2D 63^2 .. 1,
3D 15^3 .. 1), with every sweep count down to zero on either side and both
post-smoothing orders: V-cycles equal the oracle's to 1e-13 (the transfers' sums
have another order: a few eps per level)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


def _vcycle(u, f, nu1, nu2, forward):
    """The cycle from the oracle's pieces, with either post-smoothing order."""
    if u.size == 1:
        return f * 0.25 / (2 * u.ndim)
    u = oracle.rbgs(u, f, nu1)
    fc = oracle.restrict_fw(oracle.residual(u, f))
    u = oracle.prolong_add(_vcycle(np.zeros_like(fc), fc, nu1, nu2, forward), u)
    return oracle.rbgs(u, f, nu2, backward=not forward)


@pytest.mark.parametrize("dim,L", [(2, L) for L in range(2, 8)] + [(3, L) for L in range(2, 6)])
@pytest.mark.parametrize("nu", [(2, 2), (1, 1), (0, 2), (2, 0), (1, 3)])
@pytest.mark.parametrize("forward", [False, True])
def test_bottom_vcycle_matches_oracle(dim, L, nu, forward):
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    m = (1 << L) - 1
    f = wl.rhs_uniform(dim, m, seed=500 + L)
    fd = torch.from_numpy(f).cuda()
    plan = Plan(dim, L, nu1=nu[0], nu2=nu[1], flags=capi.GMG_POST_FORWARD if forward else 0)
    u = torch.zeros_like(fd)
    plan.vcycle(u, fd)
    want = _vcycle(np.zeros_like(f), f, nu[0], nu[1], forward)
    assert np.linalg.norm(u.cpu().numpy() - want) <= 1e-13 * np.linalg.norm(want)


@pytest.mark.parametrize("dim,L", [(2, L) for L in range(2, 8)] + [(3, L) for L in range(2, 6)])
@pytest.mark.parametrize("nu", [(2, 2), (1, 1), (0, 2), (3, 0)])
@pytest.mark.parametrize("kind", ["wj", "fmg", "wj_fmg"])
def test_bottom_jacobi_and_full_multigrid_match_oracle(dim, L, nu, kind):
    from paper_1208_4247_amd.solver import Plan

    m = (1 << L) - 1
    f = wl.rhs_uniform(dim, m, seed=520 + L)
    fd = torch.from_numpy(f).cuda()
    wj = kind.startswith("wj")
    plan = Plan(dim, L, nu1=nu[0], nu2=nu[1], smoother="wj" if wj else "rbgs")
    kw = dict(smoother=oracle.WJ if wj else oracle.RBGS, omega=2 * dim / (2 * dim + 1))
    u = torch.zeros_like(fd)
    if kind == "wj":
        plan.vcycle(u, fd)
        want = oracle.vcycle(np.zeros_like(f), f, nu[0], nu[1], **kw)
    else:
        plan.fmg(u, fd)
        want = oracle.fmg(f, nu[0], nu[1], **kw)
    assert np.linalg.norm(u.cpu().numpy() - want) <= 1e-13 * np.linalg.norm(want)


@pytest.mark.parametrize("dim,L", [(2, L) for L in range(2, 9)] + [(3, L) for L in range(2, 7)])
@pytest.mark.parametrize("nu", [(1, 1), (0, 2), (3, 0), (2, 3)])
@pytest.mark.parametrize("flags", [0, 0x8 | 0x100])  # GMG_POST_FORWARD, GMG_COARSE_RELAX
def test_paper_bottom_same_bits_as_kernel_per_step(dim, L, nu, flags):
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    m = (1 << L) - 1
    f = wl.rhs_uniform(dim, m, seed=560 + L)
    u0 = wl.rhs_uniform(dim, m, seed=580 + L)
    out = []
    for extra in (0, capi.GMG_NO_FUSED_COARSE):
        plan = Plan(dim, L, nu1=nu[0], nu2=nu[1], smoother="mcgs",
                    flags=flags | capi.GMG_FE_TRANSFER | extra)
        fd = torch.from_numpy(f).cuda()
        u = torch.from_numpy(u0).cuda()
        plan.vcycle(u, fd)
        v = torch.zeros_like(u)
        plan.fmg(v, fd)
        out.append((u.cpu().numpy(), v.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    if not flags:
        kw = dict(smoother=oracle.MCGS, variant=oracle.FE_TRANSFER)
        want = oracle.vcycle(u0, f, nu[0], nu[1], **kw)
        assert np.linalg.norm(out[0][0] - want) <= 1e-13 * np.linalg.norm(want)
