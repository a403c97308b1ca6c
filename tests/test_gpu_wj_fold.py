"""Jacobi pre-smoothing with the restriction folded into its last pass: the bits
of the two kernels, over the tiles, z-chunks (odd ones too) and data types."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu

NO_FUSED_RESTRICT = 0x40


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("dim,L,variant,tz", [
    (2, 8, 0, 0), (2, 8, 1, 7), (2, 10, 0, 64), (2, 11, 1, 2047),
    (3, 8, 0, 0), (3, 8, 0, 33), (3, 8, 1, 64), (3, 8, 2, 255), (3, 8, 2, 5)])
@pytest.mark.parametrize("nu1", [2, 3, 4])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_folded_restriction_same_bits(dim, L, variant, tz, nu1, prec):
    from paper_1208_4247_amd.solver import Plan

    m = (1 << L) - 1
    f = torch.from_numpy(wl.rhs_uniform(dim, m, seed=660 + L)).cuda()
    out = []
    for flags in (0, NO_FUSED_RESTRICT):
        plan = Plan(dim, L, nu1=nu1, nu2=1, smoother="wj", precision=prec, flags=flags)
        plan.set_tile(0, 2, variant, tz)
        u = torch.zeros_like(f)
        r = plan.solve(u, f, rtol=1e-30, maxit=3)
        v = torch.zeros_like(f)
        if prec == "fp64":
            plan.fmg(v, f)
        out.append((u.cpu().numpy(), v.cpu().numpy(), r))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("nu1", [1, 2, 4])
def test_batch_folds_with_the_same_bits(nu1):
    from paper_1208_4247_amd.solver import BatchPlan

    problems = [(2, 8), (2, 9), (2, 6), (3, 8), (3, 5), (2, 8), (3, 4), (2, 10)]
    fs = [torch.from_numpy(wl.rhs_uniform(d, (1 << L) - 1, seed=700 + i)).cuda()
          for i, (d, L) in enumerate(problems)]
    out = []
    for flags in (0, NO_FUSED_RESTRICT):
        plan = BatchPlan(problems, smoother="wj", nu1=nu1, nu2=1, flags=flags)
        us = [torch.zeros_like(f) for f in fs]
        plan.solve(us, fs, rtol=1e-30, maxit=3)
        out.append([u.cpu().numpy() for u in us])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
