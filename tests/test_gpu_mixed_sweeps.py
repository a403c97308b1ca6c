"""Mixed-precision plans of every sweep count reach the FP64 residual, small levels
included: three and more sweeps have no one-workgroup descent in 3D and take
the general passes there, with the same bits as a plan that has none at all."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,L,nu1,nu2", [(3, 6, 3, 1), (3, 7, 3, 3), (3, 6, 4, 2), (3, 5, 8, 0),
                                           (2, 8, 3, 3), (2, 10, 4, 1)])
def test_mixed_sweep_counts(dim, L, nu1, nu2):
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    f = wl.rhs_uniform(dim, (1 << L) - 1, seed=870 + L)
    fd = torch.from_numpy(f).cuda()
    out = []
    for flags in (0, capi.GMG_NO_FUSED_COARSE):
        plan = Plan(dim, L, nu1=nu1, nu2=nu2, precision="mixed", flags=flags)
        u = torch.zeros_like(fd)
        st, it, rel = plan.solve(u, fd, rtol=1e-9)
        assert st == 0
        out.append(u.cpu().numpy())
    assert np.array_equal(*out)
    assert oracle.norm2(oracle.residual(out[0], f)) <= 1e-9 * oracle.norm2(f)
