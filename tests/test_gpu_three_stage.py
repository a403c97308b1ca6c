"""Which tile the three-stage level-0 pass runs: the plan's own choice, before
and after a solve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,L,nu1,prec", [
    (3, 8, 2, "fp64"), (3, 8, 2, "mixed"), (3, 8, 3, "fp64"), (3, 8, 4, "fp64"), (3, 6, 3, "fp64"),
    (2, 9, 3, "fp64"), (2, 9, 3, "mixed")])
def test_a_solve_leaves_the_default_choice(dim, L, nu1, prec):
    """With more than two pre-sweeps the pass never folds the restriction in, so
    its default is a tile that runs the plain form."""
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import Plan

    f = torch.from_numpy(wl.rhs_uniform(dim, (1 << L) - 1, seed=830)).cuda()
    got = []
    for flags in (0, capi.GMG_NO_CROSS_CYCLE):
        plan = Plan(dim, L, nu1=nu1, nu2=1, precision=prec, flags=flags)
        if not flags:
            before = plan.get_tile(0, 2)
        u = torch.zeros_like(f)
        plan.solve(u, f, rtol=1e-30, maxit=3)
        if not flags:
            assert plan.get_tile(0, 2) == before
            if dim == 3 and nu1 > 2:
                assert before[:2] == (3, 9)  # 36 x 24 pairs, the rule's plain tile
        got.append(u.cpu().numpy())
    assert np.array_equal(*got)
